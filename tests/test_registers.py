"""The compiler's registers for kernels that have lost speed by needing more: instances whose operands fill the register file, at
the most that they may take.  (Built for the device alone, a few instances at a time.)"""

import os
import re
import subprocess

import pytest

from paper_2510_18239_amd import build


def _resources(tmp_path, text):
    src = tmp_path / "t.hip"
    src.write_text(text)
    cmd = ["hipcc", *build.HIPCC_FLAGS, "--cuda-device-only", "-c", str(src), "-o", os.devnull, "-I", build.CSRC, "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    number = lambda name, block: int(re.search(name + r"[^:]*: (\d+)", block).group(1))  # noqa: E731
    return [{"name": b.split()[0], "vgprs": number(" VGPRs", b), "spill": number("VGPRs Spill", b), "waves": number("Occupancy", b)}
            for b in r.stderr.split("Function Name: ")[1:]]


@pytest.mark.parametrize("m,h,tiles,heads,raw,spill,waves", [
    (128, 8, 2, 4, False, 19, 2), (128, 8, 4, 1, False, 17, 2), (96, 8, 2, 4, False, 0, 2), (96, 8, 4, 1, False, 0, 2), (96, 8, 4, 1, True, 0, 2),
    (128, 4, 2, 4, False, 0, 2), (128, 1, 4, 1, False, 0, 3), (96, 2, 4, 2, False, 0, 3), (96, 2, 4, 1, True, 0, 3),
])
def test_history_kernel(tmp_path, m, h, tiles, heads, raw, spill, waves):
    args = "RawArgs" if raw else "PackedArgs"
    got, = _resources(tmp_path, f"""
#include "history_body.hpp"
namespace lime {{ namespace {{
template __global__ void links_over_history_kernel<32, {m}, {h}, kPhiSoftmax, {heads}, {tiles}, {str(raw).lower()}>(HistArgs, {args});
}} }}""")
    assert got["spill"] <= spill and got["waves"] >= waves, got


# (the rule that counts a compute unit's workgroups takes it that so many waves fit)
@pytest.mark.parametrize("dh,m,h,waves", [(64, 64, 1, 3), (32, 32, 2, 3), (32, 64, 2, 3), (32, 128, 4, 2)])
def test_history_kernel_on_raw_operands(tmp_path, dh, m, h, waves):
    got, = _resources(tmp_path, f"""
#include "history_body.hpp"
namespace lime {{ namespace {{
static_assert(HistShape<{dh}, {m}, {h}, 1, tiles_per_step({dh}, {h}, kShort), true>::kWavesPerSimd == {waves});
template __global__ void links_over_history_kernel<{dh}, {m}, {h}, kPhiSoftmax, 1, tiles_per_step({dh}, {h}, kShort), true>(HistArgs, RawArgs);
}} }}""")
    assert got["spill"] == 0 and got["waves"] >= waves, got


@pytest.mark.parametrize("phi,weights,norm,spill", [("kPhiSilu", "false", "false", 0), ("kPhiSoftmax", "false", "false", 0),
                                                    ("kPhiSoftmax", "true", "false", 0), ("kPhiSoftmax", "false", "true", 2)])
def test_rows_over_128_links(tmp_path, phi, weights, norm, spill):
    """d = 256, four heads: the stationary operands are most of the registers."""
    kernels = open(os.path.join(build.CSRC, "mfma_candidates.hip")).read()
    kernels = kernels[: kernels.index("hipError_t launch_form")]  # without the launches of every instance
    kernels = kernels[: kernels.rindex("template <")]
    got, = _resources(tmp_path, kernels + f"""
template __global__ void queries_over_links_kernel<64, 128, 4, {phi}, {weights}, false, {norm}>(MainArgs);
}} }}""")
    assert got["spill"] <= spill, got
