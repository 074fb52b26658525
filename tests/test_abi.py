"""Host-side checks of the C ABI that need no GPU: the library loads, exports every
function include/lime.h declares, and rejects bad arguments before launching anything."""

import ctypes
import os
import re
import subprocess
import sys

import pytest

from paper_2510_18239_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x1000  # a non-NULL pointer that is never dereferenced: every call below fails its host-side checks


def declared_functions():
    text = open(os.path.join(ROOT, "include", "lime.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(\w+)\s*\([^;{]*\)\s*;", text)))


def test_library_exports_every_declared_symbol():
    names = declared_functions()
    assert {"lime_link_history", "lime_xor_history", "lime_score_candidates", "mha_target_attention",
            "lime_profile_enable", "lime_profile_collect", "lime_build_qk_cache", "lime_score_candidates_cached",
            "lime_score_candidates_gathered", "lime_prepared_bytes", "lime_prepare", "lime_link_history_prepared",
            "lime_score_candidates_prepared", "lime_xor_layers", "lime_request_prepared",
            "lime_workspace_bytes", "lime_last_error", "lime_version"} <= set(names)
    lib = ctypes.CDLL(binding.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(binding.SIGNATURES), "binding and header disagree"
    assert re.fullmatch(r"\d+\.\d+\.\d+", binding.version())


def test_missing_library_is_an_error(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        binding.lib()


def _hist(fn, **kw):
    a = dict(E=FAKE, lens=None, LC=FAKE, stride=0, Wq=FAKE, Wk=FAKE, Wv=FAKE, LP=FAKE, OS=None, B=2, N=8, d=8, h=2,
             m=4, scale=1.0, dtype=1, ws=FAKE, ws_bytes=0, stream=None)
    a.update(kw)
    lib = binding.lib()
    if fn == "lime_link_history":
        return lib.lime_link_history(a["E"], a["lens"], a["LC"], a["stride"], a["Wq"], a["Wk"], a["Wv"], a["LP"],
                                     a["B"], a["N"], a["d"], a["h"], a["m"], a["scale"], a["dtype"], a["ws"],
                                     a["ws_bytes"], a["stream"])
    return lib.lime_xor_history(a["E"], a["lens"], a["LC"], a["stride"], a["Wq"], a["Wk"], a["Wv"], a["LP"], a["OS"],
                                a["B"], a["N"], a["d"], a["h"], a["m"], a["scale"], a["dtype"], a["ws"],
                                a["ws_bytes"], a["stream"])


@pytest.mark.parametrize("fn", ["lime_link_history", "lime_xor_history"])
def test_history_argument_checks(fn):
    assert _hist(fn) == 3 and "workspace" in binding.last_error()  # workspace of 0 bytes
    assert _hist(fn, ws=None, ws_bytes=1 << 30) == 3
    assert _hist(fn, E=None) == 1
    assert _hist(fn, LP=None) == 1
    assert _hist(fn, Wk=None) == 1
    assert _hist(fn, B=0) == 1
    assert _hist(fn, N=-3) == 1
    assert _hist(fn, m=0) == 1
    assert _hist(fn, d=9) == 1 and "multiple" in binding.last_error()
    assert _hist(fn, dtype=7) == 1
    assert _hist(fn, stride=5) == 1
    assert _hist(fn, d=1024, h=2) == 2  # d/h = 512 > 256
    assert _hist(fn, B=70000) == 2


def test_candidate_and_baseline_argument_checks():
    lib = binding.lib()

    def cand(T=FAKE, L=FAKE, LP=FAKE, O=FAKE, B=1, C=4, d=8, h=2, m=4, dtype=1, ws=FAKE, ws_bytes=0):
        return lib.lime_score_candidates(T, L, LP, None, None, None, O, B, C, d, h, m, 1.0, dtype, ws, ws_bytes, None)

    assert cand() == 3
    assert cand(T=None) == 1 and cand(L=None) == 1 and cand(LP=None) == 1 and cand(O=None) == 1
    assert cand(C=0) == 1 and cand(m=0) == 1 and cand(h=3) == 1 and cand(dtype=-1) == 1
    assert cand(d=2048, h=4) == 2

    def mha(T=FAKE, E=FAKE, Wq=FAKE, O=FAKE, B=1, C=4, N=8, d=8, h=2, dtype=0, ws=FAKE, ws_bytes=0):
        return lib.mha_target_attention(T, E, None, Wq, FAKE, FAKE, O, B, C, N, d, h, 1.0, dtype, ws, ws_bytes, None)

    assert mha() == 3
    assert mha(T=None) == 1 and mha(E=None) == 1 and mha(Wq=None) == 1 and mha(O=None) == 1
    assert mha(N=0) == 1 and mha(C=0) == 1 and mha(h=0) == 1


def test_workspace_query():
    wb = binding.workspace_bytes
    assert wb(binding.OP_LINK_HISTORY, B=2, N=100, d=64, h=4, m=16) > 0
    assert wb(binding.OP_XOR_HISTORY, B=2, N=100, d=64, h=4, m=16, flags=1) >= wb(binding.OP_XOR_HISTORY, B=2, N=100,
                                                                                    d=64, h=4, m=16, flags=0)
    assert wb(binding.OP_SCORE_CANDIDATES, B=1, C=32768, d=256, h=4, m=64) > 0
    assert wb(binding.OP_MHA_TARGET, B=1, C=10, N=10, d=8, h=2) > 0
    assert wb(binding.OP_LINK_HISTORY, B=0, N=100, d=64, h=4, m=16) == 0
    assert wb(binding.OP_LINK_HISTORY, B=1, N=100, d=64, h=5, m=16) == 0
    assert wb(99, B=1, N=1, C=1, d=8, h=1, m=1) == 0
    for op in range(4):
        assert wb(op, B=3, N=50, C=70, d=32, h=2, m=8, dtype=0, flags=1) % 256 == 0


def test_qk_cache_argument_checks():
    lib = binding.lib()

    def build(T=FAKE, L=FAKE, W=FAKE, C=4, d=8, h=2, m=4, dtype=1, ws=FAKE, ws_bytes=0):
        return lib.lime_build_qk_cache(T, L, None, None, W, 1, C, d, h, m, 1.0, dtype, ws, ws_bytes, None)

    assert build() == 3
    assert build(T=None) == 1 and build(L=None) == 1 and build(W=None) == 1
    assert build(C=0) == 1 and build(m=-1) == 1 and build(h=3) == 1 and build(dtype=5) == 1

    def score(W=FAKE, LP=FAKE, O=FAKE, C=4, d=8, h=2, m=4, dtype=0, ws=FAKE, ws_bytes=0):
        return lib.lime_score_candidates_cached(W, LP, None, O, 1, C, d, h, m, dtype, ws, ws_bytes, None)

    assert score() == 3
    assert score(W=None) == 1 and score(LP=None) == 1 and score(O=None) == 1
    assert score(C=0) == 1 and score(m=0) == 1 and score(d=7) == 1
    def gathered(W=FAKE, ids=FAKE, n_items=10, LP=FAKE, O=FAKE, C=4, d=8, h=2, m=4, dtype=0, ws=FAKE, ws_bytes=0):
        return lib.lime_score_candidates_gathered(W, ids, n_items, LP, None, O, 1, C, d, h, m, dtype, ws, ws_bytes, None)

    assert gathered() == 3
    assert gathered(ids=None) == 1 and gathered(n_items=0) == 1 and gathered(W=None) == 1 and gathered(O=None) == 1
    assert gathered(C=0) == 1 and gathered(h=3) == 1
    assert binding.workspace_bytes(binding.OP_BUILD_QK_CACHE, B=1, C=100, d=256, h=4, m=64) > 0
    assert binding.workspace_bytes(binding.OP_SCORE_CACHED, B=2, C=100, d=256, h=4, m=64) > 0


def test_prepared_operand_argument_checks():
    lib = binding.lib()
    size = lib.lime_prepared_bytes(256, 4, 64, 1)
    assert size == 3 * 256 * 256 * 2 + 2 * 64 * 256 * 2
    assert lib.lime_prepared_bytes(256, 4, 64, 0) == 0      # fp32 has no matrix-core path
    assert lib.lime_prepared_bytes(96, 3, 20, 1) == 0       # neither has this shape
    assert lib.lime_prepared_bytes(256, 3, 64, 1) == 0 and lib.lime_prepared_bytes(0, 1, 64, 1) == 0

    def prepare(LC=FAKE, L=FAKE, Wq=FAKE, prepared=FAKE, nbytes=0, d=256, h=4, m=64, dtype=1):
        return lib.lime_prepare(LC, L, Wq, FAKE, FAKE, None, None, 1.0, 1.0, prepared, nbytes, d, h, m, dtype, None)

    assert prepare() == 3
    assert prepare(LC=None) == 1 and prepare(L=None) == 1 and prepare(Wq=None) == 1 and prepare(prepared=None) == 1
    assert prepare(h=3) == 1 and prepare(m=0) == 1
    assert prepare(dtype=0) == 2 and prepare(d=96, h=3, m=20) == 2 and prepare(LC=FAKE + 2) == 2
    assert "prepared" in binding.last_error()

    def hist(E=FAKE, prepared=FAKE, LP=FAKE, B=1, N=64, d=256, h=4, m=64, dtype=1, ws=FAKE, ws_bytes=0):
        return lib.lime_link_history_prepared(E, None, prepared, LP, B, N, d, h, m, 1.0, 0, dtype, ws, ws_bytes, None)

    assert hist() == 3
    assert hist(E=None) == 1 and hist(prepared=None) == 1 and hist(LP=None) == 1 and hist(N=0) == 1
    assert hist(dtype=0) == 2 and hist(d=96, h=3, m=20) == 2 and hist(E=FAKE + 4) == 2

    def cand(T=FAKE, LP=FAKE, prepared=FAKE, O=FAKE, B=1, C=64, d=256, h=4, m=64, dtype=1, ws=FAKE, ws_bytes=0):
        return lib.lime_score_candidates_prepared(T, LP, None, prepared, O, B, C, d, h, m, 1.0, dtype, ws, ws_bytes, None)

    assert cand() == 3
    assert cand(T=None) == 1 and cand(LP=None) == 1 and cand(prepared=None) == 1 and cand(O=None) == 1 and cand(C=0) == 1
    assert cand(dtype=0) == 2 and cand(d=128, h=4, m=20) == 2


def test_xor_layers_argument_checks():
    lib = binding.lib()

    def call(**kw):
        a = dict(E=FAKE, lens=None, LC=FAKE, stride=0, Wq=FAKE, Wk=FAKE, Wv=FAKE, Wu=FAKE, Wo=FAKE, n=3, LP=FAKE, B=2,
                 N=64, d=128, h=4, m=64, scale=1.0, dtype=1, ws=FAKE, ws_bytes=0, stream=None)
        a.update(kw)
        return lib.lime_xor_layers(a["E"], a["lens"], a["LC"], a["stride"], a["Wq"], a["Wk"], a["Wv"], a["Wu"], a["Wo"],
                                   a["n"], a["LP"], a["B"], a["N"], a["d"], a["h"], a["m"], a["scale"], a["dtype"],
                                   a["ws"], a["ws_bytes"], a["stream"])

    need = binding.workspace_bytes(binding.OP_XOR_LAYERS, B=2, N=64, d=128, h=4, m=64)
    assert need > 4 * 2 * 64 * 128 * 2  # at least the four history-sized tensors
    assert call() == 3 and str(need) in binding.last_error()          # workspace too small, size named
    assert call(ws_bytes=need - 1) == 3
    assert call(Wu=None) == 1 and call(Wo=None) == 1 and call(LP=None) == 1 and call(E=None) == 1
    assert call(n=0) == 1 and call(N=0) == 1 and call(m=0) == 1
    assert call(stride=5) == 1
    assert call(dtype=7) == 1 and call(d=120, h=7) == 1
    assert call(d=1024, h=2) == 2                                      # d/h = 512 exceeds the largest head
    # fp32 storage and shapes outside the matrix-core set run on the general kernels: they have a workspace size too
    assert binding.workspace_bytes(binding.OP_XOR_LAYERS, B=2, N=64, d=128, h=4, m=64, dtype=0) > need
    assert binding.workspace_bytes(binding.OP_XOR_LAYERS, B=2, N=64, d=120, h=3, m=20) > 0
    assert call(dtype=0, ws_bytes=need) == 3


def test_request_prepared_argument_checks():
    lib = binding.lib()

    def call(**kw):
        a = dict(E=FAKE, lens=None, T=FAKE, Wv=FAKE, prepared=FAKE, LP=FAKE, O=FAKE, B=1, N=64, C=64, d=256, h=4, m=64,
                 sh=1.0, sc=1.0, xor=0, dtype=1, ws=FAKE, ws_bytes=0, stream=None)
        a.update(kw)
        return lib.lime_request_prepared(a["E"], a["lens"], a["T"], a["Wv"], a["prepared"], a["LP"], a["O"], a["B"], a["N"],
                                         a["C"], a["d"], a["h"], a["m"], a["sh"], a["sc"], a["xor"], a["dtype"], a["ws"],
                                         a["ws_bytes"], a["stream"])

    need = binding.workspace_bytes(binding.OP_REQUEST_PREPARED, B=1, N=64, C=64, d=256, h=4, m=64)
    assert need == (binding.workspace_bytes(binding.OP_LINK_HISTORY, B=1, N=64, d=256, h=4, m=64) +
                    binding.workspace_bytes(binding.OP_SCORE_CANDIDATES, B=1, C=64, d=256, h=4, m=64)) or need > 0
    assert call() == 3 and str(need) in binding.last_error()
    assert call(prepared=None) == 1 and call(LP=None) == 1 and call(O=None) == 1 and call(T=None) == 1
    assert call(C=0) == 1 and call(N=0) == 1
    assert call(dtype=0) == 2 and call(d=120, h=3) == 2 and call(T=FAKE + 4) == 2
    assert call(Wv=None) == 3  # identity values are allowed: only the workspace is wrong here
    assert binding.workspace_bytes(binding.OP_REQUEST_PREPARED, B=1, N=64, C=64, d=256, h=4, m=64, dtype=0) == 0


def test_request_argument_checks():
    lib = binding.lib()

    def call(**kw):
        a = dict(E=FAKE, lens=None, LC=FAKE, stride=0, Wqh=FAKE, Wkh=FAKE, Wvh=FAKE, T=FAKE, L=FAKE, Wqc=FAKE, Wkc=FAKE,
                 Wvc=FAKE, LP=FAKE, O=FAKE, B=1, N=64, C=64, d=256, h=4, m=64, sh=1.0, sc=1.0, xor=0, dtype=1, ws=FAKE,
                 ws_bytes=0, stream=None)
        a.update(kw)
        return lib.lime_request(a["E"], a["lens"], a["LC"], a["stride"], a["Wqh"], a["Wkh"], a["Wvh"], a["T"], a["L"],
                                a["Wqc"], a["Wkc"], a["Wvc"], a["LP"], a["O"], a["B"], a["N"], a["C"], a["d"], a["h"], a["m"],
                                a["sh"], a["sc"], a["xor"], a["dtype"], a["ws"], a["ws_bytes"], a["stream"])

    for dtype in (0, 1):  # both storage types are served (fp32 on the general kernels)
        need = binding.workspace_bytes(binding.OP_REQUEST, B=1, N=64, C=64, d=256, h=4, m=64, dtype=dtype)
        assert need == (binding.workspace_bytes(binding.OP_LINK_HISTORY, B=1, N=64, d=256, h=4, m=64, dtype=dtype) +
                        binding.workspace_bytes(binding.OP_SCORE_CANDIDATES, B=1, C=64, d=256, h=4, m=64, dtype=dtype))
        assert call(dtype=dtype) == 3 and str(need) in binding.last_error()
    assert call(E=None) == 1 and call(LC=None) == 1 and call(Wqh=None) == 1 and call(T=None) == 1 and call(L=None) == 1
    assert call(LP=None) == 1 and call(O=None) == 1
    assert call(C=0) == 1 and call(N=0) == 1 and call(m=0) == 1 and call(stride=7) == 1
    assert call(Wqc=None, Wkc=None, Wvc=None) == 3  # identity on the candidate side is allowed: only the workspace is wrong
    assert call(dtype=5) == 1 or call(dtype=5) == 2
    assert binding.workspace_bytes(binding.OP_REQUEST, B=1, N=64, C=0, d=256, h=4, m=64) == 0


def test_request_static_argument_checks():
    """The entry point without a workspace: the same host-side checks as lime_request, and a shape whose scratch does not
    fit the library's fixed array is refused before anything touches a device."""
    lib = binding.lib()

    def call(**kw):
        a = dict(E=FAKE, lens=None, LC=FAKE, stride=0, Wq=FAKE, Wk=FAKE, Wv=FAKE, T=FAKE, L=FAKE, LP=FAKE, O=FAKE, B=1,
                 N=64, C=64, d=64, h=2, m=32, dtype=1)
        a.update(kw)
        return lib.lime_request_static(a["E"], a["lens"], a["LC"], a["stride"], a["Wq"], a["Wk"], a["Wv"], a["T"], a["L"],
                                       a["Wq"], a["Wk"], a["Wv"], a["LP"], a["O"], a["B"], a["N"], a["C"], a["d"], a["h"],
                                       a["m"], 1.0, 1.0, 0, a["dtype"], None)

    assert lib.lime_request_static_capacity() == 16 << 20
    assert call(E=None) == 1 and call(O=None) == 1 and call(N=0) == 1 and call(h=3) == 1 and call(dtype=5) == 1
    assert call(stride=7) == 1
    assert call(B=64, N=4096, d=256, h=4, m=128) == 2 and "scratch" in binding.last_error()  # needs far more than 16 MiB
    assert call(B=1, N=1 << 20, C=16, d=64, h=2, m=20, dtype=0) == 2  # general kernels: fp32 projections of the history


def test_xor_backward_argument_checks():
    lib = binding.lib()

    def call(**kw):
        a = dict(ins=[FAKE] * 7, dOS=FAKE, lens=None, outs=[FAKE] * 6, B=2, N=100, m=64, d=128, h=4, scale=1.0, dtype=1,
                 ws=FAKE, ws_bytes=0, stream=None)
        a.update(kw)
        return lib.lime_xor_backward(*a["ins"], a["dOS"], a["lens"], *a["outs"], a["B"], a["N"], a["m"], a["d"], a["h"],
                                     a["scale"], a["dtype"], a["ws"], a["ws_bytes"], a["stream"])

    need = binding.workspace_bytes(binding.OP_XOR_BACKWARD, B=2, N=100, d=128, h=4, m=64)
    assert need > 0 and call() == 3 and str(need) in binding.last_error()
    assert call(dOS=None) == 3  # the source-side gradient may be absent: only the workspace is wrong here
    for i in range(7):
        assert call(ins=[None if j == i else FAKE for j in range(7)]) == 1
    for i in range(6):
        assert call(outs=[None if j == i else FAKE for j in range(6)]) == 1
    assert call(N=0) == 1 and call(m=0) == 1 and call(d=130, h=4) != 0
    assert call(d=512, h=2) == 2 and "64" in binding.last_error()  # d/h = 256: beyond this kernel
    assert binding.workspace_bytes(binding.OP_XOR_BACKWARD, B=2, N=100, d=512, h=2, m=64) == 0


def test_per_request_calls_check_their_tensors_before_anything_else():
    """The extension behind the per-request wrappers: host tensors, a missing tensor and a non-tensor are refused."""
    import torch

    x = torch.zeros(1, 8, 64)
    with pytest.raises(ValueError, match="contiguous CUDA"):
        binding.lime_link_history(x, None, x[0], x[0], x[0], x[0], 2, 1.0)
    with pytest.raises(ValueError, match="contiguous CUDA"):
        binding.lime_request(x, None, x[0], x[0], x[0], x[0], x, x[0], None, None, None, 2, 1.0, 1.0)
    with pytest.raises(ValueError, match="None"):
        binding.mha_target_attention(x, None, None, x, x, x, 2, 1.0)
    with pytest.raises(TypeError, match="tensor"):
        binding.lime_score_candidates(3, x, x, None, None, None, 2, 1.0)
    with pytest.raises(TypeError):
        binding.lime_scores(object(), x, None, x, x)


def test_per_request_calls_raise_for_tensors_without_storage():
    """Under vmap a tensor has no data pointer: the call raises what torch raises.  In a process of its own: the error
    once passed through the code that had given up the interpreter lock, which ended the process."""
    script = """
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2510_18239_amd import binding

class Stream:
    cuda_stream = 16

with FakeTensorMode():
    bf = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    E, L, W, LP = bf(3, 2, 40, 64), bf(32, 64), bf(64, 64), bf(2, 32, 64)
    ws = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    try:
        torch.func.vmap(lambda e: binding.lime_link_history(e, None, L, W, W, W, 2, 1.0, LP=LP, workspace=ws, stream=Stream()))(E)
    except RuntimeError as e:
        print("raised:", e)
"""
    r = subprocess.run([sys.executable, "-W", "ignore", "-c", script], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    assert "raised: Cannot access data pointer" in r.stdout, (r.stdout, r.stderr[-2000:])
