"""Builds the HIP library (gfx950) in-tree, paper_2510_18239_amd/liblime_hip.so, and the extension with the binding's
per-request calls, paper_2510_18239_amd/_lime_torch.so (host code only)."""

from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblime_hip.so")
OBJ_DIR = os.path.join(HERE, "_build")
NATIVE_SRC = os.path.join(CSRC, "host", "torch_calls.cpp")
NATIVE = os.path.join(HERE, "_lime_torch.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # accumulators of MFMA chains are consumed by vector-ALU code right away: keep them in VGPRs
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    "-Wall", "-Wno-unused-function",
]


def sources() -> list[str]:
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str, obj_dir: str = OBJ_DIR, defines: tuple = ()) -> str:
    obj = os.path.join(obj_dir, os.path.basename(src)[:-4] + ".o")
    cmd = ["hipcc", *HIPCC_FLAGS, *[f"-D{d}" for d in defines], "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    noise = "is not a recognized feature for this target"
    warn = "\n".join(l for l in r.stderr.splitlines() if l.strip() and noise not in l)
    if warn:
        print(warn)
    return obj


def build_library(jobs: int = 8, lib: str = LIB, defines: tuple = ()) -> str:
    """Compile every csrc/*.hip for gfx950 and link the shared library.  Always recompiles.
    ``lib`` / ``defines``: another output path and preprocessor definitions (for comparing variants of a kernel)."""
    obj_dir = OBJ_DIR if lib == LIB else lib + ".objs"
    os.makedirs(obj_dir, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda src: _compile(src, obj_dir, defines), sources()))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return lib


def build_native() -> str:
    """Compile and link the binding's extension against torch and the library beside it (built before)."""
    import torch

    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *[x for d in include for x in ("-isystem", d)],
           NATIVE_SRC, "-o", NATIVE, "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-ltorch_hip", "-lc10",
           "-lc10_hip", "-L" + HERE, "-llime_hip", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for {NATIVE_SRC}:\n{r.stdout}\n{r.stderr}")
    return NATIVE


if __name__ == "__main__":
    print(build_library())
    print(build_native())
