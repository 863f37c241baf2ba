"""Builds libnoble.so (the HIP kernels and the C ABI) in-tree for gfx950, and
_noble_torch.so, the binding's calls on torch tensors (host code)."""

from __future__ import annotations

import os
import shutil
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libnoble.so")
BINDING = os.path.join(PKG, "_noble_torch.so")
SOURCES = ["noble_api.hip"]
HEADERS = ["noble_act.hpp", "noble_init.hpp", "noble_kernels.hpp", "noble_tiles.hpp", "noble_gemm.hpp", "noble_gemm_dma.hpp", "noble_gemm_tile.hpp", "noble_skinny.hpp", "noble_finish.hpp", "noble_gemm_f32.hpp", "noble_binding.h", "noble_torch.cpp"]

HIP_FLAGS = [
    "-O3",
    "-std=c++20",
    "--offload-arch=gfx950",
    "-fPIC",
    "-shared",
    "-munsafe-fp-atomics",
    # no packed-FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libnoble)")


def build(verbose: bool = False) -> str:
    """Compile libnoble.so; always recompiles.  Returns the library path."""
    tmp = LIB + ".tmp"
    cmd = [hipcc(), *HIP_FLAGS, "-I", INCLUDE, "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB)
    build_binding(verbose)
    return LIB


def build_binding(verbose: bool = False) -> str:
    """Compile _noble_torch.so (a CPython extension on torch's C++ headers)."""
    import torch
    root = os.path.dirname(torch.__file__)
    inc, tmp = os.path.join(root, "include"), BINDING + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", "-I", INCLUDE, "-isystem", inc,
           "-isystem", os.path.join(inc, "torch/csrc/api/include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "noble_torch.cpp"),
           "-L", os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python",
           "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed ({res.returncode}):\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, BINDING)
    return BINDING


if __name__ == "__main__":
    print(build(verbose=True))
