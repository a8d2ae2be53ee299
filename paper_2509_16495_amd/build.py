"""Builds libshiftattn.so (HIP kernels + C ABI) in-tree for gfx950 with hipcc, and _calls.so (the Python binding's calls)
with g++ against the installed torch."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libshiftattn.so")
CALLS = os.path.join(HERE, "_calls.so")
SOURCES = ["api.hip", "layout_kernels.hip", "attn_generic.hip", "decode_mfma.hip", "prefill_mfma.hip", "prefill_mfma64.hip", "prefill_f32.hip", "ceilings.hip", "proj_gemm.hip", "proj_stream.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC", "-shared", "-fno-gpu-rdc",
    # packed fp32 VALU forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build_library(verbose: bool = False, extra: list[str] | None = None) -> str:
    cmd = ["hipcc", *FLAGS, *(extra or []), "-o", LIB, *[os.path.join(CSRC, s) for s in SOURCES]]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd, cwd=CSRC)
    build_calls(verbose)
    return LIB


def build_calls(verbose: bool = False) -> str:
    import sysconfig
    import torch.utils.cpp_extension as ext
    includes = [os.path.join(os.path.dirname(HERE), "include"), *ext.include_paths(), os.path.join(ext.ROCM_HOME or "/opt/rocm", "include"),
                sysconfig.get_paths()["include"]]
    libs = [a for d in ext.library_paths() for a in ("-L" + d, "-Wl,-rpath," + d)]
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", *["-I" + d for d in includes],
           os.path.join(CSRC, "python_calls.cpp"), "-o", CALLS, *libs, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd, cwd=CSRC)
    return CALLS


if __name__ == "__main__":
    build_library(verbose=True, extra=sys.argv[1:])
