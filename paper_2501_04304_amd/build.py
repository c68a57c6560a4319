"""Build libdgq.so (HIP kernels + C ABI) for gfx950 with hipcc, and _hot.so, the native side of the Python
binding's hot calls, with g++; both in-tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdgq.so")
HOT = os.path.join(HERE, "_hot.so")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",  # every fused multiply-add in the kernels is written as fmaf
    # packed fp32 instructions stay disabled on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    # the direct-to-LDS loads set M0 inside their asm statement and say so in the clobber
    # list; clang warns about every reserved register named there
    "-Wno-inline-asm",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_binding(verbose: bool = False) -> str:
    """Host code only: torch's and Python's headers, linked against the library built beside it."""
    import sysconfig

    from torch.utils import cpp_extension
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",  # what the ROCm build of torch's headers expects
           "-I", os.path.join(ROOT, "include")]
    for d in cpp_extension.include_paths("cuda") + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", d]
    cmd += ["-o", HOT, os.path.join(CSRC, "binding.cpp")]
    for d in cpp_extension.library_paths("cuda"):
        cmd += ["-L" + d]
    cmd += ["-L" + HERE, "-Wl,-rpath,$ORIGIN", "-l:libdgq.so", "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return HOT


def build(verbose: bool = False, extra=()) -> str:
    cmd = ["hipcc", *FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           "-o", LIB, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    build_binding(verbose)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
    print("built", LIB)
