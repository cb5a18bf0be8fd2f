"""Builds libaspd.so (HIP, gfx950; hipcc) and the binding's _pycalls.so (host code; g++, the headers of Python and torch) in-tree.
`python -m paper_2508_08895_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libaspd.so")
CALLS = os.path.join(HERE, "_pycalls.so")
SOURCES = ["aspd_meta.hip", "aspd_seq_meta.hip", "aspd_plan.hip", "aspd_attn.hip", "aspd_rope.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def build(verbose: bool = False, extra=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, *extra, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    build_calls(verbose)
    return LIB


def build_calls(verbose: bool = False) -> str:
    """The compiled half of the binding, against the libraries of the torch it runs beside (libaspd.so it is handed)."""
    import torch
    from torch.utils.cpp_extension import include_paths
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    dirs = [*include_paths(), os.path.join(rocm, "include"), sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[x for d in dirs for x in ("-isystem" if d != dirs[-1] else "-I", d)],
           os.path.join(CSRC, "aspd_pycalls.cpp"), "-o", CALLS, "-L", torch_lib, "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return CALLS


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
    print(LIB)
