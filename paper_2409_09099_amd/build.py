"""Builds libsste.so (hand-written HIP kernels for gfx950 + the C ABI) in-tree with hipcc, and _marshal.so (the binding's native
argument marshalling, host code only) with g++.

Run as ``python -m paper_2409_09099_amd.build``.  There is one target architecture and one code
path; nothing is compiled at import time.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsste.so")
MARSHAL = os.path.join(HERE, "_marshal.so")

SOURCES = ["api.hip", "prune_pack.hip", "gemm_fwd.hip", "gemm_wgrad.hip", "gemm_wgrad_fused.hip", "gemm_dgrad.hip", "cast.hip"]

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-ffp-contract=off",           # the projection and the estimator specify every float32 rounding
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-Wno-unknown-warning-option",
]


def build_library(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass warns that it does not know the packed-fp32 feature: harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    return LIB


def build_marshal(verbose: bool = True) -> str:
    """The Python extension module next to the library; it gets the library's entry points at run time and does not link to it."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    for d in cpp_extension.include_paths("cuda") + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", d]
    cmd += [os.path.join(HERE, "ext", "marshal.cpp"), "-o", MARSHAL]
    for d in cpp_extension.library_paths("cuda"):
        cmd += ["-L" + d]
    cmd += ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout)
    if verbose and res.stdout.strip():
        print(res.stdout)
    return MARSHAL


if __name__ == "__main__":
    build_library()
    print("built", LIB)
    build_marshal()
    print("built", MARSHAL)
    sys.exit(0)
