"""Build libdora.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2609_34325_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
import warnings

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libdora.so")
# Measurement helper for bench.py (sustained MFMA rate); not part of the boundary.
CALIB_LIB = os.path.join(PKG, "libdora_calibrate.so")
CALIB_SOURCES = ["calibrate.hip"]
SOURCES = ["select_pack.hip", "varlen_attn.hip", "actor_decode.hip", "pl_sample.hip", "lc1_readout.hip", "flops.hip"]
# Native marshalling of the Python binding (host code only).
HOST_LIB = os.path.join(PKG, "_host_call.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-Wall",
    "-Wno-unused-function",
    # Keep the compiler from forming packed-fp32 VALU ops (v_pk_*_f32).
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # Queue tickets are taken by one lane; keep the atomic as written so its
    # result is not broadcast to scalar registers (and waited on) at issue.
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    # The machine scheduler's iterative ILP strategy interleaves the softmax
    # VALU work with the matrix and LDS instructions better than the default
    # occupancy-driven one (DeiT-B attention 51.8 -> 49.1 us, select/pack
    # about 0.6 us faster; no VGPR spills).
    "-mllvm", "-amdgpu-sched-strategy=iterative-ilp",
    "-I", INCLUDE,
]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    path = os.path.join(rocm, "bin", "hipcc")
    return path if os.path.exists(path) else "hipcc"


def build(verbose: bool = False) -> str:
    _build_one(SOURCES, LIB, verbose)
    _build_one(CALIB_SOURCES, CALIB_LIB, verbose)
    _build_host(verbose)
    return LIB


def _build_host(verbose: bool) -> None:
    """Needs a host compiler and torch's C++ headers; without them the binding
    goes through ctypes."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    inc = os.path.join(root, "include")
    tmp = HOST_LIB + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", INCLUDE, "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "host_call.cpp"),
           "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10",
           "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
        failed = res.stdout + res.stderr if res.returncode != 0 else None
    except OSError as e:  # no such compiler
        failed = str(e)
    if failed is None:
        os.replace(tmp, HOST_LIB)
        return
    for path in (tmp, HOST_LIB):  # one of an earlier build may not fit the library's present arguments
        if os.path.exists(path):
            os.remove(path)
    warnings.warn("the native marshalling was not built, calls will go through ctypes:\n" + failed)


def _build_one(sources, lib: str, verbose: bool) -> None:
    srcs = [os.path.join(CSRC, s) for s in sources]
    tmp = lib + ".tmp%d" % os.getpid()
    cmd = [hipcc(), *HIPCC_FLAGS, *srcs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # The host pass does not know the packed-fp32 feature and says so; that is harmless.
    noise = "'-packed-fp32-ops' is not a recognized feature for this target"
    msgs = [l for l in (res.stdout + res.stderr).splitlines() if noise not in l]
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + "\n".join(msgs))
    if verbose and msgs:
        print("\n".join(msgs))
    os.replace(tmp, lib)


if __name__ == "__main__":
    print(build(verbose=True))
