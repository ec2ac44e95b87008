"""Build libssmq.so (the HIP kernels and the C ABI) for gfx950 with hipcc, and the
CPython module that marshals torch tensors to it (_native.so) with g++.

Floating-point flags matter for parity: no contraction (every product and sum
is rounded where the source says), IEEE denormals, correctly rounded fp32
division, and no packed-fp32 instructions.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIBRARY = os.path.join(PKG, "libssmq.so")
NATIVE = os.path.join(PKG, "_native.so")
NATIVE_SOURCE = "ssmq_native.cpp"
SOURCES = ["ssmq_kernels.hip", "ssmq_abi.cpp"]
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-gpu-flush-denormals-to-zero",
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libssmq.so)")


def build(verbose: bool = False) -> str:
    """Compile every source into libssmq.so and the module beside it; returns the
    library path. Without the module (no g++, no torch headers) every call still works,
    through ctypes: its failure is reported, and no older one is left."""
    tmp = LIBRARY + ".tmp"
    cmd = [hipcc(), *HIPCC_FLAGS, "-I", INCLUDE, "-I", CSRC, "-o", tmp,
           *[os.path.join(CSRC, s) for s in SOURCES]]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIBRARY)
    if os.path.exists(NATIVE):
        os.remove(NATIVE)
    try:
        build_native(verbose)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        print(f"warning: {NATIVE} was not built ({e}); calls go through ctypes", file=sys.stderr, flush=True)
    return LIBRARY


def build_native(verbose: bool = False) -> str:
    """Compile the CPython module against torch's headers and libssmq.so."""
    import torch

    base = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(hipcc()))
    tmp = NATIVE + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DSSMQ_TORCH_VERSION="{torch.__version__}"',
           "-I", INCLUDE, "-isystem", sysconfig.get_paths()["include"],
           "-isystem", os.path.join(base, "include"), "-isystem", os.path.join(rocm, "include"),
           os.path.join(CSRC, NATIVE_SOURCE), "-o", tmp, "-L", PKG, "-lssmq",
           "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
           "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, NATIVE)
    return NATIVE


if __name__ == "__main__":
    print(build(verbose=True))
