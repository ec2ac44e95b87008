"""Build tests/exp_check (test infrastructure), a HIP program that checks the decay's
exponential of the device code for every fp32 argument."""
from __future__ import annotations

import os
import subprocess

from paper_2609_39185_amd import build as hip_build

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(HERE, "exp_check.hip")
BINARY = os.path.join(HERE, "exp_check")


def build(verbose: bool = False) -> str:
    """hipcc with the library's own floating-point flags."""
    tmp = BINARY + ".tmp"
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    cmd = [hip_build.hipcc(), *flags, "-I", hip_build.CSRC, SOURCE, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    if os.path.exists(BINARY):
        os.remove(BINARY)  # a failed compile leaves no older program to be run in its place
    subprocess.run(cmd, check=True)
    os.replace(tmp, BINARY)
    return BINARY
