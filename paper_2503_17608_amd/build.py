"""Compile the HIP library libemstep.so for gfx950 (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "emstep.hip")
LIB = os.path.join(HERE, "libemstep.so")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-munsafe-fp-atomics",
    # no packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no hoisting of loop-invariant machine code: it keeps the constants of
    # log, exp and sincos in registers across whole kernels, which then spill
    # or hold fewer waves (k_steps FP64 in a field: 256 registers and 430 bytes
    # of scratch with it, 220 and none without).  No other kernel is the worse
    # for it; 10^4 x 1 GeV, hoisted and not: block-local loops 15.0 and 13.3 ms,
    # radix 30.5 and 30.0, mixed precision 28.5 and 27.5, without field 36.3
    # and 31.6, queue 86.0 and 85.8, separate interactions 48.0 and 47.6;
    # masked kernels, 2000 showers, 32.5 and 28.4; deterministic, 300, 19.8 and 19.6
    "-mllvm", "-disable-machine-licm",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


def build(verbose: bool = False) -> str:
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    tmp = LIB + ".tmp"
    cmd = [hipcc, *FLAGS, "-o", tmp, SRC]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
