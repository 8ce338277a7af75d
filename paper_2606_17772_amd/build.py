"""Build libfdcgks.so (gfx950) in-tree with hipcc.

Usage: python -m paper_2606_17772_amd.build [--verbose]
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfdcgks.so")
SOURCES = [os.path.join(CSRC, "fdcgks.hip"), os.path.join(CSRC, "fdcgks3d.hip")]
DEPS = SOURCES + [os.path.join(CSRC, "gks_device.hpp"), os.path.join(CSRC, "gks3d_device.hpp"),
                  os.path.join(CSRC, "adjoint.inc.hip"), os.path.join(CSRC, "gks_adjoint.hpp"),
                  os.path.join(ROOT, "include", "fdcgks.h"), os.path.join(ROOT, "include", "fdcgks3d.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    # no packed-FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # multiply-adds fused only within one source expression: the rounding of
    # the inlined stage code then does not depend on the kernel it sits in
    # (single problems, batches, fused and separate sweeps agree bit for bit)
    "-ffp-contract=on",
    # instruction scheduling that groups memory clauses.  The solver from moment
    # vectors needed it to fit its registers (246 VGPRs, a 2048^2 step 1%
    # faster); with the solver in primitive slopes it is within 1% of the
    # compiler's own on every kernel (2048^2 step 3.72 ms either way).  The
    # arithmetic does not depend on it
    "-mllvm", "-amdgpu-sched-strategy=max-memory-clause",
    # no machine-level loop-invariant code motion: hoisted out of the row loop of
    # the fused stage (and of the 1D step and persistent batch loops), the 64-bit
    # constants of exp and erf and similar invariants are held in registers
    # through every iteration.  Without the flag a 2048^2 step takes 5.22 instead
    # of 3.72 ms, a 1024^2 characteristic one 1.51 instead of 1.11, a step of 600
    # nodes in 1D 35.9 instead of 29.1 us, the persistent batch 2.18 instead of
    # 2.03 ms; the unfused sweeps and the adjoint are within 2%
    "-mllvm", "-disable-machine-licm",
    "-I", os.path.join(ROOT, "include"),
]


def build(verbose: bool = False, extra=()) -> str:
    tmp = LIB + ".tmp"
    cmd = [HIPCC, *FLAGS, *extra, *SOURCES, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed building libfdcgks.so")
    if verbose and r.stderr:
        sys.stderr.write(r.stderr)
    os.replace(tmp, LIB)
    return LIB


def build_test_kernels() -> str:
    """tests/libdevice_math.so: the library's elementary device routines behind
    an entry that the GPU tests call (small: a few seconds)."""
    src = os.path.join(ROOT, "tests", "device_math.hip")
    out = os.path.join(ROOT, "tests", "libdevice_math.so")
    r = subprocess.run([HIPCC, *FLAGS, src, "-o", out + ".tmp"], capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed building libdevice_math.so")
    os.replace(out + ".tmp", out)
    return out


if __name__ == "__main__":
    build(verbose="--verbose" in sys.argv,
          extra=["-Rpass-analysis=kernel-resource-usage"] if "--usage" in sys.argv else [])
