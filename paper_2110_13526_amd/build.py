"""Build the HIP library ``libkct.so`` for gfx950 in-tree.

    python -m paper_2110_13526_amd.build

Compiles every source under ``csrc/`` with hipcc as HIP (device code for
gfx950 only), with floating-point contraction off (the weight function must
round identically in the forward and the backward kernel) and packed-FP32
instructions disabled.  The projector kernels (which form no NaN: every
infinity they use is an explicit sentinel) are compiled without IEEE-mode
min/max, so fminf/fmaxf need no operand canonicalisation; the solver kernels,
which test for non-finite values, keep the default.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libkct.so")
ARCH = "gfx950"


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def flags():
    return [
        f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-Wall", "-Wno-unused-result", "-I" + os.path.join(os.path.dirname(HERE), "include"),
    ]


PROJECTOR_SOURCES = {"projector.hip", "forward_r1.hip", "forward_r2.hip", "forward_r3.hip", "forward_r4.hip",
                     "backproject.hip", "backproject_wave.hip", "tt.hip", "tt_forward.hip", "tt_backward.hip"}


def source_flags(src):
    if os.path.basename(src) in PROJECTOR_SOURCES:
        return ["-fno-honor-nans", "-mno-amdgpu-ieee"]
    return []


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile each source to an object in parallel, then link the shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in sources():
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        objs.append(obj)
        cmd = [hipcc, *flags(), *source_flags(src), "-x", "hip", "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        if len(procs) >= jobs:
            _wait(procs.pop(0))
    for p in procs:
        _wait(p)
    tmp = LIB + ".tmp"
    cmd = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


def _wait(item):
    src, p = item
    out, _ = p.communicate()
    text = out.decode(errors="replace")
    if p.returncode != 0:
        sys.stderr.write(text)
        raise RuntimeError(f"hipcc failed on {os.path.basename(src)}")
    if text.strip():
        lines = [ln for ln in text.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
        if lines:
            sys.stderr.write("\n".join(lines) + "\n")


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
