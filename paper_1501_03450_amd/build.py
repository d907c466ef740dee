"""Build the HIP library libspintrack.so in-tree for gfx950 with hipcc."""

from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libspintrack.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # multiply-adds fused only within one expression, so that every kernel
    # instantiation rounds the same source the same way (the mixed-precision
    # kernel reproduces the double-precision orbit bit for bit)
    "-ffp-contract=on",
    # machine LICM moves the literal constants of every element body of the
    # tracking kernel out of the element loop into registers: 256 VGPRs and 52
    # to 184 B of scratch a lane, against 238 and none without it
    "-mllvm", "-disable-machine-licm=1",
    # no packed-FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-I", CSRC,
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = False, extra=()) -> str:
    """Compile every source to an object, side by side, and link the library."""
    tmp = LIB + ".tmp%d" % os.getpid()

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    with tempfile.TemporaryDirectory() as objects:
        def compile_one(source):
            obj = os.path.join(objects, os.path.basename(source) + ".o")
            run([HIPCC, *FLAGS, *extra, "-c", source, "-o", obj])
            return obj

        jobs = int(os.environ.get("MAX_JOBS") or os.cpu_count() or 1)
        with ThreadPoolExecutor(min(jobs, len(sources()))) as pool:
            objs = list(pool.map(compile_one, sources()))
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
