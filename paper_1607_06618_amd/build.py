"""Build libgerbil.so (gfx950) in-tree with hipcc."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgerbil.so")
ARCH = os.environ.get("GERBIL_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp"

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    # one compiler per source, eight at a time (one after the other: three minutes)
    with tempfile.TemporaryDirectory(dir=HERE) as objs, ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
        out = {s: os.path.join(objs, os.path.basename(s) + ".o") for s in sources()}
        list(pool.map(lambda s: run([hipcc, *HIPCC_FLAGS, "-I", os.path.join(HERE, "..", "include"), "-c", s, "-o", out[s]]),
                      sources()))
        run([hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", *out.values(), "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
