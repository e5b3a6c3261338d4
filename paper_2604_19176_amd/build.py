"""Build libpat.so (the gfx950 HIP library) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpat.so")
SOURCES = ["ring_adj.hip", "ring_fwd.hip", "grid_adj.hip", "grid_fwd.hip", "api.hip", "plan.hip", "tune.hip", "sim.hip"]
HEADERS = ["pat_internal.hpp", "device_util.hpp", "fft.hpp", "cfft.hpp", "grid.hpp", "ring.hpp",
           "kernels.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep packed-FP32 instructions out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


def build(verbose: bool = False) -> str:
    """Compiles every source (side by side: the kernels of one translation unit
    do not refer to another's) and links the library."""
    tmp = LIB + ".tmp%d" % os.getpid()
    with tempfile.TemporaryDirectory() as objs:
        def compile_one(s):
            obj = os.path.join(objs, s + ".o")
            cmd = [HIPCC] + FLAGS + ["-I", os.path.join(HERE, "..", "include"), "-c", os.path.join(CSRC, s), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
            return obj
        with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as pool:
            made = list(pool.map(compile_one, SOURCES))
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + made)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
