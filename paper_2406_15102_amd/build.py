"""Build the HIP library (``libhlq.so``) for gfx950 in-tree with hipcc.

``python -m paper_2406_15102_amd.build`` compiles every ``csrc/*.hip`` into one shared
object next to this file.  hipcc cross-compiles without a GPU.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhlq.so")
OBJDIR = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    # no packed-fp32 instructions: some of their forms have given wrong results
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    # the k loops of the matrix products are written to be unrolled in full (a step of 256 MFMAs with
    # everything that issues between them); the default size limit for `#pragma unroll` is below that
    "-mllvm", "-pragma-unroll-threshold=1000000",
    # every nested guard restores the lanes of the one around it: without that the register allocator's reloads at the end of
    # a guarded store missed the lanes that only the inner guard had switched off.  The epilogues that showed it have no guard inside
    # another any more and pass tests/test_gpu_edge_columns.py without this option too; it stays for the other kernels.  It costs
    # scalar spills in the convolution's products (40 and 47 -> 49), which do not show: whole passes of convolutions without / with
    # it 48.2 / 47.7 us (12544 x 256 over 256, 3 x 3), 68.9 / 69.4 (50176 x 128 over 128), 54.7 / 54.9 (fp32).
    "-mllvm", "-amdgpu-remove-redundant-endcf=false",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = True, jobs: int = 8) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = sources()
    objs = [os.path.join(OBJDIR, os.path.basename(s)[:-4] + ".o") for s in srcs]

    def compile_one(pair):
        src, obj = pair
        cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        list(ex.map(compile_one, zip(srcs, objs)))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build()
    print("built", LIB)
    sys.exit(0)
