"""Builds the HIP library (csrc/*.hip -> libfastpoint_hip.so) for gfx950 with hipcc.

-ffp-contract=off: every binary32 operation of a squared distance is rounded on
its own (index results are compared bit for bit with a CPU reference).  Packed
fp32 instructions are switched off for all device code."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfastpoint_hip.so")
# (source, points per thread): the sampler is compiled once per number of points a thread holds
SOURCES = [("sampler.hip", p) for p in (16, 8, 4, 2)] + [(f, 0) for f in ("local_sampler.hip", "ball_query.hip", "knn.hip", "excl_lists.hip", "abi.hip")]
FLAGS = ["--offload-arch=gfx950", "-O3", *os.environ.get("FASTPOINT_EXTRA_FLAGS", "").split(), "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wall", "-Wno-unused-function"]


def _compile(unit) -> str:
    src, points = unit
    obj = os.path.join(CSRC, os.path.splitext(src)[0] + ("_p%d" % points if points else "") + ".o")
    define = ["-DFASTPOINT_SAMPLER_P=%d" % points] if points else []
    if points == 2:
        # The pick chain of these kernels is a short loop of one wave, 1-3 % slower or faster with where it falls among the
        # cache lines: at their start, exact FPS of 16 x 1024 points 117.5 -> 114.5 us, of 4096 points 326 -> 322.  (Kernels
        # with four points per thread lose 2 % by it on the LiDAR batch.)
        define.append("-falign-loops=64")
    subprocess.run(["hipcc", *FLAGS, *define, "-c", os.path.join(CSRC, src), "-o", obj], check=True)
    return obj


def build(verbose: bool = False) -> str:
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
