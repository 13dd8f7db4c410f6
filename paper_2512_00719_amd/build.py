"""Builds libsimple_sample.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libsimple_sample.so")
SOURCES = [os.path.join(PKG, "csrc", f) for f in ("simple_kernels.hip", "simple_fast.hip", "simple_wide.hip", "simple_pattern.hip", "simple_state.hip", "simple_constraints.hip", "simple_hotfirst.hip", "simple_probe.hip", "simple_api.hip")]
OBJ_DIR = os.path.join(PKG, "_build")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # selection keys must be bit-identical to individually rounded float32 operations
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    # keep the compiler from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


# The single-pass kernel reserves list slots with one LDS atomic issued by one lane of a wave; the
# compiler's wave-level aggregation of atomics would wrap that single lane in a second reduction.
# The kernels behind it loop over rows and slices; constants of the double-precision functions, moved in front of those
# loops, took up to 40 registers from end to end (the finishing kernel spills 8 so, and a kernel that uses scratch memory
# starts 2 us later).  Of the bins and classifying kernels none spills a vector register as built (79 to 128 of them), four of
# those with a hot set 3 to 10 with the constants moved; calls that run all three, with them moved and as built: 256
# float32 rows of 128,256 columns, temperature alone, 67.8 and 66.2 us; 128 bfloat16 rows of 262,144 136.6 and 136.1; 1024 float32
# rows of 128,256, 128 of 50,001 and 4096 bfloat16 rows of 256,000 the same.
PER_SOURCE_FLAGS = {"simple_fast.hip": ["-mllvm", "-amdgpu-atomic-optimizer-strategy=None"],
                    "simple_wide.hip": ["-mllvm", "-disable-machine-licm"]}


def build(verbose: bool = False, extra_flags: tuple = (), lib: str = LIB) -> str:
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    os.makedirs(OBJ_DIR, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]

    def compile_one(src: str) -> str:
        obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
        cmd = [hipcc, *HIPCC_FLAGS, *PER_SOURCE_FLAGS.get(os.path.basename(src), []), *extra_flags, *inc, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return lib


if __name__ == "__main__":
    print(build(verbose=True))
