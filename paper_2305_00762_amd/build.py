"""Build the C-ABI library libgbr.so (HIP, gfx950) in-tree.

hipcc -O3 --offload-arch=gfx950; packed FP32 instructions are switched off
(-Xclang -target-feature -Xclang -packed-fp32-ops) for every HIP source, and
matrix-core instructions take their accumulators in VGPRs.
"""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgbr.so")
SOURCES = ["gbr_api.hip", "batch.hip", "stage3d.hip", "stage_fp64.hip", "stage_fp64_mlp.hip",
           "stage_f32.hip", "stage_f32_mlp.hip", "stage_cons.hip", "stage_order4.hip", "stage_shock_stable.hip",
           "stage_mpe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # multiply-adds fuse as the source groups them, so one tile function
         # rounds alike in every kernel it is inlined into
         "-ffp-contract=on",
         # matrix-core results in VGPRs (no accumulator-register copies)
         "-mllvm", "-amdgpu-mfma-vgpr-form=1",
         "-Wall", "-Wno-unused-function", "-I", os.path.join(ROOT, "include")]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


def build(verbose: bool = False, extra=None) -> str:
    """Compiles the units side by side, then links them."""
    flags = FLAGS + (extra or [])
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.splitext(s)[0] + ".o") for s in SOURCES]
        with ThreadPoolExecutor(min(len(SOURCES), os.cpu_count() or 1)) as pool:
            for f in [pool.submit(_run, [HIPCC] + flags + ["-c", os.path.join(CSRC, s), "-o", o],
                                  verbose) for s, o in zip(SOURCES, objs)]:
                f.result()
        _run([HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared"] + objs + ["-o", LIB + ".tmp"],
             verbose)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    extra = sys.argv[1:]
    build(verbose=True, extra=extra)
