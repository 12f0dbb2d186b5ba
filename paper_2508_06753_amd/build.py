"""Builds libw2mm.so (HIP, gfx950 only) in-tree with hipcc.

Usage: python -m paper_2508_06753_amd.build [--force]
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libw2mm.so")
SOURCES = ["api.hip", "prepack.hip", "quantize.hip", "matmul_a8_small.hip",
           "matmul_midm.hip", "matmul_shared.hip", "matmul_a8_tiled.hip", "matmul_a8_tiled128.hip", "matmul_a8_gemv.hip", "matmul_a16.hip", "matmul_a16_fold.hip",
           "comparators.hip", "splitk.hip"]
HEADERS = ["w2_layout.h", "w2_internal.h", "w2_small_common.h", "midm_common.h", "midm_plan.h", "shared_plan.h", "tile_plan.h", "tall_waits.h", "auto_plan.h", os.path.join("..", "..", "include", "w2mm.h")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Wall", "-Wno-unused-function",
         # the mid-M and prefill w2a8 kernels read int32 accumulators as fp32 denormals (one-fma dequant):
         # denormals must be kept (HIP's default), never flushed; the sources refuse -ffast-math as well
         "-fno-gpu-flush-denormals-to-zero",
         # packed-fp32 VALU forms are kept out of the generated code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


# per-file additions: the decode kernel asks for the first dwords of its scalar kernel arguments to be
# handed over in registers at wave launch (the compiled entry still fetches them itself where the machine does not)
_PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
# (also the row quantiser and the streaming-read probe the decode kernel is compared with: scalar parameters already)
EXTRA_FLAGS = {"matmul_a8_gemv.hip": _PRELOAD, "quantize.hip": _PRELOAD, "api.hip": _PRELOAD,
               "matmul_midm.hip": _PRELOAD, "matmul_shared.hip": _PRELOAD}


def _newer(target, deps):
    if not os.path.exists(target):
        return False
    t = os.path.getmtime(target)
    return all(os.path.getmtime(d) <= t for d in deps)


def build(force=False, verbose=True):
    os.makedirs(OBJDIR, exist_ok=True)
    hdrs = [os.path.normpath(os.path.join(CSRC, h)) for h in HEADERS]
    jobs = []
    objs = []
    for s in SOURCES:
        src = os.path.join(CSRC, s)
        obj = os.path.join(OBJDIR, s.replace(".hip", ".o"))
        objs.append(obj)
        if force or not _newer(obj, [src] + hdrs):
            jobs.append([HIPCC] + FLAGS + EXTRA_FLAGS.get(s, []) + ["-c", src, "-o", obj])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed:\n{r.stdout}\n{r.stderr}")
        if verbose and r.stderr.strip():
            # hipcc's host pass warns that it does not know the packed-fp32 feature: harmless
            lines = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip()]
            if lines:
                print("\n".join(lines), flush=True)

    with ThreadPoolExecutor(max_workers=min(6, max(1, len(jobs)))) as ex:
        list(ex.map(run, jobs))
    if jobs or force or not os.path.exists(LIB):
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    return LIB


if __name__ == "__main__":
    build(force="--force" in sys.argv)
    print(LIB)
