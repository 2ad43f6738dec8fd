"""Build the fftgal shared library for gfx950 with hipcc (in-tree).

    python -m paper_1412_2033_amd.build

Produces ``paper_1412_2033_amd/_lib/libfftgal.so`` from ``csrc/*.hip`` and
``csrc/*.cpp``.  Every HIP compilation disables packed FP32 instructions.
"""

from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "_lib")
LIB = os.path.join(LIBDIR, "libfftgal.so")

FAST_PARTS = 8  # kFastParts: the specialised kernels are compiled in parts, side by side
# (source, object, extra flags)
UNITS = [("fftgal_fast.hip", "fftgal_fast%d.o" % p, ["-DFFTGAL_PART=%d" % p]) for p in range(FAST_PARTS)] + [
    ("fftgal_kernels.hip", "fftgal_kernels.o", []), ("fftgal.cpp", "fftgal.o", [])]
HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc():
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose=True):
    os.makedirs(LIBDIR, exist_ok=True)

    def compile_unit(unit):
        src, obj, extra = unit
        obj = os.path.join(LIBDIR, obj)
        cmd = [hipcc()] + HIPCC_FLAGS + extra + ["-x", "hip", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                                                 "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    jobs = int(os.environ.get("MAX_JOBS", min(8, os.cpu_count() or 1)))
    with concurrent.futures.ThreadPoolExecutor(max_workers=max(1, jobs)) as pool:
        objs = list(pool.map(compile_unit, UNITS))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs + \
        ["-Wl,-rpath,/opt/rocm/lib"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    for obj in objs:
        os.remove(obj)
    return LIB


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
