"""Build libfsei.so (HIP kernels for gfx950 + host plan code) in-tree."""
from __future__ import annotations

import os
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libfsei.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["fsei_api.hip", "fsei_plan.cpp"]
HEADERS = ["fsei_plan.h", "fsei_fft.h", "fsei_transforms.h", "fsei_lengths.h", "fsei_z.h", "fsei_kernels.h", "fsei_viscous.h",
           "fsei_momentum.h", "fsei_ibm.h"]
# fsei_len.hip holds the transform kernels of one length and is compiled once
# per length with kernels of its own: every 2^a 3^b from 16 to 1024
LENGTH_SOURCE = "fsei_len.hip"
# fsei_z.hip holds the z solves of one type
Z_SOURCE = "fsei_z.hip"
LENGTHS = sorted(2 ** a * 3 ** b for a in range(11) for b in range(7) if 16 <= 2 ** a * 3 ** b <= 1024)

# -packed-fp32-ops: hipcc -O3 may otherwise emit packed FP32 instructions
# from ordinary float code; this keeps them out of every kernel.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


def build(verbose: bool = True) -> str:
    include = ["-I", os.path.join(PKG, "..", "include")]
    objdir = tempfile.mkdtemp(prefix="fsei_build_")
    try:
        jobs = [(s, []) for s in SOURCES] + [(Z_SOURCE, [f"-DFSEI_REAL={t}"]) for t in ("double", "float")]
        jobs += [(LENGTH_SOURCE, [f"-DFSEI_LEN={n}"]) for n in reversed(LENGTHS)]

        def compile_one(job):
            src, defs = job
            obj = os.path.join(objdir, src.split(".")[0] + "".join(d.split("=")[1] for d in defs) + ".o")
            cmd = [HIPCC, *FLAGS, *defs, *include, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        workers = max(1, min(int(os.environ.get("MAX_JOBS", "8")), os.cpu_count() or 1))
        with ThreadPoolExecutor(workers) as pool:
            objs = list(pool.map(compile_one, jobs))
        tmp = LIB + ".tmp"
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp], check=True)
        os.replace(tmp, LIB)
    finally:
        shutil.rmtree(objdir, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    build()
