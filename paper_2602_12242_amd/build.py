"""Builds libmagx.so (gfx950) in-tree with hipcc.

    python -m paper_2602_12242_amd.build          # or build() from Python

Every source is compiled by itself, in parallel; conv.hip, column.hip and
pencil.hip once per element type (MAGX_REAL = 32 or 64), pencil.hip also once per
order of the x spectrum (MAGX_COLS = 0 or 1).  Packed-FP32 instructions are
disabled for the device code.  The sign of a zero result is not significant
anywhere in the library, so x + 0 may fold to x (the zero-padded halves of the
first FFT passes then cost no arithmetic).
"""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libmagx.so")
# (source, macros of each time it is compiled), the longest first
REALS = [{"MAGX_REAL": 64}, {"MAGX_REAL": 32}]
SOURCES = [("pencil.hip", [{**r, "MAGX_COLS": c} for c in (0, 1) for r in REALS]), ("column.hip", REALS),
           ("conv.hip", REALS), ("mri.hip", [{}]), ("tensor.hip", [{}]), ("magx_api.cpp", [{}])]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-fno-signed-zeros", "-Wno-unused-command-line-argument", "-I", INCLUDE]


def hipcc():
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building libmagx.so")


def build(verbose=False):
    with tempfile.TemporaryDirectory() as tmp:
        jobs, objs = [], []
        for src, variants in SOURCES:
            for macros in variants:
                obj = os.path.join(tmp, f"{len(objs)}_{os.path.splitext(src)[0]}.o")
                define = [f"-D{k}={v}" for k, v in macros.items()]
                jobs.append([hipcc(), *FLAGS, *define, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj])
                objs.append(obj)
        with ThreadPoolExecutor(len(jobs)) as pool:
            list(pool.map(lambda c: _run(c, verbose), jobs))
        out = LIB + ".tmp"
        _run([hipcc(), "--offload-arch=gfx950", "-fPIC", "-shared", "-o", out, *objs], verbose)
    os.replace(out, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
