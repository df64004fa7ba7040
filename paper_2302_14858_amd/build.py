"""Build the HIP library ``libcfd_mi355x.so`` in-tree for gfx950.

Every source is compiled with hipcc; the device code targets gfx950 only.
Objects are compiled in parallel and linked into one shared library next to
this file, which the Python binding loads.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libcfd_mi355x.so")
BUILD = os.path.join(HERE, "_build")

SOURCES = ["scheme_design.cpp", "cfd_host.cpp", "cfd_kernels.hip", "cfd_kernels_f32.hip", "cfd_kernels_ext.hip",
           "cfd_kernels_ext_f32.hip", "cfd_aux.hip", "cfd_dense.hip", "cfd_noalloc.hip", "cfd_iterate.hip",
           "cfd_biased.hip", "cfd_biased_f32.hip", "cfd_biased_wide.hip", "cfd_biased_wide_f32.hip",
           "cfd_biased_big.hip", "cfd_biased_big_f32.hip"]

COMMON = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + INCLUDE, "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]

# A wave of the biased kernel holds its rows in arrays that unrolling turns into
# registers.  Promoted to vectors before that, the FP32 arrays are copied whole
# at every row guard: 253 VGPRs and 218 AGPRs instead of 70 and 0.
EXTRA = {s: ["-mllvm", "-disable-promote-alloca-to-vector=1"] for s in SOURCES if s.startswith("cfd_biased")}


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    cmd = [hipcc()] + COMMON + EXTRA.get(src, []) + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compiling {src} failed:\n{r.stdout}\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950"] + objs + ["-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"linking failed:\n{r.stdout}\n{r.stderr}")
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
