"""Build libhelm.so (HIP, gfx950) in-tree.

Every call compiles all sources (one hipcc process per translation unit, in
parallel) and links ``paper_2405_12380_amd/libhelm.so``.  Run as
``python -m paper_2405_12380_amd.build``.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libhelm.so")
SOURCES = ["stencil.hip", "relax.hip", "blas1.hip", "gmres.hip", "dense.hip", "trunk.hip", "gram.hip", "coarse.hip", "deeponet.hip", "meta.hip", "prof.hip",
           "adjoint.hip", "batch.hip", "train.hip", "mg.hip", "noalloc.hip", "pool.hip", "api.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         # keep the compiler from emitting packed-fp32 VALU forms
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # fuse a multiply into an add only within one source expression, so
         # every kernel's rounding follows its source and not the optimizer's
         # choices (which otherwise change from build to build)
         "-ffp-contract=on",
         "-Wno-unused-result", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(jobs: int | None = None) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(len(SOURCES), os.cpu_count() or 4, 8)
    with ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", f"--offload-arch={ARCH}", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
    sys.exit(0)
