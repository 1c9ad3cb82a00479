"""Build the HIP library ``libamrlbm.so`` for gfx950 with hipcc (in-tree).

Usage: ``python -m paper_2308_08085_amd.build`` or ``build()`` from Python.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libamrlbm.so")
BUILD_DIR = os.path.join(HERE, "_build")
# (object, source, defines); the lattice Boltzmann kernels of each lattice and
# storage (enum amr_storage) are a unit of their own, the slowest first
STORAGES = ("AMR_F64", "AMR_F32", "AMR_F32S", "AMR_F16S", "AMR_BF16S")
UNITS = [("lbm_q%d_%s" % (q, s[4:].lower()), "lbm_kernels.hip", ["-DAMR_TU_Q=%d" % q, "-DAMR_TU_S=" + s])
         for q in (27, 19, 9) for s in STORAGES] + \
        [(n, n + ".hip", []) for n in ("lbm_kernels", "mesh_kernels", "runtime", "transfer", "batch")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # multiply-adds fuse only within one source expression: every kernel that
    # shares an arithmetic routine (the plain, joined and batched sweeps, and
    # their variants) then rounds it the same way, whatever code surrounds it
    "-ffp-contract=on",
    "-Wall", "-Wno-unused-function",
]


def _compile(unit) -> str:
    name, src, defines = unit
    obj = os.path.join(BUILD_DIR, name + ".o")
    cmd = [HIPCC] + FLAGS + defines + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (name, " ".join(cmd), r.stderr))
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=max(1, min(16, os.cpu_count() or 1))) as ex:
        objs = list(ex.map(_compile, UNITS))
    tmp = OUT + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (" ".join(cmd), r.stderr))
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
