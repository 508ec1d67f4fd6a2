"""Build the gfx950 shared library libweno_l2is.so in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libweno_l2is.so")
SOURCES = ["wl2_capi.hip", "wl2_batch.hip", "wl2_fused3d.hip", "wl2_row.hip", "wl2_row1d.hip", "wl2_line.hip",
           "wl2_tile.hip", "wl2_weno3d.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no packed-FP32 instructions anywhere
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # FMA contraction only inside one source expression: the arithmetic of a
    # face then follows the source and not the code it is inlined into, so
    # every launch shape, pencil length, z chunk, batch or single-grid path
    # gives the same bits (cross-statement contraction saved <1% here)
    "-ffp-contract=on",
    "-Wall", "-Wno-unused-result",
]


def compile_flags(src: str) -> list:
    """The hipcc flags one source is compiled with."""
    return list(HIPCC_FLAGS)


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    bdir = os.path.join(PKG, "_build")
    os.makedirs(bdir, exist_ok=True)
    objs, procs = [], []
    for src in SOURCES:
        obj = os.path.join(bdir, src.replace(".hip", ".o"))
        cmd = ([hipcc] + compile_flags(src) + ["-I", os.path.join(ROOT, "include"),
               "-c", "-o", obj, os.path.join(PKG, "csrc", src)])
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd)))
        objs.append(obj)
    failed = [src for src, pr in procs if pr.wait() != 0]
    if failed:
        raise RuntimeError("hipcc failed on " + ", ".join(failed))
    tmp = LIB + ".tmp"
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
