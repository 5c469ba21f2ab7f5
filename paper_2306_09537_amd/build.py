"""Build the HIP library libquadswarm.so for gfx950 (in-tree).

Run as ``python -m paper_2306_09537_amd.build``; ``__graft_entry__.build()``
calls :func:`build`.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libquadswarm.so")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
DEPS = SOURCES + sorted(glob.glob(os.path.join(CSRC, "*.h"))) + [
    os.path.join(INCLUDE, "quadswarm.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # multiply-adds fuse only within one source expression, so every kernel
    # specialisation (and the adjoint's recomputation) rounds identically
    "-ffp-contract=on",
    # no packed-FP32 instructions: plain float code only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # leading kernel arguments arrive in SGPRs instead of through a scalar
    # load of the argument segment (a fallback prologue loads them where the
    # firmware does not preload)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument",
    "-I", INCLUDE, "-I", CSRC,
]


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile the translation units side by side and link them."""
    if not force and os.path.exists(LIB) and all(
            os.path.getmtime(LIB) >= os.path.getmtime(d) for d in DEPS):
        return LIB

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)

    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as objs:
        out = [os.path.join(objs, os.path.basename(s) + ".o") for s in SOURCES]
        with concurrent.futures.ThreadPoolExecutor(len(SOURCES)) as pool:
            list(pool.map(lambda so: run([HIPCC, *FLAGS, "-c", so[0], "-o", so[1]]),
                          zip(SOURCES, out)))
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *out, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose="-v" in sys.argv))
