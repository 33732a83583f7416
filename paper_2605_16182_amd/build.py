"""Compile the HIP library (csrc/*.hip) into libtw.so for gfx950 with hipcc.

Each translation unit compiles in its own hipcc process (in parallel), then
one link step produces the shared library next to this file.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build", "tw")
LIB = os.path.join(HERE, "libtw.so")
SOURCES = ["prim.hip", "index.hip", "nodeview.hip", "weights.hip", "adjacency.hip", "walk.hip",
           "queue.hip", "serve.hip", "capi.hip"]
# roofline probes for the benchmark, a separate library
PROBE_LIB = os.path.join(HERE, "libtw_probe.so")
PROBE_SOURCES = ["probe.hip"]

# walk.hip: keep the FP64 functions' constants out of registers. Hoisted out of
# the hop loops, the polynomial coefficients of log, exp and their variants held
# up to 60 VGPRs for the whole walk: exponential hops took 128 VGPRs (68 now),
# node2vec's 128 with 24 spilled (76), so fewer wavefronts were in flight. (Not
# for queue.hip, whose kernels write rows piecemeal and lose 10-15 % with more
# wavefronts in flight.) A compiler that does not know the option refuses the file;
# one that knows it and hoists all the same shows in the resource report
# (-Rpass-analysis=kernel-resource-usage), not in the results.
EXTRA_FLAGS = {"walk.hip": ["-mllvm", "-disable-machine-licm"]}

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # identical FP64 rounding to a plain C evaluation of the pickers
    "-ffp-contract=off",
    # no packed FP32 instructions anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"),
    "-I", CSRC,
]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, *EXTRA_FLAGS.get(src, []), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return obj


def _link(objs, lib, verbose):
    tmp = lib + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, lib)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = SOURCES + PROBE_SOURCES
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    _link(objs[:len(SOURCES)], LIB, verbose)
    _link(objs[len(SOURCES):], PROBE_LIB, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
