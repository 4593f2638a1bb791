"""Compile the HIP sources in csrc/ into paper_2512_17917_amd/libkvr.so for gfx950.

hipcc cross-compiles without a GPU.  Objects go to paper_2512_17917_amd/_build/.
The host extension of the binding (csrc/kvr_fast.c) is built beside it where there is
a C compiler and Python.h; without it the binding makes the same calls through ctypes.
Usage: python -m paper_2512_17917_amd.build
"""
from __future__ import annotations

import importlib.machinery
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libkvr.so")
OBJ_DIR = os.path.join(HERE, "_build")
# host code: the two calls of a decode step, checked and made in C; the suffix names the interpreter it is built for
FAST = os.path.join(HERE, "_kvr_fast" + importlib.machinery.EXTENSION_SUFFIXES[0])
CC = "gcc"

SOURCES = ["kvr_api.hip", "kvr_reconstruct.hip", "kvr_attend.hip", "kvr_attend_staged.hip", "kvr_attend_staged64.hip", "kvr_attend_staged16.hip", "kvr_attend_retained.hip", "kvr_select.hip", "kvr_compact.hip",
           "kvr_encode.hip", "kvr_swap.hip", "kvr_attend_multi.hip", "kvr_attend_multi_staged.hip"]

# packed-FP32 instruction selection is switched off on purpose (ordinary float
# code only); the host pass warns that it does not know the feature.
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unused-command-line-argument"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(" ".join(cmd) + "\n" + r.stdout + r.stderr)
        raise RuntimeError(os.path.basename(cmd[0]) + " failed: " + cmd[-1])
    return r


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    hipcc = _hipcc()
    jobs = []
    for s in SOURCES:
        obj = os.path.join(OBJ_DIR, s.replace(".hip", ".o"))
        jobs.append((obj, [hipcc, *HIP_FLAGS, "-c", os.path.join(CSRC, s), "-o", obj]))
    with ThreadPoolExecutor(max_workers=min(8, len(jobs))) as ex:
        for r in ex.map(lambda j: _run(j[1]), jobs):
            if verbose and r.stderr:
                sys.stderr.write(r.stderr)
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT, *[j[0] for j in jobs]])
    build_fast()
    return OUT


def build_fast() -> bool:
    """The binding's host extension, or a message and none (nor one from before, made from other sources)."""
    if os.path.exists(FAST):
        os.remove(FAST)
    try:
        _run([CC, "-O2", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"], "-o", FAST, os.path.join(CSRC, "kvr_fast.c")])
    except (OSError, RuntimeError) as e:
        sys.stderr.write(f"{os.path.basename(FAST)} left out ({e}): the binding checks and calls through ctypes\n")
        return False
    return True


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
