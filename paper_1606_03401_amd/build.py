"""Builds the C-ABI library ``libmebptt.so`` in-tree with hipcc for gfx950.

Run as ``python -m paper_1606_03401_amd.build``; ``__graft_entry__.build()`` calls ``build()``.
Every source is compiled to an object of its own, several at a time, then linked.
"""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import tempfile

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libmebptt.so")
SOURCES = ["resident_wide_2.hip", "resident_wide_1.hip", "resident_wide_3.hip", "resident_sweep_bf16.hip", "resident_sweep_fp32.hip", "resident_chain_bf16_k4.hip",
           "resident_chain_bf16_k8.hip", "resident_chain_fp32_k8.hip", "resident_back_bf16.hip",
           "resident_chain_fp32_k4.hip", "kernels.hip", "run.hip", "resident.hip", "chain_run.hip", "measure_sync.hip",
           "planner.cpp", "chain_planner.cpp"]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wall", "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build(verbose: bool = True) -> str:
    exe = hipcc()
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.splitext(s)[0] + ".o") for s in SOURCES]
        jobs = min(len(SOURCES), int(os.environ.get("MAX_JOBS", "8")), 8)
        with concurrent.futures.ThreadPoolExecutor(jobs) as pool:
            for f in [pool.submit(_run, [exe, *FLAGS, "-c", os.path.join(CSRC, s), "-o", o], verbose)
                      for s, o in zip(SOURCES, objs)]:
                f.result()
        _run([exe, "--offload-arch=gfx950", "-fPIC", "-shared", *objs, "-o", LIB_PATH + ".tmp"], verbose)
    os.replace(LIB_PATH + ".tmp", LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build()
    sys.exit(0)
