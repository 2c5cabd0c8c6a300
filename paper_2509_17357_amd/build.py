"""Builds libcronus.so (HIP kernels + C ABI) for gfx950, in-tree, with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcronus.so")
SOURCES = ["api.cpp", "plan.cpp", "balancer.cpp", "kv_append.hip", "kv_gather.hip", "attn_mixed.hip", "mfma_probe.hip"]
# Loops on cache lines: the steady loop of the chunk tiles takes up to 1 % more or less with its place in memory
# (attention of 28 k-key fp8 chunks 5.93 ms at one place, 5.98 at another; 5.94 aligned).
FLAGS = ["--offload-arch=gfx950", "-O3", "-falign-loops=64", "-std=c++17", "-fPIC", "-shared", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-x", "hip"]


def build(extra_flags=(), out=LIB, verbose=True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, *extra_flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", out]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    log = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + log)
    if verbose and log.strip():
        print(log)
    return out


if __name__ == "__main__":
    build(tuple(sys.argv[1:]))
