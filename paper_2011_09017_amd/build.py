"""Builds libcmpz.so (HIP, gfx950) in-tree with hipcc.  Run: python -m paper_2011_09017_amd.build"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcmpz.so")
SOURCES = ["cmpz_api.hip", "cmpz_compress.hip", "cmpz_sweep1.hip", "cmpz_codebook.hip", "cmpz_pack.hip", "cmpz_decompress.hip", "cmpz_decode_fused.hip",
           "cmpz_controller.hip"]

# -ffp-contract=off: the quantiser multiplies must stay single roundings (no FMA).
# Packed fp32 instructions are disabled for the device code.
# -falign-loops=32: where a loop begins in its cache line made the decode of small tensors, one wave per SIMD bound by
# the fetch of its instructions, up to 6 % slower or faster with any change of the code around it.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math", "-falign-loops=32",
         "-Wall", "-Wno-unused-result",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build_library(verbose: bool = False, defines=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, *["-D" + d for d in defines], "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd)))
        objs.append(obj)
    for cmd, p in procs:
        if p.wait() != 0:
            raise RuntimeError("compile failed: " + " ".join(cmd))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv, defines=[a[2:] for a in sys.argv[1:] if a.startswith("-D")]))
