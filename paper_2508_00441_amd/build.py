"""Builds libozaki.so (the C-ABI HIP library) in-tree with hipcc for gfx950.

    python -m paper_2508_00441_amd.build          # compile every translation unit and link

hipcc cross-compiles without a GPU.  Objects go to csrc/_build/, the library next to this file.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libozaki.so")
SOURCES = ["api.hip", "split.hip", "pair_gemm.hip", "pair_gemm_fp8.hip", "pair_gemm_measured.hip", "pair_gemm_small.hip", "pair_gemm_small_behind.hip", "accumulate.hip",
           "ladder_sums.hip", "off_ladder.hip", "off_ladder_fp8.hip", "off_ladder_int8.hip"] + [f"ladder_sums_{fmt}_{mode}.hip" for mode in ("emu", "exact", "hw") for fmt in ("fp8", "fp6", "fp6_e3m2", "int8")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # keep packed-FP32 instructions out of the code
    "-ffp-contract=off",                                           # never fuse a multiply into an FP64 add
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option", "-Wno-option-ignored",
]


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{out}")
    if out.strip():
        print(out)
    return obj


def build_library(verbose: bool = True) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.check_call(cmd)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build_library()
    sys.exit(0)
