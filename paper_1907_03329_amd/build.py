"""Compile the HIP library for gfx950 into paper_1907_03329_amd/libesrnn_hip.so.

hipcc cross-compiles without a GPU.  Each source is compiled to an object in
parallel, then linked into one shared library that exports the C ABI of
include/esrnn.h.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libesrnn_hip.so")
SOURCES = ["esrnn_api.cpp", "plan.cpp", "es_kernels.hip", "lstm_kernels.hip", "lstm_backward_kernels.hip", "lstm_backward_large_kernels.hip",
           "lstm_forward_kernels.hip", "lstm_forward_residual_kernels.hip", "lstm_narrow_kernels.hip", "lstm_narrow_fwd_residual_kernels.hip", "lstm_narrow_bwd_kernels.hip", "lstm_narrow_bwd_split_kernels.hip", "lstm_together_kernels.hip",
           "lstm_together_wide_kernels.hip", "lstm_together_forecast_kernels.hip", "lstm_together_reverse_kernels.hip", "head_kernels.hip", "opt_kernels.hip",
           "static_scratch.hip", "probe_kernels.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wall", "-Wno-unused-function"]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if warn and os.environ.get("ESRNN_BUILD_VERBOSE"):
        print(warn, file=sys.stderr)
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return LIB


if __name__ == "__main__":
    print(build())
