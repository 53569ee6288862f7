"""Builds the HIP library libhbsjd.so for gfx950 in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(ROOT, "_build", "obj")
LIB = os.path.join(HERE, "libhbsjd.so")
SOURCES = ["abi.hip", "gemm.hip", "attention.hip", "rowops.hip", "sampler.hip", "score.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         # packed fp32 instructions stay off: some of their forms have given
         # wrong results on this hardware without any error
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # MFMA accumulators in VGPRs: with the AGPR form the compiler moves
         # loop-carried accumulators between AGPRs and VGPRs every K step
         # (60-400 v_accvgpr moves per main-loop iteration of the smaller GEMM
         # tiles and the attention kernels) and lowers their occupancy
         "-mllvm", "-amdgpu-mfma-vgpr-form",
         # the first kernel arguments arrive in SGPRs at dispatch instead of by
         # a load the kernel waits for: 0.05-0.2 us of every latency-bound
         # launch (norm 2.85 -> 2.72 us, attention of a B round 8.49 -> 8.36,
         # 32-row W1|W3 3.87 -> 3.71), a B round has 89
         "-mllvm", "-amdgpu-kernarg-preload-count=16",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _compile(src: str) -> str:
    out = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return out


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + f".tmp{os.getpid()}"
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
