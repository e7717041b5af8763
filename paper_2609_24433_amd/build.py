"""Build libfq.so in-tree with hipcc for gfx950.

  python -m paper_2609_24433_amd.build        (or __graft_entry__.build())

Every HIP source is compiled with -ffp-contract=off (the prologue's codes must be
reproducible bit for bit: no multiply-add may be fused) and with packed-fp32
instructions disabled.  ``fq_gemm.hip`` and ``fq_small.hip`` keep MFMA accumulators in
ordinary VGPRs (``-amdgpu-mfma-vgpr-form``): with them in AGPRs the register allocator
splits the budget in half and spills their double-buffered operands into AGPRs.  The
k-group GEMM (``fq_gemm_kg.hip``, 128 accumulators and three register sets of operands) and
the wide-tile GEMMs (``fq_gemm_wide.hip``) need the AGPRs.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfq.so")
SOURCES = ["fq_api.cpp", "fq_quant.hip", "fq_rotate.hip", "fq_gemm.hip", "fq_gemm_kg.hip", "fq_gemm_wide.hip", "fq_gptq.hip",
           "fq_small.hip"]
ARCH = "gfx950"

COMMON_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-I", os.path.join(ROOT, "include"),
]


EXTRA_FLAGS = {"fq_gemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"], "fq_small.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OUT_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *COMMON_FLAGS, *EXTRA_FLAGS.get(src, []), "-x", "hip", "-c",
           os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "'-packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip() and verbose:
        print(err, file=sys.stderr)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OUT_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
