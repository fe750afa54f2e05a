"""Build libkvqp.so (the C-ABI library) in-tree with hipcc for gfx950.

    python -m paper_2412_12706_amd.build

Every translation unit is compiled for gfx950 only, with packed-FP32 code
generation switched off and without floating-point contraction (the quantizer
is a fixed sequence of individually rounded binary32 operations; kernels that
want a fused multiply-add ask for it explicitly).
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libkvqp.so")
# (the decode kernels, most of the work, are one object per bit width)
SOURCES = [f"decode_attn.hip:{bits}" for bits in (4, 8, 2, 16)] + ["quant_pack.hip", "score_select.hip", "decode_attn.hip", "kvqp_api.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-mllvm", "-amdgpu-mfma-vgpr-form",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _compile(src: str) -> str:
    src, _, bits = src.partition(":")
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + bits + ".o")
    cmd = ["hipcc", "-x", "hip"] + FLAGS + ([f"-DKVQP_DECODE_BITS={bits}"] if bits else []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "not a recognized feature" not in l)
    if r.returncode:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
