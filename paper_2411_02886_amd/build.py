"""Builds libtokenselect.so (HIP, gfx950) in-tree with hipcc.

Usage: python -m paper_2411_02886_amd.build [--force]
Objects go to paper_2411_02886_amd/_build/, the library to paper_2411_02886_amd/libtokenselect.so.
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
LIB = os.path.join(HERE, "libtokenselect.so")
SOURCES = ["api.hip", "score_decode.hip", "soft_vote.hip", "topk.hip", "selcache.hip", "sparse_attn_decode.hip", "sparse_attn_stream.hip", "prefill_select.hip", "sparse_attn_chunk.hip", "sparse_attn_chunk_wide.hip",
           "chunk_mean_query.hip", "select_variants.hip", "select_compact.hip", "score_codes_mfma.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wall", "-Wno-unused-function"] + os.environ.get("TS_EXTRA_FLAGS", "").split()

# Flags of single files.  sparse_attn_chunk_wide: its kernel runs one wave per SIMD and needs both halves of the register file; the
# results of its matrix products are read by vector instructions, which see the first half only, and without this option the
# compiler keeps all of them in the second half and moves every score over (2113 moves in the kernel, with it 182).
FILE_FLAGS = {"sparse_attn_chunk_wide.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _deps():
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    hs.append(os.path.join(ROOT, "include", "tokenselect.h"))
    hs.append(os.path.abspath(__file__))                     # the flags
    return hs


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    srcp = os.path.join(CSRC, src)
    newest = max(os.path.getmtime(p) for p in [srcp] + _deps())
    if force or not os.path.exists(obj) or os.path.getmtime(obj) < newest:
        subprocess.check_call([HIPCC, *FLAGS, *FILE_FLAGS.get(src, []), "-c", srcp, "-o", obj])
    return obj


def build(force: bool = False, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, force), SOURCES))
    if force or not os.path.exists(LIB) or os.path.getmtime(LIB) < max(os.path.getmtime(o) for o in objs):
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
        os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(force="--force" in sys.argv, verbose=True)
