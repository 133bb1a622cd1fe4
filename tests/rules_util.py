"""The host-side dispatch rules of csrc/ts_common.h through ctypes: dispatch_rules.cpp compiled once per process."""
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile
from types import SimpleNamespace

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(maxsize=None)
def rules():
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    rocm = os.path.dirname(os.path.dirname(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")))
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "dispatch_rules.so")
        subprocess.check_call([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                               "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2411_02886_amd", "csrc"),
                               os.path.join(ROOT, "tests", "dispatch_rules.cpp"), "-o", so])
        L = ctypes.CDLL(so)
    L.rule_attn_streams.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_int]
    L.rule_stream_span.argtypes = [ctypes.c_long, ctypes.c_int]
    L.rule_zeroed_bytes.restype = ctypes.c_long
    return L


def decode_attention(B, H, H_kv, D, total):
    """(streamed, splits) of a bf16 decode attention over lists of `total` entries."""
    L, chunks = rules(), (total + 63) // 64
    if not L.rule_attn_streams(H // H_kv, D, H_kv * B, total):
        wgs = chunks * H_kv * B
        nch = min(4 if wgs >= 8192 else 1, chunks)
        return False, (chunks + nch - 1) // nch
    span = L.rule_stream_span(H_kv * B, total)
    return True, (total + span - 1) // span


TESTED, MASKED, WHOLE = 0, 1, 2


def score_shape(B, H, H_kv, D, max_len, dense, scan):
    """The matrix-core score launch of a call: shared (by the batch), grid, RR, SR, NU, lds, run_stat_bytes; None on the vector kernel."""
    if not rules().rule_score_cores(B, H, H_kv, D, max_len, int(dense), scan):
        return None
    out = (ctypes.c_long * 7)()
    rules().rule_score_shape(B, H, H_kv, D, max_len, int(dense), scan, out)
    return SimpleNamespace(**dict(zip(("shared", "grid", "RR", "SR", "NU", "lds", "run_stat_bytes"), out)))


def score_share(B, H, H_kv, D, max_len, dense, lens, skip):
    """Waves of a shared score grid that have work: rows of workgroup, wave, sequence, x, n, first tile, tiles, uw."""
    grid = score_shape(B, H, H_kv, D, max_len, dense, WHOLE if skip is None else MASKED).grid
    out = np.zeros((grid, 4, 6), np.int32)
    lens = np.asarray(lens, np.int32)
    skip_b = np.zeros(B, np.uint8) if skip is None else np.asarray(skip, np.uint8)
    rules().rule_score_share(B, H, H_kv, D, max_len, int(dense), int(skip is not None), lens.ctypes.data_as(ctypes.c_void_p),
                             skip_b.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p))
    wg, wave = np.nonzero(out[:, :, 0] >= 0)
    return np.column_stack([wg, wave, out[wg, wave]])


def score_units(B, H, H_kv, D, max_len, dense, lens, skip):
    """Units that a workgroup of the shared grid takes, over the fewest it could: more than 1 once the grid is full."""
    shape = score_shape(B, H, H_kv, D, max_len, dense, WHOLE if skip is None else MASKED)
    rows = score_share(B, H, H_kv, D, max_len, dense, lens, skip)
    return int(rows[0, 7]) // (4 // shape.NU if skip is None else 1)
