"""The host-side dispatch rules of csrc/ts_common.h through ctypes: dispatch_rules.cpp compiled once per process."""
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

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
