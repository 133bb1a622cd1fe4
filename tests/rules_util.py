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
    L.rule_stream_span.argtypes = [ctypes.c_long, ctypes.c_int]
    return L
