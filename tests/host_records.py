"""Builds and loads tests/host_records.cpp, the planner's records for CPU tests."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2602_24082_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(maxsize=1)
def lib() -> ctypes.CDLL:
    tmp = tempfile.mkdtemp(prefix="pp_records_")
    so = os.path.join(tmp, "host_records.so")
    # the launch wrappers stay unresolved: no record needs one, and symbols bind on first use
    cmd = [build.hipcc(), *build.COMMON, "-O1", "-shared", os.path.join(HERE, "host_records.cpp"), "-o", so]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    L = ctypes.CDLL(so, mode=os.RTLD_LAZY)
    L.rec_stage_blocks.restype = ctypes.c_int64
    return L
