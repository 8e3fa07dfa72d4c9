"""Builds and loads tests/host_records.cpp, the planner's records for CPU tests."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

from paper_2602_24082_amd import binding, build

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
    L.rec_stage_blocks.restype = L.rec_list.restype = ctypes.c_int64
    return L


_I4 = "<i4"
_RECORDS = [  # in the order of the enumeration in host_records.cpp, laid out as in csrc/pp_plan.h
    *[(n, [(f, _I4) for f in fields.split()]) for n, fields in (
        ("fwd_items", "tok0 q0 q_end P valid kt_off kt_cnt row"), ("fwd_ktiles", "k0 cls"),
        ("dq_items", "tok0 q0 q_end P valid kt_off kt_cnt row"), ("dq_ktiles", "k0 cls"),
        ("kv_items", "tok0 k0 k_end valid q_begin q_end row part"), ("cut_items", "tok0 k0 k_end valid q_begin q_end row part"),
        ("cut_parts", "n_begin n_end slot pad"), ("cut_splits", "tok0 k0 k_end slot0 parts pad"))],
    ("row_kb0", _I4), ("panels", [("off", _I4), ("len", _I4)]), ("seg_lo", _I4), ("seg_hi", _I4),
    ("lp_rows", [("logit_row", "<i8"), ("label_off", _I4), ("label_cnt", _I4)]), ("lp_labels", _I4),
    ("lp_resp", [("tok_begin", _I4), ("len", _I4), ("out", _I4), ("pad", _I4)]), ("lp_label_out", _I4), ("lp_row_item", _I4),
    ("rm_slot_row", "<i8"), ("rm_rows", [("row", "<i8"), ("slot_off", _I4), ("slot_cnt", _I4)]), ("rm_slots", _I4)]


def records(pack, name, hq=4, hkv=2, d=64):
    """The plan's record list `name` as a numpy (structured) array."""
    what = [n for n, _ in _RECORDS].index(name)
    dt = np.dtype(_RECORDS[what][1])
    h = binding._DescHolder(pack)
    n = lib().rec_list(h.ref, what, hq, hkv, d, None, ctypes.c_int64(0))
    assert n >= 0 and n % dt.itemsize == 0, (name, n)
    out = np.empty(n // dt.itemsize, dt)
    if n:
        assert lib().rec_list(h.ref, what, hq, hkv, d, out.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(n)) == n
    return out
