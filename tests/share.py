"""The batched form's queue segments on the CPU (tests/share_shim.cpp), for the
tests that are about the extensions of one of them."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NAMES = ("solo", "split", "lane", "narrow", "wide_solo", "wide_split", "wide", "first128",
         "first256", "invalid")
_lib = None


def _load():
    global _lib
    if _lib is None:
        so = os.path.join(tempfile.mkdtemp(), "libshare.so")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared",
                               "-Wno-unknown-pragmas",
                               "-I" + os.path.join(ROOT, "paper_2001_10049_amd", "csrc"),
                               "-o", so, os.path.join(ROOT, "tests", "share_shim.cpp")])
        _lib = ctypes.CDLL(so)
    return _lib


def segments(x, cost, limits=(32, 80), by_cost=1, cus=256):
    """Extensions in each segment, and the workgroups of the split ones, for
    extensions with these X (negative: invalid) and estimated antidiagonals."""
    x = np.ascontiguousarray(x, np.int32)
    cost = np.ascontiguousarray(cost, np.uint32)
    seg = (ctypes.c_uint32 * 13)()
    _load().queue_segments(x.ctypes.data_as(ctypes.c_void_p), cost.ctypes.data_as(ctypes.c_void_p),
                           len(x), limits[0], limits[1], by_cost, cus, seg)
    out = {name: seg[i + 1] - seg[i] for i, name in enumerate(NAMES)}
    out["split_blocks"], out["wide_split_blocks"] = seg[11], seg[12]
    return out


def of_workload(w, **kw):
    """The segments of a workload's extensions (none of its tasks refused)."""
    la, lb = w.length[w.ra].astype(np.int64), w.length[w.rb].astype(np.int64)
    pa, pb = w.pa.astype(np.int64), w.pb.astype(np.int64)
    ok = (pa + w.k <= la) & (pb + w.k <= lb)
    left, right = np.minimum(pa, pb), np.minimum(la - pa, lb - pb) - w.k
    cost = 2 * np.where(ok[:, None], np.stack([left, right], 1), 0) + 2
    x = np.where(ok, w.x, -1)
    return segments(np.repeat(x, 2), cost.reshape(-1), **kw)
