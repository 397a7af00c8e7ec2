"""Evaluated cells as the lane tiers carry them from window to window: whole up
to what the widest window of the longest reads can hold."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STEPS = 2 * (1 << 22)  # antidiagonals of two reads of the largest length


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("count") / "libcount.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wno-unknown-pragmas",
                           "-I" + os.path.join(ROOT, "paper_2001_10049_amd", "csrc"),
                           "-o", so, os.path.join(ROOT, "tests", "count_shim.cpp")])
    lib = ctypes.CDLL(so)
    lib.lane_count.restype = ctypes.c_uint64
    lib.lane_count.argtypes = [ctypes.c_int, ctypes.c_uint64, ctypes.c_uint32]
    return lib


@pytest.mark.parametrize("lanes", [4, 8, 16, 32])
def test_counts_are_whole(lib, lanes):
    before = 16 * lanes * STEPS  # the narrower window's, at most
    for cells in (0, 1, lanes - 1, lanes, 12345, before // 2 + 1, before - 1, before):
        for own in (0, 1, 0xffff, 0x10000, 32 * STEPS):
            assert lib.lane_count(lanes, cells, own) == cells + lanes * own, (cells, own)
