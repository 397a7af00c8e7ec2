"""The rule that chooses a batch's kernels, on the CPU: each kind of batch in the
kernels that were measured the faster for it, on both sides of each line."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OUT = ("queue", "packed", "solo", "lane_blocks", "solo_blocks", "tier1", "tier2")


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("route") / "libroute.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared",
                           "-I" + os.path.join(ROOT, "paper_2001_10049_amd", "csrc"),
                           "-o", so, os.path.join(ROOT, "tests", "route_shim.cpp")])
    lib = ctypes.CDLL(so)

    def f(n, x=None, mean=10_000, batched=False, pair=True, lane=True, tiers=(32, 80)):
        a = (ctypes.c_int64 * 10)(batched, pair, lane, x is not None, x or 0, 2 * n, mean,
                                  tiers[0], tiers[1], 256)
        o = (ctypes.c_int64 * 7)()
        lib.batch_route(a, o)
        return dict(zip(OUT, o))
    return f


@pytest.mark.parametrize("n,x,mean,lane,queue", [
    # (tasks, X, mean read, lanes, through the queue)
    (1000, 25, 10_000, True, False), (2999, 25, 10_000, True, False),
    (3000, 25, 10_000, True, True), (3000, None, 10_000, True, True),
    (3000, 25, 2499, True, False), (3000, 25, 2500, True, True),
    (16_383, 25, 1300, True, False), (16_384, 25, 1300, True, True),
    (16_384, 25, 1300, False, False), (10_000_000, None, 1300, False, False),
    (500, 38, 10_000, True, False), (500, 39, 10_000, True, True), (500, 67, 1300, True, True),
    (999, 68, 1300, True, False), (1000, 68, 1300, True, True), (999, 80, 10_000, True, False),
    (2999, 81, 10_000, True, False), (2999, 112, 1300, True, False), (3000, 81, 1300, True, True),
    (100, 113, 1300, True, True), (100, 1000, 10_000, True, True),
])
def test_plain(route, n, x, mean, lane, queue):
    r = route(n, x, mean, lane=lane)
    assert r["queue"] == queue, r
    if queue:  # up to 1.2 times the limits in the narrower window
        assert (r["tier1"], r["tier2"]) == (38, 96), r


def test_plain_limits_grow_with_the_scores(route):
    assert not route(500, 72, tiers=(64, 160), pair=False, lane=False)["queue"]
    assert route(500, 80, tiers=(64, 160), pair=False, lane=False)["queue"]
    assert route(4000, 80, tiers=(64, 160), pair=False, lane=False)["tier1"] == 76


def test_batched(route):
    small, large = route(12_287, 25, batched=True), route(12_288, 25, batched=True)
    assert (small["queue"], small["solo"], small["packed"], small["lane_blocks"]) == (1, 1, 0, 0)
    assert (large["queue"], large["packed"], large["lane_blocks"]) == (1, 1, 256)
    assert (small["tier1"], small["tier2"]) == (32, 80)
    assert large["solo_blocks"] == 1024 and route(32_768, batched=True)["solo_blocks"] == 768
    other = route(18_001, 25, batched=True, lane=False)
    assert (other["packed"], other["lane_blocks"]) == (1, 0)
    general = route(50_000, 25, batched=True, pair=False, lane=False)
    assert (general["queue"], general["packed"], general["solo"]) == (1, 0, 0)


@pytest.mark.parametrize("n,x,mean,lane,kernels", [
    (18_000, 7, 10_000, True, "solo"), (18_001, 7, 10_000, True, "packed"),
    (24_575, 14, 5_000, True, "packed"), (24_576, 14, 5_000, True, "lanes"),
    (12_288, 14, 4_999, True, "lanes"), (12_288, 15, 10_000, True, "lanes"),
    (12_288, None, 10_000, True, "lanes"), (12_287, None, 10_000, True, "solo"),
    (12_288, None, 10_000, False, "packed"), (18_000, 32, 10_000, False, "solo"),
    (18_001, 32, 10_000, False, "packed"), (12_287, 33, 5_000, True, "solo"),
    (7_500, 33, 4_999, True, "solo"), (7_501, 33, 4_999, True, "packed"),
    (12_288, 33, 4_999, True, "lanes"),
])
def test_batched_kernels(route, n, x, mean, lane, kernels):
    r = route(n, x, mean, batched=True, lane=lane)
    got = "lanes" if r["lane_blocks"] else "solo" if r["solo"] else "packed"
    assert got == kernels and r["packed"] == (not r["solo"]), r
