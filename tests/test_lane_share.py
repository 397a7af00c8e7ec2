"""The sharing of the batched form's queue on the CPU: every extension lies in
one segment, and a segment that holds any has workgroups that open it."""
import numpy as np
import pytest

import share


def check(x, cost, **kw):
    s = share.segments(x, cost, **kw)
    cus = kw.get("cus", 256)
    assert sum(s[n] for n in share.NAMES) == len(x), s
    for seg, rest, blocks in (("split", "lane", "split_blocks"),
                              ("wide_split", "wide", "wide_split_blocks")):
        if s[seg]:
            assert 1 <= s[blocks] < cus, s
        assert s[blocks] < max(cus, 1), s
    return s


@pytest.mark.parametrize("X", [7, 25, 50])
@pytest.mark.parametrize("n,steps,short", [(4000, 200_000, 50), (6000, 100_000, 50),
                                           (30_000, 250_000, 10), (4000, 200_000, 300)])
def test_many_long_and_one_short(X, n, steps, short):
    # the short one's steps are lost in a float32 sum of the long ones'
    check(np.full(n + 1, X), np.r_[np.full(n, steps), short])


@pytest.mark.parametrize("cus", [1, 2, 3, 32, 256])
def test_random_batches(cus):
    rng = np.random.default_rng(cus)
    for _ in range(120):
        x, cost = [], []
        for _ in range(int(rng.integers(1, 5))):  # groups of like extensions
            n = int(2 ** rng.uniform(0, 15))
            x.append(np.full(n, rng.choice([0, 7, 14, 15, 25, 30, 31, 50, 62, 63, 200, -1])))
            cost.append(np.full(n, int(2 ** rng.uniform(1, 23))))
        check(np.concatenate(x), np.concatenate(cost), cus=cus, by_cost=int(rng.integers(2)))


def test_narrow_class_alone():
    # its lanes run after its longest, so thousands of long ones do not wait
    # for a launch of lanes: 16,000 pairs of 10 kbp at X = 7
    rng = np.random.default_rng(1)
    length = np.exp(rng.normal(9.1, 0.47, 32_000)).clip(3000, 50_000)
    cost = (1.4 * length * rng.random(32_000)).astype(np.uint32) + 2
    s = check(np.full(32_000, 7), cost)
    assert s["solo"] + s["split"] > 8000, s


def test_narrow_class_beside_another():
    # where a 64-row class fills the chip, the narrow one's wavefronts of one
    # extension take its issue slots: 400,000 tasks at X of 7 and 25
    rng = np.random.default_rng(1)
    length = np.exp(rng.normal(9.1, 0.47, 800_000)).clip(1000, 50_000)
    cost = (1.6 * length * rng.random(800_000)).astype(np.uint32) + 2
    s = check(rng.choice([7, 25], 800_000), cost)
    assert s["narrow"] and s["solo"] < 1000, s


def test_one_workgroup_splits_nothing():
    s = check(np.full(5000, 50), np.full(5000, 20_000), cus=1)
    assert s["split"] == s["wide_split"] == 0, s


def test_no_lane_tiers():
    x = np.resize([7, 25, 33, 80, 81, 5000, -1], 7000)
    s = check(x, np.full(7000, 5000), cus=0)
    assert (s["solo"], s["first128"], s["first256"], s["invalid"]) == (2000, 2000, 2000, 1000), s
