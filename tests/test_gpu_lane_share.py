"""The shares of the lane tiers on the GPU against the oracle: batches whose
extensions lie in the segments a test is about (tests/share.py says which)."""
import numpy as np
import pytest

import oracle
import share
from helpers import mutate_codes, rand_codes, workload_from
from test_gpu_parity import assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2001_10049_amd as xd  # noqa: E402

LANES = 12288  # tasks (two extensions each) from which the lane tiers run


def check(w, at, label, scheme=(1, -1, -1), tuning=None):
    """Tasks at[] of w (negative: a refused one), in the batched form; its
    profile counters."""
    print(label, len(at), flush=True)
    xd.profile_enable(True)
    xd.profile_read(reset=True)
    many = w.subset(np.maximum(at, 0))
    many.ra = np.where(at < 0, w.n_reads, many.ra).astype(np.uint32)
    ref = oracle.align_workload(w, match=scheme[0], mismatch=scheme[1], gap=scheme[2])
    ref = {k: ref[k][np.maximum(at, 0)] for k in ("status", "score", "beg", "end", "cells")}
    ref["status"][at < 0] = oracle.TASK_BAD_READ
    ref["score"][at < 0] = np.iinfo(np.int32).min
    for k in ("beg", "end", "cells"):
        ref[k][at < 0] = 0
    pairs, seeds, x = xd.workload_tensors(many, "cuda")
    with xd.ReadStore.from_workload(w) as store:
        out = xd.align_batch(store, pairs, seeds, x=x, k=w.k, match=scheme[0],
                             mismatch=scheme[1], gap=scheme[2], persistent=True, tuning=tuning)
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy() for k, v in out.items()}
    prof = xd.profile_read(reset=True)
    xd.profile_enable(False)
    assert_same(got, ref, label=label)
    return prof


@pytest.mark.parametrize("x", [7, 25, 50])
def test_many_long_and_one_short(x):
    # beside 6,000 extensions of 200,000 antidiagonals two of 50, which a
    # 32-bit float sum of their steps does not show: every one of them has to run
    rng = np.random.default_rng(x)
    a = rand_codes(rng, 200_017)
    b = a.copy()
    hit = rng.integers(0, a.size, 20_000)
    b[hit] = rng.integers(0, 4, hit.size)
    b[100_000:100_017] = a[100_000:100_017]
    c = rand_codes(rng, 67)
    w = workload_from([a, b, c, c.copy()], [(0, 1, 100_000, 100_000, x), (2, 3, 25, 25, x)])
    check(w, np.r_[np.zeros(3000, np.int64), 1, np.full(LANES - 3001, -1)], "x %d" % x)


def tail(kind, x, seed=3):
    """600 tasks, 3 in 100 of them on reads of 2 to 12 kbp, the rest up to 1.8
    kbp: related ones, or two-letter ones whose bands widen all along."""
    rng = np.random.default_rng(seed)
    reads, tasks = [], []
    for q in range(600):
        n = int(rng.integers(2000, 12_000) if q % 33 == 7 else 2 ** rng.uniform(5, 10.8))
        if kind == "related":
            a = rand_codes(rng, n)
            b = mutate_codes(rng, a, 0.15)
            b = b if len(b) >= 17 else a.copy()
        else:
            a, b = rand_codes(rng, n) & 1, rand_codes(rng, n) & 1
        pa = int(rng.integers(0, n - 16))
        pb = min(pa, len(b) - 17)
        b[pb:pb + 17] = a[pa:pa + 17]
        reads += [a, b]
        tasks.append((2 * q, 2 * q + 1, pa, pb, x[q % len(x)]))
    return workload_from(reads, tasks)


@pytest.mark.parametrize("kind", ["related", "widening"])
@pytest.mark.parametrize("x,n,parts", [
    ((14,), 30_000, ("solo", "split")), ((14,), 90_000, ("solo", "narrow")),
    ((0, 7, 14), 90_000, ("solo", "narrow")),
    ((15,), 30_000, ("solo", "split", "lane")), ((30,), 30_000, ("solo", "split", "lane")),
    ((31,), 40_000, ("wide_solo", "wide_split", "wide")),
    ((62,), 40_000, ("wide_solo", "wide_split", "wide")),
    ((7, 25, 50), 60_000, ("solo", "split", "lane", "wide_solo", "wide_split", "wide")),
])
def test_every_share(kind, x, n, parts):
    # each class at the ends of its X, with extensions in each of its shares;
    # widening bands leave each of them for the lists with their states
    w = tail(kind, x)
    at = np.arange(n) % w.n_tasks
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    got = share.of_workload(w.subset(at), cus=cus)
    assert all(got[p] > 0 for p in parts), got
    prof = check(w, at, "%s %s" % (kind, x))
    if kind == "widening" and max(x) >= 14:
        assert prof["to_tier2"] + prof["to_tier3"] > 1000 and prof["resumed"] > 1000, prof
