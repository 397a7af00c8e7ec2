"""The shares of the lane tiers on the GPU against the oracle: batches whose
extensions lie in the segments a test is about (tests/share.py says which)."""
import numpy as np
import pytest

import oracle
from helpers import rand_codes, workload_from
from test_gpu_parity import assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2001_10049_amd as xd  # noqa: E402

LANES = 12288  # tasks (two extensions each) from which the lane tiers run


def check(w, at, label, scheme=(1, -1, -1), tuning=None):
    """Tasks at[] of w (negative: a refused one), in the batched form."""
    print(label, len(at), flush=True)
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
    assert_same(got, ref, label=label)


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
