"""Banded Smith-Waterman, two tasks to a wavefront, where it can go wrong: the
ends of its blocks of 128 antidiagonals, every band width, unlike tasks side by
side, the scores' ends, and the longest pair that 16 bits hold next to the
shortest that they do not."""
import numpy as np
import pytest

from helpers import mutate_codes, rand_codes, workload_from
from test_gpu_banded import assert_same, run

pytestmark = pytest.mark.gpu


def mixed(seed, n, lo, hi):
    """n tasks on related reads of lo..hi bases, some with the band partly or
    wholly outside the grid, some of equal reads, some refused."""
    rng = np.random.default_rng(seed)
    reads, tasks = [], []
    for q in range(n):
        a = rand_codes(rng, int(rng.integers(lo, hi + 1)))
        b = a.copy() if q % 5 == 0 else mutate_codes(rng, a, 0.2)
        if q % 7 == 3:
            a[:] = q & 3  # one base over and over: ties on every antidiagonal
            b[:] = q & 3
        b = b if len(b) >= 17 else a.copy()
        reads += [a, b]
        pa = int(rng.integers(0, len(a) - 16))
        pb = min(max(pa + int(rng.integers(-20, 21)), 0), len(b) - 17)
        if q % 11 == 5:
            pa, pb = len(a) - 17, 0
        if q % 13 == 6:
            pa = len(a)  # no seed fits
        tasks.append((2 * q, 2 * q + 1, pa, pb, 0))
    return workload_from(reads, tasks)


@pytest.mark.parametrize("scheme", [(1, -1, -1), (1, -127, -1), (127, -127, -127), (2, -3, -2),
                                    (3, -1, -127), (2, 0, -1), (2, 1, -1)])
@pytest.mark.parametrize("lo,hi", [(17, 90), (120, 136), (190, 400)])
def test_sizes_and_scores(scheme, lo, hi):
    rng = np.random.default_rng(lo)
    w = mixed(lo, 403, lo, hi)
    got, ref = run(w, rng.integers(0, 49, w.n_tasks).astype(np.int32), scheme)
    assert_same(got, ref, "%s %d-%d" % (scheme, lo, hi))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 16384, 16385, 16387])
def test_task_counts(n):
    w = mixed(3, min(n, 500), 17, 200)
    w = w.subset(np.arange(n) % w.n_tasks)
    got, ref = run(w, np.full(n, 11, np.int32))
    assert_same(got, ref, "n=%d" % n)


@pytest.mark.parametrize("match,fits", [(127, 516), (100, 655), (3, 21845), (1, 65535)])
def test_largest_score(match, fits):
    # equal reads reach match * length: the last that 16 bits hold, and one more
    rng = np.random.default_rng(match)
    a = rand_codes(rng, fits + 1)
    reads = [a[:fits].copy(), a, a[:fits - 1].copy(), rand_codes(rng, 300)]
    w = workload_from(reads, [(0, 0, 5, 5, 0), (1, 1, 5, 5, 0), (0, 1, 9, 9, 0), (2, 2, 0, 0, 0),
                              (3, 1, 100, 400, 0), (1, 3, 100, 100, 0)])
    ws = np.array([0, 3, 48, 32, 20, 48], np.int32)
    got, ref = run(w, ws, (match, -1, -1))
    assert ref["score"][0] == match * fits and ref["score"][1] == match * (fits + 1)
    assert_same(got, ref, "match=%d" % match)
