"""The packed kernels (two extensions per wavefront in 64, 128 and 256 cells) on
the GPU against the oracle, in batches large enough to take them (12,288 tasks of
unknown X) under schemes that the lane tiers do not: walls, reads of length k,
early exits, X up to the packed limit and past it, bands that outgrow each
window and resume in the next."""
import numpy as np
import pytest

from helpers import workload_from
from test_batch_route import route  # noqa: F401
from test_gpu_lane import short_reads
from test_gpu_lane_share import check
from test_gpu_parity import band_workload, edge_workload, random_flank_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

N = 12_400
SCHEMES = [(1, -1, -2), (1, -2, -1), (1, -3, -48)]
# the first window of every extension with X > 1: by the default limits (64 cells,
# mostly), 128 cells, 256 cells
FIRST = {64: None, 128: dict(x_tier1=1, x_tier2=5000), 256: dict(x_tier1=1, x_tier2=1)}


def with_filler(w, n=N, seed=8):
    """w's tasks once, and short ones up to n tasks."""
    s = short_reads(seed, 200)
    s.x = np.resize(np.array([7, 25, 50, 90], np.int32), s.n_tasks)
    reads = [v.codes[int(o):int(o) + int(m)] for v in (w, s) for o, m in zip(v.off, v.length)]
    base = len(w.length)
    tasks = [(int(a), int(b), int(p), int(q), int(x))
             for a, b, p, q, x in zip(w.ra, w.rb, w.pa, w.pb, w.x)]
    # (a refused task of w names a read past its store: past this one's too)
    tasks = [(a if a < base else 1 << 30, b if b < base else 1 << 30, p, q, x)
             for a, b, p, q, x in tasks]
    tasks += [(int(a) + base, int(b) + base, int(p), int(q), int(x))
              for a, b, p, q, x in zip(s.ra, s.rb, s.pa, s.pb, s.x)]
    both = workload_from(reads, tasks, k=w.k)
    at = np.concatenate([np.arange(w.n_tasks), w.n_tasks + np.arange(n - w.n_tasks) % s.n_tasks])
    return both, at


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("first", sorted(FIRST))
@pytest.mark.parametrize("wl", ["edge", "band", "flank", "short"])
def test_packed_windows(route, wl, first, scheme):  # noqa: F811
    assert route(N, None, batched=True, lane=False)["packed"]
    w = {"edge": edge_workload, "band": band_workload, "flank": random_flank_workload,
         "short": lambda: short_reads(9, 300)}[wl]()
    both, at = with_filler(w)
    prof = check(both, at, "packed %d %s %s" % (first, wl, scheme), scheme, FIRST[first])
    if first == 64 and wl == "flank" and scheme == (1, -2, -1):
        assert prof["to_tier2"] and prof["to_tier3"], prof
    if first == 256:  # (X of 0 and 1 start in 64 cells)
        assert prof["to_tier3"] == 0, prof


@pytest.mark.parametrize("n", [12_287, 12_288])
def test_both_sides_of_the_line(n):
    both, at = with_filler(short_reads(10, 150), n)
    check(both, at, "line", (1, -1, -2))


@pytest.mark.parametrize("gap", [-30, -31, -47, -48, -49])
def test_large_gaps(gap):
    # the largest the packed kernels take (one group between rebases from 31
    # on), and the first that they do not
    both, at = with_filler(short_reads(11, 150))
    check(both, at, "gap %d" % gap, (1, -3, gap))
