"""The lane tiers and the rules that choose them, on the GPU against the oracle:
X at the ends of each plane count, bands that outgrow every window up to the
last one, batches on both sides of each rule, the reverse strand, plans."""
import numpy as np
import pytest

import oracle
import synth
from helpers import mutate_codes, rand_codes, workload_from
from oracle import pairs as op
from test_gpu_pairs import gpu_pairs, multiseed_pairs, same
from test_gpu_parity import assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2001_10049_amd as xd  # noqa: E402

LANES = 12288  # tasks (two extensions each) from which the lane tiers run


def check(w, n, form="persistent", scheme=(1, -1, -1), x_scalar=None, label=""):
    """w's tasks over and over, n in all, against the oracle's w."""
    print(label, form, n, flush=True)
    xs = w.x if x_scalar is None else np.full(w.n_tasks, x_scalar, np.int32)
    ref = oracle.align_workload(w, x=xs, match=scheme[0], mismatch=scheme[1], gap=scheme[2])
    at = np.arange(n) % w.n_tasks
    ref = {k: ref[k][at] for k in ("status", "score", "beg", "end", "cells")}
    many = w.subset(at)
    store = xd.ReadStore.from_workload(w)
    pairs, seeds, x = xd.workload_tensors(many, "cuda")
    x = None if x_scalar is not None else x
    kw = dict(x=x, x_scalar=x_scalar or 0, k=w.k, match=scheme[0], mismatch=scheme[1],
              gap=scheme[2])
    outs = []
    if form == "plan":
        plan = xd.Plan(store, pairs, seeds, **kw)
        for _ in range(3):
            out = plan.launch()
            torch.cuda.synchronize()
            outs.append({k: v.cpu().numpy() for k, v in out.items()})
        plan.close()
    else:
        out = xd.align_batch(store, pairs, seeds, persistent=form == "persistent", **kw)
        torch.cuda.synchronize()
        outs.append({k: v.cpu().numpy() for k, v in out.items()})
    store.close()
    for got in outs:
        assert_same(got, ref, label=label)


def short_reads(seed=4, n=400):
    """Reads of 17 to 900 bases: related, equal, of one base, of two bases,
    unrelated; seeds anywhere, reads of the seed alone, refused tasks."""
    rng = np.random.default_rng(seed)
    reads, tasks = [], []
    for q in range(n):
        a = rand_codes(rng, 17 if q % 29 == 0 else int(rng.integers(17, 900)))
        b = mutate_codes(rng, a, float(rng.choice([0.02, 0.1, 0.25])))
        if q % 5 == 1:
            b = a.copy()
        elif q % 9 == 2:
            a[:], b[:] = q & 3, q & 3
        elif q % 9 == 4:
            a &= 1
            b = rand_codes(rng, 700) & 1
        elif q % 9 == 6:
            b = rand_codes(rng, int(rng.integers(17, 900)))
        if len(b) < 17:
            b = a.copy()
        pa = int(rng.integers(0, len(a) - 16))
        pb = min(pa, len(b) - 17) if q % 3 else int(rng.integers(0, len(b) - 16))
        if q % 31 == 7:
            pb = len(b)
        reads += [a, b]
        tasks.append((2 * q, 2 * q + 1, pa, pb, 0))
    return workload_from(reads, tasks)


@pytest.mark.parametrize("x", [(0,), (14,), (15,), (30,), (31,), (62,), (63,), (7, 25),
                               (0, 1, 7, 13, 14, 15, 16, 29, 30, 31, 32, 61, 62, 63, 200)])
def test_plane_counts(x):
    w = short_reads()
    w.x = np.resize(np.array(x, np.int32), w.n_tasks)
    check(w, LANES + 77, label="x %s" % (x,))


def flanks(seed, n, length, x):
    """Two-letter reads with a planted seed: bands widen all along."""
    rng = np.random.default_rng(seed)
    reads, tasks = [], []
    for q in range(n):
        a, b = rand_codes(rng, length) & 1, rand_codes(rng, length - 13 * q) & 1
        pa, pb = int(rng.integers(0, 60)), int(rng.integers(0, 60))
        b[pb:pb + 17] = a[pa:pa + 17]
        reads += [a, b]
        tasks.append((2 * q, 2 * q + 1, pa, pb, x[q % len(x)]))
    return workload_from(reads, tasks)


@pytest.mark.parametrize("n", [LANES, 36000])
def test_outgrown_windows(n):
    # few go straight to 512 rows; past 65,536 of them each window in turn
    check(flanks(6, 60, 1800, (7, 14, 25, 30, 50, 62)), n, label="outgrown")


def test_past_the_last_window():
    # bands of more than 1,024 rows, one side of the seed short, among many
    # ordinary extensions
    w = flanks(7, 2, 62000, (62,))
    s = short_reads(5, 300)
    s.x = np.resize(np.array([7, 25, 50], np.int32), s.n_tasks)
    codes = [w.codes[int(o):int(o) + int(l)] for o, l in zip(w.off, w.length)]
    codes += [s.codes[int(o):int(o) + int(l)] for o, l in zip(s.off, s.length)]
    t = [(int(a), int(b), int(p), int(q), int(x)) for a, b, p, q, x in
         zip(w.ra, w.rb, w.pa, w.pb, w.x)]
    t += [(int(a) + 4, int(b) + 4, int(p), int(q), int(x)) for a, b, p, q, x in
          zip(s.ra, s.rb, s.pa, s.pb, s.x)]
    both = workload_from(codes, t)
    wide = oracle.extend(codes[0][int(w.pa[0]) + 17:], codes[1][int(w.pb[0]) + 17:], 62,
                         with_stats=True)[4]["width_max"]
    assert wide > 1024
    # the wide ones once, the others over and over
    at = np.concatenate([[0, 1], 2 + np.arange(LANES) % s.n_tasks])
    ref = oracle.align_workload(both)
    store = xd.ReadStore.from_workload(both)
    xd.profile_enable(True)
    xd.profile_read(reset=True)
    pairs, seeds, x = xd.workload_tensors(both.subset(at), "cuda")
    out = xd.align_batch(store, pairs, seeds, x=x, k=both.k, persistent=True)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    prof = xd.profile_read(reset=True)
    xd.profile_enable(False)
    store.close()
    assert_same(got, {k: ref[k][at] for k in got}, label="past the last window")
    assert prof["to_band"] > 0, prof


@pytest.mark.parametrize("form,n", [("persistent", LANES - 1), ("plan", LANES - 1),
                                    ("persistent", LANES), ("plan", LANES), ("plain", LANES),
                                    ("plain", 2999), ("plain", 3000)])
def test_batch_sizes(form, n):
    w = synth.config("c3-small")
    check(w.subset(np.arange(min(w.n_tasks, 700))), n, form, label="sizes")


@pytest.mark.parametrize("scheme,limit", [((1, -1, -1), 32), ((2, -3, -2), 64),
                                          ((5, -4, -8), 224), ((1, -1, -20), 437)])
@pytest.mark.parametrize("form", ["plain", "persistent"])
def test_first_windows(scheme, limit, form):
    # X up to which an extension starts in the narrowest window, and one more
    w = short_reads(8, 200)
    for x in (limit, limit + 1):
        check(w, 500, form, scheme, x_scalar=x, label="first %s x %d" % (scheme, x))
    w.x = np.resize(np.array([limit - 1, limit, limit + 1, 2 * limit], np.int32), w.n_tasks)
    check(w, 3100, form, scheme, label="first %s mixed" % (scheme,))


def test_reverse_strand_in_lanes():
    d = multiseed_pairs()
    n = len(d["pairs"])
    reps = LANES // len(d["seeds"]) + 2
    kept = np.tile(np.arange(n), reps)
    size = np.diff(d["seed_off"].astype(np.int64))
    many = dict(d, pairs=d["pairs"][kept], rc=d["rc"][kept], x=d["x"][kept],
                seeds=np.tile(d["seeds"], (reps, 1)),
                seed_off=np.concatenate([[0], np.cumsum(size[kept])]).astype(np.uint64))
    ref = op.align_pairs(d["codes"], d["off"], d["length"], d["pairs"], d["seed_off"],
                         d["seeds"], rc=d["rc"], x=d["x"], min_dist=0, max_seeds=0)
    store = xd.ReadStore(d["codes"], d["off"], d["length"])
    got = gpu_pairs(many, store, many["rc"], many["pairs"][:, 1], 0, 0)
    store.close()
    same(got, {k: np.asarray(v)[kept] for k, v in ref.items()}, "reverse strand")


def test_many_reads():
    # more reads than the planes' kernel has workgroups
    rng = np.random.default_rng(11)
    reads = [rand_codes(rng, int(n)) for n in rng.integers(17, 60, 70001)]
    tasks = []
    for q in range(600):
        r = int(rng.integers(0, 300)) if q % 2 else 70000 - int(rng.integers(0, 5000))
        n = len(reads[r]) - 17
        tasks.append((r, r, int(rng.integers(0, n + 1)), int(rng.integers(0, n + 1)), 20))
    check(workload_from(reads, tasks), LANES, label="many reads")
