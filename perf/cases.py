"""Performance cases: what users of the aligner have it do, through its public
entry points, on synthetic long reads.

The recipes follow the workloads the repository is benchmarked and tested on
(uniform genome, reads with independent substitutions, insertions and
deletions, seeds that are error-free 17-base windows of the template in both
reads):

  align   align_batch in its plain, batched and allocation-free forms, and a
          captured plan: one task per candidate pair or many, one X or a mix,
          unit or general scores, with or without spurious repeat-induced
          overlaps
  pairs   align_pairs: several seeds per pair, reverse-strand pairs
  overlap find_overlaps: candidate pairs from shared k-mers, one or both strands
  banded  banded_batch and banded_traceback over whole reads
  serve   a request server, host arrays in, host arrays out

Inputs are drawn on the GPU from the seed alone.
"""
import math

import numpy as np
import torch

import paper_2001_10049_amd as xd

K = 17
DEV = "cuda"

# ---- cases -------------------------------------------------------------------

_READS = dict(genome=4_600_000, mean=10_000, sd=5_000, lmin=1_000, lmax=50_000, err=0.05)


def listed():
    return [
        # the smallest batch form: a pipeline stage that may not allocate hands
        # over 1,000 short-read pairs at a strict X (the repository's c1)
        dict(name="noalloc_1k_x7", kind="align", form="noalloc", tasks=1_000, x="7",
             genome=200_000, mean=3_500, sd=800, lmin=2_000, lmax=5_000, err=0.05),
        # a service replaying one captured plan of a few dozen pairs: latency
        dict(name="plan_64_x7_25", kind="align", form="plan", tasks=64, x="7,25",
             genome=500_000, mean=10_000, sd=5_000, lmin=1_000, lmax=100_000, err=0.05),
        # the headline workload: 100,000 pairs of a 30x E. coli sized read set,
        # one seed each, in one plain call (c2)
        dict(name="plain_100k_x25", kind="align", form="plain", tasks=100_000, x="25", **_READS),
        # the same in the batched form
        dict(name="batched_100k_x25", kind="align", form="batched", tasks=100_000, x="25",
             **_READS),
        # every seed of many pairs, a mix of X (c3)
        dict(name="batched_400k_mix", kind="align", form="batched", tasks=400_000, x="7,25,50",
             all_seeds=True, **_READS),
        # a repeat-rich genome, a tenth of the tasks spurious: bands widen past
        # the first window (c4)
        dict(name="batched_150k_spurious", kind="align", form="batched", tasks=150_000, x="25",
             all_seeds=True, spurious=0.1, genome=4_500_000, mean=12_000, sd=6_000, lmin=1_000,
             lmax=60_000, err=0.04),
        # a general scoring scheme with a mid-sized odd batch
        dict(name="batched_20011_scores", kind="align", form="batched", tasks=20_011, x="50",
             match=2, mismatch=-3, gap=-2, genome=1_150_000, mean=10_000, sd=5_000, lmin=1_000,
             lmax=50_000, err=0.05),
        # multi-seed pairs on both strands, seeds at least 1 kbp apart
        dict(name="pairs_30k_1kbp", kind="pairs", tasks=30_000, x="25", min_dist=1_000,
             max_seeds=0, genome=1_150_000, mean=10_000, sd=5_000, lmin=1_000, lmax=50_000,
             err=0.05),
        # candidate pairs of the whole 30x read set
        dict(name="overlap_138m", kind="overlap", strands=1, k=17, m=8, **_READS),
        # banded scores of whole reads, and the same with the alignment paths
        dict(name="banded_50k_w32", kind="banded", trace=False, tasks=50_000, w=32,
             genome=1_150_000, mean=10_000, sd=5_000, lmin=1_000, lmax=50_000, err=0.05),
        dict(name="trace_10k_w32", kind="banded", trace=True, tasks=10_000, w=32,
             genome=500_000, mean=10_000, sd=5_000, lmin=1_000, lmax=50_000, err=0.05),
        # a serving burst: 24 requests of 1 to 10,000 pairs, X per request (c5)
        dict(name="serve_24_requests", kind="serve", requests=24, max_size=10_000, x="7,25",
             genome=2_300_000, mean=10_000, sd=5_000, lmin=1_000, lmax=100_000, err=0.05),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["align"] * 6 + ["pairs", "overlap", "banded", "banded", "serve"])
    mean = rng.choice([3_500, 10_000, 10_000, 12_000])
    reads = dict(genome=_log(rng, 200_000, 4_600_000), mean=mean,
                 sd=800 if mean == 3_500 else mean // 2, lmin=1_000,
                 lmax=5_000 if mean == 3_500 else rng.choice([50_000, 60_000, 100_000]),
                 err=rng.choice([0.04, 0.05]))
    if kind == "align":
        form = rng.choice(["plain", "batched", "batched", "plan", "noalloc"])
        c = dict(kind=kind, form=form, tasks=_log(rng, 16, 100_000),
                 x=rng.choice(["7", "25", "25", "50", "7,25", "7,25,50"]), **reads)
        c["all_seeds"] = rng.random() < 0.5
        if rng.random() < 0.2:
            c["spurious"] = 0.1
        if rng.random() < 0.2:
            c["match"], c["mismatch"], c["gap"] = rng.choice([(2, -3, -2), (1, -1, -2), (5, -4, -8)])
        return c
    if kind == "pairs":
        return dict(kind=kind, tasks=_log(rng, 100, 30_000), x=rng.choice(["7", "25"]),
                    min_dist=rng.choice([17, 1_000]), max_seeds=rng.choice([0, 1, 4]),
                    **dict(reads, genome=min(reads["genome"], 1_150_000)))
    if kind == "overlap":
        return dict(kind=kind, strands=rng.choice([1, 2]), k=rng.choice([17, 21, 31]),
                    m=rng.choice([2, 4, 8]), **reads)
    if kind == "banded":
        trace = rng.random() < 0.5
        return dict(kind=kind, trace=trace, tasks=_log(rng, 16, 10_000 if trace else 50_000),
                    w=rng.randint(4, 48), **dict(reads, genome=min(reads["genome"], 1_150_000)))
    return dict(kind=kind, requests=rng.randint(1, 24), max_size=_log(rng, 16, 10_000),
                x=rng.choice(["7", "25", "7,25"]), **dict(reads, genome=min(reads["genome"], 2_300_000)))


# ---- inputs ------------------------------------------------------------------


class _Reads:
    """A read set on the GPU: codes back to back, and for each template base of
    each read its position in the read and whether a seed may start there."""

    def __init__(self, c, gen, depth=30):
        G = c["genome"]
        genome = torch.randint(0, 4, (G,), generator=gen, device=DEV, dtype=torch.uint8)
        self.rep_len, self.copies = 5_000, None
        if c.get("spurious"):
            # 1 of 9 bases sits in a copy of one of few segments
            n_copy = max(4, G // 45_000)
            n_src = max(1, n_copy // 10)
            src = torch.randint(0, 4, (n_src, self.rep_len), generator=gen, device=DEV,
                                dtype=torch.uint8)
            slot = torch.randperm(G // self.rep_len, generator=gen, device=DEV)[:n_copy]
            self.copies = (slot * self.rep_len).sort().values
            self.seg = torch.arange(n_copy, device=DEV) % n_src
            at = (self.copies[:, None] + torch.arange(self.rep_len, device=DEV)).reshape(-1)
            genome[at] = src[self.seg].reshape(-1)
        n = max(2, int(depth * G / c["mean"]))
        s2 = math.log(1 + (c["sd"] / c["mean"]) ** 2)
        L = torch.exp(torch.randn(n, generator=gen, device=DEV, dtype=torch.float64) *
                      math.sqrt(s2) + math.log(c["mean"]) - s2 / 2)
        L = L.clamp(c["lmin"], min(c["lmax"], G // 2)).long()
        start, by = (torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) *
                     (G - L)).long().sort()
        L = L[by]
        self.n, self.start, self.end = n, start, start + L
        self.toff = L.cumsum(0) - L                       # first template base of each read
        total = int(L.sum())
        tpos = torch.arange(total, device=DEV) + (start - self.toff).repeat_interleave(L)
        code = genome[tpos]
        p = c["err"]
        r = torch.rand(total, generator=gen, device=DEV)
        gone, sub = r < p, (r >= p) & (r < 2 * p)
        ins = torch.rand(total, generator=gen, device=DEV) < p
        code = torch.where(sub, (code + torch.randint(1, 4, (total,), generator=gen, device=DEV,
                                                      dtype=torch.uint8)) & 3, code)
        count = (~gone).to(torch.int8) + ins.to(torch.int8)
        out = torch.cumsum(count, 0, dtype=torch.int64)
        codes = torch.randint(0, 4, (int(out[-1]),), generator=gen, device=DEV, dtype=torch.uint8)
        out -= count
        keep = ~gone
        codes[out[keep]] = code[keep]
        first = out[self.toff]
        self.off = first
        self.length = torch.cat([first[1:], torch.tensor([codes.numel()], device=DEV)]) - first
        self.rpos = (out - first.repeat_interleave(L)).int()
        bad = torch.cumsum((gone | sub | ins).int(), 0, dtype=torch.int32)
        flag = torch.zeros(total, dtype=torch.bool, device=DEV)
        flag[1:total - K] = bad[K:total - 1] == bad[:total - K - 1]
        left = self.end.repeat_interleave(L) - (start - self.toff).repeat_interleave(L) - \
            torch.arange(total, device=DEV)
        self.seedable = flag & (left >= K)
        self.codes = codes

    def store(self, twins=False, flipped=False):
        codes, off, length = self.codes, self.off, self.length
        if twins or flipped:
            at = torch.arange(codes.numel(), device=DEV)
            end = (2 * off + length - 1).repeat_interleave(length)
        if flipped:  # every other read comes from the reverse strand
            odd = (torch.arange(self.n, device=DEV) % 2 == 1).repeat_interleave(length)
            codes = torch.where(odd, 3 - codes[end - at], codes)
        if twins:  # read n + r is read r reverse-complemented
            codes = torch.cat([codes, 3 - codes[end - at]])
            off = torch.cat([off, off + self.codes.numel()])
            length = torch.cat([length, length])
        return xd.ReadStore(codes.cpu().numpy(), off.cpu().numpy().astype(np.uint64),
                            length.cpu().numpy().astype(np.uint32))

    def pairs(self, n, gen, min_overlap=1_000):
        """Up to n distinct read pairs (r < s by template start) that overlap."""
        hi = torch.searchsorted(self.start, self.end - min_overlap, right=True)
        cnt = (hi - torch.arange(self.n, device=DEV) - 1).clamp(min=0)
        cum = cnt.cumsum(0)
        total = int(cum[-1])
        t = torch.randperm(total, generator=gen, device=DEV)[:2 * n + 64]
        r = torch.searchsorted(cum, t, right=True)
        s = r + 1 + (t - (cum[r] - cnt[r]))
        ok = torch.minimum(self.end[r], self.end[s]) - self.start[s] >= min_overlap
        return r[ok], s[ok]

    def seeds(self, r, s, chunk=24_000_000):
        """Every shared seed of each pair, in order: (pair, pos in r, pos in s)."""
        lo, hi = self.start[s], torch.minimum(self.end[r], self.end[s]) - K
        span = (hi - lo).clamp(min=0)
        cum = span.cumsum(0).cpu()
        got, a = [], 0
        while a < r.numel():
            base = int(cum[a - 1]) if a else 0
            b = max(a + 1, int(torch.searchsorted(cum, torch.tensor(base + chunk), right=True)))
            sp = span[a:b]
            q = torch.arange(a, b, device=DEV).repeat_interleave(sp)
            u = torch.arange(q.numel(), device=DEV) - (sp.cumsum(0) - sp).repeat_interleave(sp)
            tr = self.toff[r[a:b]] + lo[a:b] - self.start[r[a:b]]
            ts = self.toff[s[a:b]]
            ir, is_ = tr.repeat_interleave(sp) + u, ts.repeat_interleave(sp) + u
            hit = (self.seedable[ir] & self.seedable[is_]).nonzero().squeeze(1)
            got.append(torch.stack([q[hit], self.rpos[ir[hit]].long(), self.rpos[is_[hit]].long()]))
            a = b
        return torch.cat(got, 1)

    def spurious(self, n, gen):
        """Tasks whose reads cover two different copies of one segment."""
        out, have = [], 0
        while have < n:
            m = 2_000_000
            a = torch.randint(0, self.copies.numel(), (m,), generator=gen, device=DEV)
            b = torch.randint(0, self.copies.numel(), (m,), generator=gen, device=DEV)
            u = torch.randint(0, self.rep_len - K, (m,), generator=gen, device=DEV)
            ok = (a != b) & (self.seg[a] == self.seg[b])
            side = []
            for cp in (a, b):
                g = self.copies[cp] + u
                r = torch.searchsorted(self.start, g, right=True) - 1 - \
                    torch.randint(0, 40, (m,), generator=gen, device=DEV)
                ok &= r >= 0
                r = r.clamp(min=0)
                ok &= self.end[r] >= g + K
                t = (self.toff[r] + g - self.start[r]).clamp(max=self.seedable.numel() - 1)
                ok &= self.seedable[t]
                side += [r, self.rpos[t].long()]
            ok &= side[0] != side[2]
            got = torch.stack([side[0], side[2], side[1], side[3]])[:, ok]
            out.append(got)
            have += got.shape[1]
        return torch.cat(out, 1)[:, :n]


def _apart(q, pa, dist):
    """Marks each seed at least `dist` past the one before it in its pair."""
    keep = torch.ones_like(q, dtype=torch.bool)
    keep[1:] = (q[1:] != q[:-1]) | (pa[1:] - pa[:-1] >= dist)
    return keep


def _tasks(R, c, n, gen):
    """n alignment tasks (ra, rb, pa, pb): one random seed of each of n pairs,
    or, with all_seeds, a sample of the seeds of fewer pairs."""
    n_sp = int(n * c.get("spurious", 0))
    need = n - n_sp
    r, s = R.pairs(max(8, need // 8) if c.get("all_seeds") else need + need // 4 + 32, gen)
    q, pa, pb = R.seeds(r, s)
    if c.get("all_seeds"):
        keep = _apart(q, pa, K)
        q, pa, pb = q[keep], pa[keep], pb[keep]
        pick = torch.randperm(q.numel(), generator=gen, device=DEV)
    else:
        cnt = torch.bincount(q, minlength=r.numel())
        first = cnt.cumsum(0) - cnt
        pick = (first + (torch.rand(cnt.numel(), generator=gen, device=DEV,
                                    dtype=torch.float64) * cnt).long())[cnt > 0]
        pick = pick[torch.randperm(pick.numel(), generator=gen, device=DEV)]
    pick = pick[torch.arange(need, device=DEV) % pick.numel()]
    t = torch.stack([r[q[pick]], s[q[pick]], pa[pick], pb[pick]])
    if n_sp:
        t = torch.cat([t, R.spurious(n_sp, gen)], 1)
    t = t[:, torch.randperm(n, generator=gen, device=DEV)]
    flip = torch.rand(n, generator=gen, device=DEV) < 0.5  # which read comes first
    t = torch.where(flip, t[[1, 0, 3, 2]], t)
    return t[:2].T.contiguous().int(), t[2:].T.contiguous().int()


def _xs(c, n, gen):
    xs = [int(v) for v in c["x"].split(",")]
    if len(xs) == 1:
        return None, xs[0]
    pick = torch.randint(0, len(xs), (n,), generator=gen, device=DEV)
    return torch.tensor(xs, dtype=torch.int32, device=DEV)[pick], 0


def _scores(c):
    return dict(match=c.get("match", 1), mismatch=c.get("mismatch", -1), gap=c.get("gap", -1))


def _inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    R = _Reads(case, gen)
    pairs, seeds = _tasks(R, case, case["tasks"], gen)
    x, xs = _xs(case, case["tasks"], gen)
    return R, pairs, seeds, x, xs


def prepare(case, seed):
    kind = case["kind"]
    if kind == "align":
        R, pairs, seeds, x, xs = _inputs(case, seed)
        s = dict(case=case, store=R.store(), pairs=pairs, seeds=seeds, x=x, x_scalar=xs)
        if case["form"] == "plan":
            s["plan"] = xd.Plan(s["store"], pairs, seeds, x=x, x_scalar=xs, k=K, **_scores(case))
        if case["form"] == "noalloc":
            n = case["tasks"]
            s["out"] = dict(score=torch.empty(n, dtype=torch.int32, device=DEV),
                            beg=torch.empty((n, 2), dtype=torch.int32, device=DEV),
                            end=torch.empty((n, 2), dtype=torch.int32, device=DEV),
                            status=torch.empty(n, dtype=torch.int32, device=DEV),
                            cells=torch.empty(n, dtype=torch.int64, device=DEV))
        return s
    gen = torch.Generator(device=DEV).manual_seed(seed)
    R = _Reads(case, gen)
    if kind == "overlap":
        return dict(case=case, store=R.store(flipped=case["strands"] == 2))
    if kind == "pairs":
        r, t = R.pairs(case["tasks"], gen)
        q, pa, pb = R.seeds(r, t)
        keep = _apart(q, pa, K)
        q, pa, pb = q[keep], pa[keep], pb[keep]
        # every other pair lists its second read's reverse-complemented twin
        used, q = torch.unique(q, return_inverse=True)
        used = used[:case["tasks"]]
        keep = q < used.numel()
        q, pa, pb = q[keep], pa[keep], pb[keep]
        r, t = r[used], t[used]
        rc = (torch.arange(used.numel(), device=DEV) % 2).to(torch.uint8)
        pairs = torch.stack([r, t + rc.long() * R.n], 1).int()
        cnt = torch.bincount(q, minlength=used.numel())
        seed_off = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), cnt.cumsum(0)])
        return dict(case=case, store=R.store(twins=True), pairs=pairs, rc=rc, seed_off=seed_off,
                    seeds=torch.stack([pa, pb], 1).int().contiguous(), n_seeds=int(q.numel()),
                    x=int(case["x"]))
    if kind == "banded":
        pairs, seeds = _tasks(R, case, case["tasks"], gen)
        return dict(case=case, store=R.store(), pairs=pairs, seeds=seeds)
    # serve: request sizes log-uniform in [1, max_size], one X each
    rng = np.random.default_rng(case["requests"])
    sizes = np.exp(rng.uniform(0, math.log(case["max_size"] + 1), case["requests"])).astype(int)
    sizes = np.clip(sizes, 1, case["max_size"])
    rng = np.random.default_rng(seed)
    pairs, seeds = _tasks(R, case, int(sizes.sum()), gen)
    pairs, seeds = pairs.cpu().numpy().astype(np.uint32), seeds.cpu().numpy().astype(np.uint32)
    cut = np.concatenate([[0], np.cumsum(sizes)])
    xs = rng.choice([int(v) for v in case["x"].split(",")], case["requests"])
    store = R.store()
    return dict(case=case, store=store, server=xd.Server(store, hbm_budget_bytes=2 << 30, k=K),
                requests=[(pairs[a:b], seeds[a:b], int(v))
                          for a, b, v in zip(cut[:-1], cut[1:], xs)])


# ---- one pass ----------------------------------------------------------------


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "align":
        if c["form"] == "plan":
            return state["plan"].launch()
        return xd.align_batch(state["store"], state["pairs"], state["seeds"], x=state["x"],
                              x_scalar=state["x_scalar"], k=K, out=state.get("out"),
                              persistent=c["form"] == "batched", noalloc=c["form"] == "noalloc",
                              **_scores(c))
    if kind == "pairs":
        return xd.align_pairs(state["store"], state["pairs"], state["seed_off"], state["seeds"],
                              rc=state["rc"], x_scalar=state["x"], min_dist=c["min_dist"],
                              max_seeds=c["max_seeds"], k=K, n_seeds=state["n_seeds"])
    if kind == "overlap":
        # room for any read set of this size; the outputs filled up to it
        room = (30 * c["genome"] // 16, 30 * c["genome"] // 4)
        out = xd.find_overlaps(state["store"], k=c["k"], m=c["m"], strands=c["strands"],
                               capacity=room)
        # what the filters saw on the way is a diagnostic, not a result
        n = out.pop("counts")
        pad = torch.nn.functional.pad
        return dict(pairs=pad(out["pairs"], (0, 0, 0, room[0] - n["pairs"])),
                    rc=pad(out["rc"], (0, room[0] - n["pairs"])),
                    seed_off=pad(out["seed_off"], (0, room[0] - n["pairs"])),
                    seeds=pad(out["seeds"], (0, 0, 0, room[1] - n["seeds"])),
                    counts=[n[f] for f in ("kmers", "non_singletons", "retained", "occurrences",
                                           "seeds", "pairs")])
    if kind == "banded":
        if not c["trace"]:
            return xd.banded_batch(state["store"], state["pairs"], state["seeds"],
                                   w_scalar=c["w"], k=K)
        out = xd.banded_traceback(state["store"], state["pairs"], state["seeds"],
                                  w_scalar=c["w"], k=K)
        # a row's entries past n_ops are not written
        col = torch.arange(out["ops"].shape[1], device=DEV, dtype=torch.int32)
        out["ops"].masked_fill_(col >= out["n_ops"][:, None], -1)
        return out
    ids = [state["server"].submit(p, s, x_scalar=x) for p, s, x in state["requests"]]
    got = [state["server"].poll(i, timeout_ms=-1) for i in ids]
    return {f: np.concatenate([g[f].view(np.int64 if f == "cells" else np.int32) for g in got])
            for f in ("score", "beg", "end", "status", "cells")}


# ---- what a pass cannot do without --------------------------------------------


def work(case):
    """Bytes: the packed reads, task arrays and results once.  Flops: eight
    integer operations per evaluated cell (three compares and selects, the
    diagonal's add, the gap's add, the live test), about X cells on each
    antidiagonal of an overlap; for the candidate stage, ten per k-mer."""
    bases = 30 * case["genome"]
    kind = case["kind"]
    if kind == "overlap":
        return dict(bytes=bases / 4 + bases / 8 * 24, flops=10.0 * bases)
    if kind == "banded":
        cells = case["tasks"] * case["mean"] * (2 * case["w"] + 1)
        b = case["tasks"] * (40 + (2 * case["mean"] / 8 if case["trace"] else 0))
        return dict(bytes=bases / 4 + b, flops=8.0 * cells)
    n = case["tasks"] if kind != "serve" else \
        case["requests"] * (case["max_size"] - 1) / math.log(case["max_size"] + 1)
    per_pair = 1.0
    if kind == "pairs":  # seeds kept per pair
        per_pair = case["max_seeds"] or max(1.0, case["mean"] / 2 / max(case["min_dist"], 700))
    xs = [int(v) for v in case["x"].split(",")]
    # an overlap of two reads is about half a read long on average
    cells = n * per_pair * 1.1 * case["mean"] * sum(xs) / len(xs) / max(1, case.get("match", 1))
    return dict(bytes=min(bases, n * 2 * case["mean"]) / 4 + n * per_pair * 52,
                flops=8.0 * cells)


# ---- the definition, in 64-bit integers ----------------------------------------


def _extend(codes, oa, da, m, ob, db, n, X, sc, Q=256):
    """X-drop extensions by the definition, one row of a table per extension:
    antidiagonal by antidiagonal, rows base .. base + Q - 1 of each.  Returns
    (best, i, j, cells), or None when a band outgrows the table."""
    M, MM, G = sc
    E, low = m.numel(), -(1 << 40)
    col = torch.arange(Q, device=DEV)[None]
    base = torch.zeros(E, 1, dtype=torch.int64, device=DEV)
    S1 = torch.full((E, Q), low, dtype=torch.int64, device=DEV)
    S1[:, 0] = 0
    S2 = torch.full_like(S1, low)
    T, bi, bd, cells = (torch.zeros(E, dtype=torch.int64, device=DEV) for _ in range(4))
    down = lambda v: torch.cat([torch.full_like(v[:, :1], low), v[:, :-1]], 1)  # noqa: E731
    top = codes.numel() - 1
    steps = int((m + n).max()) if E else 0
    for d in range(1, steps + 1):
        i = base + col
        j = d - i
        inside = (i <= m[:, None]) & (j <= n[:, None]) & (j >= 0)
        ca = codes[(oa[:, None] + da[:, None] * (i - 1)).clamp(0, top)]
        cb = codes[(ob[:, None] + db[:, None] * (j - 1)).clamp(0, top)]
        dg, up = down(S2), down(S1)
        seen = ((dg > low) | (up > low) | (S1 > low)) & inside
        s = torch.maximum(torch.maximum(up, S1) + G, dg + torch.where(ca == cb, M, MM))
        live = seen & (s >= (T - X)[:, None])
        S2, S1 = S1, torch.where(live, s, low)
        cells += seen.sum(1)
        v = S1.max(1)
        better = v.values > T
        first = (S1 == v.values[:, None]).to(torch.int8).argmax(1)
        bi = torch.where(better, base[:, 0] + first, bi)
        bd = torch.where(better, d, bd)
        T = torch.maximum(T, v.values)
        if d % 32 == 0:
            any2 = (S1 > low) | (S2 > low)
            if not bool(any2.any()):
                break
            if bool(any2[:, Q - 40:].any()) and bool((any2[:, :40].any(1) & any2[:, Q - 40:].any(1)).any()):
                return None
            sl = torch.where(any2.any(1), any2.to(torch.int8).argmax(1), 0)[:, None]
            src = col + sl
            ok = src < Q
            src = src.clamp(max=Q - 1)
            S1 = torch.where(ok, S1.gather(1, src), low)
            S2 = torch.where(ok, S2.gather(1, src), low)
            base = base + sl
    return T, bi, bd - bi, cells


def exact(case, seed):
    """Small align cases by the definition; None where that takes too long
    (results are whole numbers, and are the same for every implementation)."""
    if case["kind"] != "align" or case["tasks"] > 2_000:
        return None
    R, pairs, seeds, x, xs = _inputs(case, seed)
    ra, rb = pairs[:, 0].long(), pairs[:, 1].long()
    pa, pb = seeds[:, 0].long(), seeds[:, 1].long()
    X = (x.long() if x is not None else torch.full_like(ra, xs)).repeat(2)
    la, lb = R.length[ra], R.length[rb]
    m, n = torch.cat([pa, la - pa - K]), torch.cat([pb, lb - pb - K])
    if int((m + n).max()) > 60_000:
        return None
    sc = tuple(_scores(case).values())
    A, B = R.off[ra], R.off[rb]
    one = torch.ones_like(pa)
    step = torch.cat([-one, one])
    codes = R.codes.long()
    got = _extend(codes, torch.cat([A + pa - 1, A + pa + K]), step, m,
                  torch.cat([B + pb - 1, B + pb + K]), step, n, X, sc)
    if got is None:
        return None
    best, bi, bj, cells = (v.view(2, -1) for v in got)
    u = torch.arange(K, device=DEV)
    eq = codes[(A + pa)[:, None] + u] == codes[(B + pb)[:, None] + u]
    score = best.sum(0) + torch.where(eq, sc[0], sc[1]).sum(1)
    return dict(score=score.int(),
                beg=torch.stack([pa - bi[0], pb - bj[0]], 1).int(),
                end=torch.stack([pa + K + bi[1], pb + K + bj[1]], 1).int(),
                status=torch.zeros_like(score).int(), cells=cells.sum(0))
