// The batched form's queue: the sort key of an extension, the segments the
// sorted extensions fall into, and how a lane class's extensions are shared out
// among one lane, several lanes and a wavefront each.  Host and device code: the
// kernels k_bin_* of xdrop.hip do it with a workgroup, the tests with a loop.
#pragma once

#include <math.h>

#include "lane_core.h"

namespace xd {
namespace queue {

// classes (by X), 73 length bins each, in 512 bins (the last class is the
// invalid tasks', whose length does not matter)
constexpr int kCostBins = 73;
constexpr int kBins = 512;
enum { kClsNarrow = 0, kClsLane, kCls64, kClsWide, kCls128, kCls256, kClsInvalid };

// queue segments, in queue order (with lane tiers kSeg64 holds the
// extensions of the narrow and the 64-row class that run one per wavefront
// and kSegLong those of the 96-row class; kSegSplit and kSegWideSplit those
// that run in several lanes each)
enum { kSeg64 = 0, kSegSplit, kSegLane, kSegNarrow, kSegLong, kSegWideSplit, kSegWide, kSeg128,
       kSeg256, kSegInvalid, kSegEnd,
       kSplitBlocks,      // workgroups of kSegSplit's extensions
       kWideSplitBlocks,  // and of kSegWideSplit's
       kSegWords };

struct BinRule {
  int32_t x_tier1, x_tier2;  // X limits of the 64- and 128-cell first tiers
  int32_t by_cost;           // 0: keep task order inside a tier
  uint32_t lanes;            // workgroups of a lane tier's launch, one per CU (0: no lane tiers)
};

// Length bin of an estimated antidiagonal count, 6 per octave from 64 on.
XD_HD uint32_t cost_bin(uint32_t cost) {
  if (cost < 64u) return 0u;
  const uint32_t ex = 31u - (uint32_t)__builtin_clz(cost);
  const uint32_t sub = (((cost >> (ex - 3)) & 7u) * 6u) >> 3;
  const uint32_t b = 1u + (ex - 6u) * 6u + sub;
  return b < (uint32_t)kCostBins ? b : (uint32_t)kCostBins - 1u;
}
// the middle and the end of a length bin
XD_HD uint32_t bin_cost(uint32_t cb) {
  if (cb == 0) return 32u;
  const uint32_t ex = (cb - 1) / 6, sub = (cb - 1) % 6;  // (sub: 2, 1, 1, 2, 1, 1 eighths)
  return (4u << ex) * (uint32_t)((0x1f1d1a171512ull >> (8 * sub)) & 255u);
}
XD_HD float bin_end(uint32_t cb) {
  if (cb == 0) return 64.f;
  const uint32_t ex = (cb - 1) / 6, sub = (cb - 1) % 6;
  return (float)(4u << ex) * (float)((0x201e1c181614ull >> (8 * sub)) & 255u);
}

// Sort key of an extension of a valid task: class from X (its first tier), then
// the length bin of the estimated antidiagonal count `cost`, longest first.
XD_HD uint32_t bin_key(const BinRule& R, int32_t X, uint32_t cost) {
  uint32_t cls = X <= R.x_tier1 ? kCls64 : X <= R.x_tier2 ? kCls128 : kCls256;
  if (R.lanes && X <= lane::x_limit(7))  // the planes a lane needs
    cls = X <= lane::x_limit(5) ? kClsNarrow : X <= lane::x_limit(6) ? kClsLane : kClsWide;
  else if (R.lanes && cls == kCls64)
    cls = kCls128;
  return cls * kCostBins + (R.by_cost ? kCostBins - 1 - cost_bin(cost) : 0u);
}

// How a lane class's extensions are shared out: the longest run one per
// wavefront, the next in several lanes each, the rest in one lane, because
// the fewer share a wavefront the sooner a step is done and the more
// instructions it costs.  A CU runs one workgroup of single lanes or of split
// extensions, and the wavefronts of the longest beside it, ahead of it in
// priority.  The narrow class's lanes alone come after its longest, in a launch
// of their own, so its times add up; where the 64-row class runs beside its
// longest (x.beside), what they issue is not hidden behind the longest's chain
// either (400,000 tasks of 10 kbp at X of 7 and 25: 15.4 ms, 14.8 so).  In issue
// slots of a SIMD (vector instructions; a wavefront's share from timing 12,500 to
// 100,000 pairs of 1.3 to 20 kbp reads with shares of 9 to 12):
struct LaneCost {
  float lane_step, split_step, solo_step;  // from one step of an extension to the next
  float solo;                              // one step's share of the instructions
  uint32_t split_group;                    // split extensions a workgroup holds
};
XD_HD LaneCost lane_cost(uint32_t cls) {
  return cls == kClsNarrow ? LaneCost{82.f, 120.f, 25.f, 10.5f, 128u}
         : cls == kClsLane ? LaneCost{160.f, 120.f, 25.f, 12.f, 128u}
                           : LaneCost{260.f, 130.f, 45.f, 20.f, 64u};
}

// The classes that are shared out: narrow, 64 rows, 96 rows, the first two as one.
constexpr int kKinds = 4;
XD_HD uint32_t cls_of(int kind) {
  return kind == 0 ? kClsNarrow : kind == 2 ? kClsWide : kClsLane;
}

// What split_time reads of a class: for each length bin, longest first, the
// first bin from it on that is not empty, and the steps and extensions of the
// bins before it (whole numbers: in 32-bit floats a short bin is lost beside
// long ones, and its extensions with it).
struct ClassBins {
  uint32_t next[kCostBins + 1], before[kCostBins + 1];
  uint64_t sum[kCostBins + 1];
  uint32_t beside;  // (narrow class) extensions of the 64-row class
};

XD_HD void class_bins(const uint32_t* h, int kind, ClassBins& x) {
  constexpr uint32_t N = kCostBins;
  const uint32_t* c = h + cls_of(kind) * N;
  const uint32_t* c2 = h + kClsNarrow * N;
  auto count = [&](uint32_t q) { return c[q] + (kind == 3 ? c2[q] : 0u); };
  uint64_t v = 0;
  uint32_t n = 0, nx = N;
  for (uint32_t q = 0; q < N; ++q) {
    x.sum[q] = v;
    x.before[q] = n;
    n += count(q);
    v += (uint64_t)count(q) * bin_cost(N - 1 - q);
  }
  x.sum[N] = v;
  x.before[N] = n;
  x.beside = 0;
  if (kind == 0)
    for (uint32_t q = 0; q < N; ++q) x.beside += h[kClsLane * N + q];
  x.next[N] = N;
  for (uint32_t q = N; q-- > 0;) {
    if (count(q)) nx = q;
    x.next[q] = nx;
  }
}

// Estimated end of a class (kind) whose first s1 length bins run alone and whose
// next s2 - s1 run split, and the workgroups the latter get of cus: as many as
// hold those longer than half the longest at once, and make the average load
// no more than the longest one's, at least one and not all of them (infinite
// where that is no number).
XD_HD float split_time(const ClassBins& x, int kind, uint32_t s1, uint32_t s2, float cus,
                       float& groups) {
  constexpr uint32_t N = kCostBins;
  const LaneCost c = lane_cost(cls_of(kind));
  auto longest = [&](uint32_t from, uint32_t to) -> float {
    const uint32_t q = x.next[from];
    return q < to ? bin_end(N - 1 - q) : 0.f;
  };
  const float solo = (float)x.sum[s1] * c.solo / (4.f * cus),
              split = (float)(x.sum[s2] - x.sum[s1]), rest = (float)(x.sum[N] - x.sum[s2]);
  const float l0 = longest(0, s1), l1 = longest(s1, s2), l2 = longest(s2, N);
  // (six bins an octave)
  const uint32_t half = s2 < x.next[s1] + 6u ? s2 : x.next[s1] + 6u;
  const bool any = x.before[s2] > x.before[s1];
  groups = any ? fminf(ceilf(fmaxf(split / l1, (float)(x.before[half] - x.before[s1])) /
                             (float)c.split_group), cus - 1.f)
               : 0.f;
  if (any && groups < 1.f) return INFINITY;
  const float t1 = any ? fmaxf(l1, split / (groups * (float)c.split_group)) : 0.f;
  const float t2 = fmaxf(l2, rest / (256.f * (cus - groups)));
  if (kind == 0 && x.beside)
    return fmaxf(l0 * c.solo_step, t1 * c.split_step + solo + t2 * c.lane_step);
  if (kind == 0) return fmaxf(l0 * c.solo_step, t1 * c.split_step + solo) + t2 * c.lane_step;
  return fmaxf(l0 * c.solo_step, fmaxf(t1 * c.split_step, t2 * c.lane_step) + solo);
}

// Shares of one class, numbered: candidate q runs its first q / (N + 1) bins
// alone and those up to q % (N + 1) alone or split.  The smallest rank wins.
constexpr uint32_t kCandidates = (kCostBins + 1) * (kCostBins + 1);
XD_HD uint64_t share_rank(const ClassBins& x, int kind, uint32_t q, uint32_t cus) {
  const uint32_t s1 = q / (kCostBins + 1), s2 = q % (kCostBins + 1);
  if (s1 > s2) return ~0ull;
  float g;
  const float e = split_time(x, kind, s1, s2, (float)cus, g);
  return (uint64_t)__builtin_bit_cast(uint32_t, e) << 32 | q;
}

// The chosen shares: bins [0, alone), [alone, split) and the rest of each kind.
struct Shares {
  uint32_t alone[kKinds] = {0, 0, 0, 0}, split[kKinds] = {0, 0, 0, 0};
  float groups[kKinds] = {0.f, 0.f, 0.f, 0.f}, time[kKinds] = {0.f, 0.f, 0.f, 0.f};

  XD_HD void choose(const ClassBins& x, int kind, uint64_t rank, uint32_t cus) {
    const uint32_t q = (uint32_t)rank;
    alone[kind] = q / (kCostBins + 1);
    split[kind] = q % (kCostBins + 1);
    time[kind] = split_time(x, kind, alone[kind], split[kind], (float)cus, groups[kind]);
  }
  // The narrow class's lanes run after the 64-row class's and its own longest, in a
  // launch of their own; when that would take longer than running them all in 64
  // rows (two chains of steps instead of one), they join that class.  32,000 pairs
  // of 10 kbp at X of 7 and 25: 4.0 ms against 5.8; at X = 7, with the times added
  // up and without (and the packed kernels): 4.0, 4.6 (4.7), 16,000 pairs 3.4, 4.2
  // (3.1).
  XD_HD bool merged() const { return time[0] > 0.f && time[3] < time[0] + time[1]; }
};

// where bin b comes in the queue (a permutation of the bins)
XD_HD uint32_t slot_of(uint32_t b, const Shares& S, bool merged) {
  constexpr uint32_t N = kCostBins;
  const uint32_t s0 = S.alone[0], s1 = S.alone[1], t0 = S.split[0], t1 = S.split[1];
  const uint32_t c = b / N, cls = c < (uint32_t)kClsInvalid ? c : (uint32_t)kClsInvalid,
                 q = b - cls * N;
  if (cls == kCls64) return q;
  if (merged && (cls == kClsLane || cls == kClsNarrow))
    return N + 2 * q + (cls == kClsNarrow ? 1u : 0u);
  if (cls == kClsLane)
    return q < s1 ? N + q : q < t1 ? N + s1 + s0 + (q - s1) : N + t1 + t0 + (q - t1);
  if (cls == kClsNarrow)
    return q < s0 ? N + s1 + q : q < t0 ? N + t1 + s0 + (q - s0) : 2 * N + t0 + (q - t0);
  if (cls == kClsWide) return 3 * N + q;  // (its longest come first already)
  if (cls == kCls128) return 4 * N + q;
  return b;  // the classes from 256 cells on keep their place
}

// seg: the segments' first entries, then the workgroups of split extensions.
// upto: extensions in the first so many slots.
template <class F>
XD_HD void segments(const Shares& S, bool merged, uint32_t n_ext, uint32_t cus, F&& upto,
                    uint32_t* seg) {
  constexpr uint32_t N = kCostBins;
  const uint32_t s0 = S.alone[0], s1 = S.alone[1], t0 = S.split[0], t1 = S.split[1];
  seg[kSeg64] = 0;
  seg[kSegSplit] = upto(merged ? N + 2 * S.alone[3] : N + s1 + s0);
  seg[kSegLane] = upto(merged ? N + 2 * S.split[3] : N + t1 + t0);
  seg[kSegNarrow] = upto(merged ? 3 * N : 2 * N + t0);
  seg[kSegLong] = upto(3 * N);
  seg[kSegWideSplit] = upto(3 * N + S.alone[2]);
  seg[kSegWide] = upto(3 * N + S.split[2]);
  seg[kSeg128] = upto(4 * N);
  seg[kSeg256] = upto(5 * N);
  seg[kSegInvalid] = upto(6 * N);
  seg[kSegEnd] = n_ext;
  seg[kSplitBlocks] = seg[kWideSplitBlocks] = 0;
  if (cus) {
    seg[kSplitBlocks] =
        (uint32_t)(merged ? S.groups[3] : fminf(S.groups[0] + S.groups[1], (float)cus - 1.f));
    seg[kWideSplitBlocks] = (uint32_t)S.groups[2];
  }
}

}  // namespace queue
}  // namespace xd
