// The lane tier's wavefront: 64 extensions at a time, one per lane, in bit
// planes (lane_core.h), fed from a work queue.
//
// All lanes step together.  Every kMaxSteps antidiagonals, or earlier when a
// band comes near its window's edge, the wave stops for an "event": lanes
// whose extension ended write its result and take the next one, a band too
// wide for the window is handed to the next tier with its state, the windows
// are centred on their bands if one of them was near an edge, and the next 32
// bases of each sequence are read.  Descriptions of the next extensions wait in LDS, read
// kFifo at a time, so an event does not wait for the chain of loads that sets
// an extension up.
#pragma once

#include "lane_core.h"
#include "xdrop_device.h"

namespace xd {
namespace lane {

constexpr int kFifo = 32;  // extension descriptions read ahead
// LDS record of one description (words)
enum { kLe = 0, kLraLo, kLraHi, kLrbLo, kLrbHi, kLca, kLcb, kLoa, kLob, kLm, kLn, kLX, kLflags,
       kLWords };
constexpr int LDS_WORDS = kFifo * kLWords;

// Extension e's description from its task (Ext, per lane) and planar reads.
struct Item {
  uint32_t e;
  Task t;
};

// number of lanes below this one that are set in mask
__device__ __forceinline__ uint32_t rank_in(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint32_t read_lane(uint32_t v, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int32_t)v, l);
}

// Lane l's state at antidiagonal d as a ResumeHead and two rows of Q int32 at
// dst (global memory), in the 32-bit tiers' units (U = V + kBias0), its first
// row the lowest live one.
template <int P, int W>
__device__ __forceinline__ void save(const Core<P, W>& c, int l, int32_t d, int32_t base,
                                     int32_t lo, int32_t bi, int32_t dstar, uint8_t* dst) {
  constexpr int Q = 32 * W;
  const int lane = lane_id();
  const int32_t thr = (int32_t)read_lane((uint32_t)c.thr, l);
  const int32_t lo_l = (int32_t)read_lane((uint32_t)lo, l);
  int32_t* rows = (int32_t*)(dst + sizeof(ResumeHead));
  // bit q of a row of words (wave-uniform l, per-lane q)
  auto bit = [&](const uint32_t (&x)[W], int32_t q) -> uint32_t {
    uint32_t v = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const uint32_t s = read_lane(x[w], l);
      v = (q >> 5) == w ? s : v;
    }
    return q >= 0 && q < Q ? (v >> (q & 31)) & 1u : 0u;
  };
  auto value = [&](const uint32_t (&x)[P][W], const uint32_t (&live)[W], int32_t q) -> int32_t {
    uint32_t v = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) v |= bit(x[p], q) << p;
    // V - thr as a P-bit signed number
    const int32_t rel = (int32_t)((v - (uint32_t)thr) << (32 - P)) >> (32 - P);
    return bit(live, q) ? thr + rel + kBias0 : 0;
  };
  for (int q = lane; q < Q; q += 64) {
    rows[q] = value(c.U, c.L, q + lo_l);
    rows[Q + q] = value(c.D, c.LD, q + lo_l - 1);
  }
  if (lane == l) {
    ResumeHead h = {};
    h.d = d;
    h.base = base + lo;
    h.thr = c.thr + kBias0;
    h.bi = bi;
    h.dstar = dstar;
    h.top_prev = 0;
    h.q_rows = Q;
    h.rebased = 0;
    h.cells = c.cnt;
    *(ResumeHead*)dst = h;
  }
}

// Runs the work W supplies: W.grab(n, idx) claims up to n consecutive queue
// entries (wave-uniform count), W.describe(idx, item) reads one per lane,
// W.done(e, result) takes a lane's result, W.overflow(e, l) claims a place
// in the next tier's list for lane l's extension (wave-uniform; returns where
// its state goes, or null) and W.list(e, kept) is told when it is written.
template <int P, int W, class Work>
__device__ __forceinline__ void run(Work& wk, uint32_t* lds, const Chunk* planes) {
  using C = Core<P, W>;
  constexpr int Q = C::Q;
  const int lane = lane_id();
  C c;
  c.clear();
  Item it;
  it.e = 0;
  // idle lanes read the first read (planes is its chunk 0)
  it.t = Task{planes, planes, 0, 0, 0, 0, 0, 0, 0, 0};
  int32_t d = 0, base = 0, bi = 0, dstar = 0;
  bool active = false, more = true;
  uint32_t have = 0, pos = 0;  // descriptions in LDS, and the next of them
  for (;;) {
    int32_t lo, hi;
    const bool live = c.extent(lo, hi);
    const bool ended = active && !live;
    const bool wide = active && live && hi - lo > C::kMaxSpan;
    bool fresh = false;
    const uint64_t leave = ballot64(ended || wide);
    if (leave | (more ? ballot64(!active) : 0ull)) {
      if (ended) {
        ExtOut o;
        o.best = c.thr - (d + 1);
        o.bi = bi;
        o.bj = dstar - bi;
        o.flags = kExtDone;
        o.cells = c.cnt;
        wk.done(it.e, o);
      }
      for (uint64_t mask = ballot64(wide); mask; mask &= mask - 1) {
        const int l = __builtin_ctzll(mask);
        const uint32_t e = read_lane(it.e, l);
        uint32_t slot;
        uint8_t* dst = wk.overflow(slot);
        if (dst) save<P, W>(c, l, d, base, lo, bi, dstar, dst);
        wk.list(slot, e, dst != nullptr);
      }
      if (ended || wide) {
#pragma unroll
        for (int w = 0; w < W; ++w) c.L[w] = c.LD[w] = 0;
        active = false;
      }
      // hand the waiting descriptions to the idle lanes
      for (;;) {
        const uint64_t need = ballot64(!active);
        if (!need || !more) break;
        if (pos == have) {
          uint32_t idx;
          have = wk.grab(kFifo, idx);
          pos = 0;
          if (!have) {
            more = false;
            break;
          }
          wave_lds_fence();
          if ((uint32_t)lane < have) {
            Item x;
            wk.describe(idx + lane, x);
            uint32_t* r = lds + lane * kLWords;
            r[kLe] = x.e;
            r[kLraLo] = (uint32_t)(uintptr_t)x.t.ra;
            r[kLraHi] = (uint32_t)((uintptr_t)x.t.ra >> 32);
            r[kLrbLo] = (uint32_t)(uintptr_t)x.t.rb;
            r[kLrbHi] = (uint32_t)((uintptr_t)x.t.rb >> 32);
            r[kLca] = (uint32_t)x.t.ca;
            r[kLcb] = (uint32_t)x.t.cb;
            r[kLoa] = (uint32_t)x.t.oa;
            r[kLob] = (uint32_t)x.t.ob;
            r[kLm] = (uint32_t)x.t.m;
            r[kLn] = (uint32_t)x.t.n;
            r[kLX] = (uint32_t)x.t.X;
            r[kLflags] = x.t.flags;
          }
          wave_lds_fence();
        }
        const uint32_t at = pos + rank_in(need);
        if (!active && at < have) {
          const uint32_t* r = lds + at * kLWords;
          it.e = r[kLe];
          it.t.ra = (const Chunk*)(((uint64_t)r[kLraHi] << 32) | r[kLraLo]);
          it.t.rb = (const Chunk*)(((uint64_t)r[kLrbHi] << 32) | r[kLrbLo]);
          it.t.ca = (int32_t)r[kLca];
          it.t.cb = (int32_t)r[kLcb];
          it.t.oa = (int32_t)r[kLoa];
          it.t.ob = (int32_t)r[kLob];
          it.t.m = (int32_t)r[kLm];
          it.t.n = (int32_t)r[kLn];
          it.t.flags = r[kLflags];
          c.start((int32_t)r[kLX]);
          d = 0;
          base = -Q / 2;
          bi = dstar = 0;
          active = fresh = true;
        }
        pos = min(have, pos + (uint32_t)__builtin_popcountll(need));
      }
      if (!ballot64(active)) break;
    }
    // every window is centred when one band has come near an edge; otherwise
    // the windows only need new bases at their ends
    const bool move = ballot64(c.edge() != 0) != 0;
    if (move) {
      int32_t s = live && active && !fresh ? ((lo + hi + 1) >> 1) - Q / 2 : 0;
      s = min(31, max(-31, s));
      c.slide(s);
      base += s;
    }
    if (move || ballot64(fresh))
      c.refill(it.t, d, base);
    else
      c.feed(it.t, d, base);
    int32_t k = 0;
    do {
      c.group(k);
      k += C::kGroup;
    } while (k < C::kMaxSteps && !ballot64(c.edge() != 0));
    c.settle(d, base, bi, dstar);
    d += k;
    base += k >> 1;
  }
}

}  // namespace lane
}  // namespace xd
