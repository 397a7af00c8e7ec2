// The lane tiers' wavefront: 64 / S extensions at a time, S lanes each, in bit
// planes (lane_core.h), fed from a work queue.
//
// All lanes step together.  Every kMaxSteps antidiagonals, or earlier when a
// band comes near its window's edge, the wave stops for an "event":
// extensions that ended leave their result and the next ones take their
// lanes, a band too wide for the window is handed to the next tier with its
// state, the windows are centred on their bands if one of them was near an
// edge, and the next 32 bases of each sequence are read.  Descriptions of the
// next extensions wait in LDS, read several at a time, so an event does not
// wait for the chain of loads that sets an extension up.
#pragma once

#include "lane_core.h"
#include "xdrop_device.h"

namespace xd {
namespace lane {

// extensions whose descriptions are read ahead, for S lanes each
constexpr int fifo_size(int S) { return S == 1 ? 32 : S == 2 ? 16 : S == 4 ? 8 : 4; }
// LDS record of one description (words)
enum { kLe = 0, kLraLo, kLraHi, kLrbLo, kLrbHi, kLca, kLcb, kLoa, kLob, kLm, kLn, kLX, kLflags,
       kLstLo, kLstHi, kLWords };
// with one lane an extension (W words), also the bases its first steps need
constexpr int fifo_words(int W, int S) { return kLWords + (S == 1 ? 4 * (W + 1) : 0); }
constexpr int lds_words(int W, int S) { return fifo_size(S) * fifo_words(W, S); }

// An extension to run: its task and, when it comes from a narrower window,
// the state that left (null: from its seed).
struct Item {
  uint32_t e;
  Task t;
  const uint8_t* state;
};

// number of lanes below this one that are set in mask
__device__ __forceinline__ uint32_t rank_in(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// f over the S lanes of a group (f commutative and associative)
template <int S, class F>
__device__ __forceinline__ int32_t over_group(int32_t v, F f) {
  if constexpr (S >= 2) v = f(v, (int32_t)dpp<0xB1>((uint32_t)v));
  if constexpr (S >= 4) v = f(v, (int32_t)dpp<0x4E>((uint32_t)v));
  if constexpr (S >= 8) v = f(v, (int32_t)dpp<0x141>((uint32_t)v));
  if constexpr (S >= 16) v = f(v, (int32_t)dpp<0x140>((uint32_t)v));
  if constexpr (S >= 32) {
    auto r = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    v = f((int32_t)r[0], (int32_t)r[1]);
  }
  return v;
}

// Runs the work wk supplies: wk.grab(n, idx) claims up to n consecutive
// entries (wave-uniform), wk.describe(idx, item) reads one, wk.done(e, result)
// takes a result, and wk.overflow(e) claims a place in the next tier's list
// for e, returning where its state goes (null: it is not kept).
template <int P, int W, int S, class Work>
__device__ __forceinline__ void run(Work& wk, uint32_t* lds, const Chunk* planes) {
  using C = Core<P, W, S>;
  constexpr int Q = C::Q;
  constexpr uint32_t kFifo = (uint32_t)fifo_size(S);
  constexpr int kRec = fifo_words(W, S);
  const int lane = lane_id();
  const int s = lane & (S - 1);
  const int32_t part = C::kLaneRows * s;  // the lane's first row in the window
  const bool first = s == 0;
  C c;
  c.clear(s);
  Item it;
  it.e = 0;
  // idle lanes read the first read (planes is its chunk 0)
  it.t = Task{planes, planes, 0, 0, 0, 0, 0, 0, 0, 0};
  it.state = nullptr;
  int32_t d = 0, base = 0, bi = 0, dstar = 0;  // base: of the lane's rows
  bool active = false, more = true;
  typename C::Ahead ahead = {};
  int32_t k = C::kMaxSteps;  // steps of the last period
  uint32_t have = 0, pos = 0;  // descriptions in LDS, and the next of them
  int32_t lo, hi;
  auto band = [&]() -> bool {
    c.extent(lo, hi);
    lo += part;
    hi += hi < 0 ? 0 : part;
    lo = over_group<S>(lo, [](int32_t a, int32_t b) { return min(a, b); });
    hi = over_group<S>(hi, [](int32_t a, int32_t b) { return max(a, b); });
    return hi >= 0;
  };
  for (;;) {
    bool live = band();
    const bool ended = active && !live;
    const bool wide = active && live && hi - lo > C::kMaxSpan;
    bool fresh = false;
    const uint64_t leave = ballot64(ended || wide);
    if (leave | (more ? ballot64(!active) : 0ull)) {
      auto add = [](int32_t a, int32_t b) { return a + b; };
      uint64_t cells;
      if constexpr (kWholeCount<S>)
        cells = (uint32_t)over_group<S>((int32_t)c.cnt, add);
      else
        cells = count_of((uint32_t)over_group<S>((int32_t)(c.cnt & 0xffffu), add),
                         (uint32_t)over_group<S>((int32_t)(c.cnt >> 16), add));
      if (ended && first) {
        ExtOut o;
        o.best = c.thr - (d + 1);
        o.bi = bi;
        o.bj = dstar - bi;
        o.flags = kExtDone;
        o.cells = cells;
        wk.done(it.e, o);
      }
      if (ballot64(wide)) {
        uint64_t dst = 0;
        if (wide && first) dst = (uint64_t)(uintptr_t)wk.overflow(it.e);
        if constexpr (S > 1) {
          const int src = lane & ~(S - 1);
          const uint32_t a = (uint32_t)__shfl((int)(uint32_t)dst, src, 64);
          const uint32_t b = (uint32_t)__shfl((int)(uint32_t)(dst >> 32), src, 64);
          dst = ((uint64_t)b << 32) | a;
        }
        if (wide && dst) {
          c.save_words(s, (uint8_t*)dst);
          if (first) {
            StateHead h = {d, base, c.thr, bi, dstar, (uint32_t)cells, (uint32_t)(S * W),
                           (uint32_t)(cells >> 32)};
            *(StateHead*)dst = h;
          }
        }
      }
      if (ended || wide) {
#pragma unroll
        for (int w = 0; w < W; ++w) c.L[w] = c.LD[w] = 0;
        active = false;
      }
      // hand the waiting descriptions to the idle groups
      for (;;) {
        const uint64_t need = ballot64(!active && first);
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
            uint32_t* r = lds + lane * kRec;
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
            r[kLstLo] = (uint32_t)(uintptr_t)x.state;
            r[kLstHi] = (uint32_t)((uintptr_t)x.state >> 32);
            if constexpr (S == 1) {
              typename C::Bases b;
              C::bases(x.t, 0, -Q / 2, b);
#pragma unroll
              for (int w = 0; w <= W; ++w) {
                r[kLWords + 4 * w] = b.a0[w];
                r[kLWords + 4 * w + 1] = b.a1[w];
                r[kLWords + 4 * w + 2] = b.b0[w];
                r[kLWords + 4 * w + 3] = b.b1[w];
              }
            }
          }
          wave_lds_fence();
        }
        const uint32_t at = pos + rank_in(need) - (first ? 0u : active ? 0u : 1u);
        if (!active && at < have) {
          const uint32_t* r = lds + at * kRec;
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
          const uint8_t* st = (const uint8_t*)(((uint64_t)r[kLstHi] << 32) | r[kLstLo]);
          c.start((int32_t)r[kLX], s);
          d = 0;
          base = part - Q / 2;
          bi = dstar = 0;
          if (Work::kResumes && st) {  // continue from a narrower window's state
            const StateHead h = *(const StateHead*)st;
            c.load_words(s, (int32_t)h.words, st);
            d = h.d;
            base = h.base + part;
            bi = h.bi;
            dstar = h.dstar;
            c.thr = h.thr;
            c.cnt = kWholeCount<S> ? (first ? h.cells : 0u) : count_part<S>(h, s);
          }
          active = fresh = true;
          if constexpr (S == 1 && !Work::kResumes) {
            typename C::Bases b;
#pragma unroll
            for (int w = 0; w <= W; ++w) {
              b.a0[w] = r[kLWords + 4 * w];
              b.a1[w] = r[kLWords + 4 * w + 1];
              b.b0[w] = r[kLWords + 4 * w + 2];
              b.b1[w] = r[kLWords + 4 * w + 3];
            }
            c.refill(it.t, 0, -Q / 2, b);
          }
        }
        pos = min(have, pos + (uint32_t)__builtin_popcountll(need));
      }
      if (!ballot64(active)) break;
      if (Work::kResumes && ballot64(fresh)) live = band();
    }
    // every window is centred when one band has come near an edge; otherwise
    // the windows only need new bases at their ends
    const bool move = ballot64(c.edge() != 0) != 0;
    if (move) {
      int32_t by = live && active && (Work::kResumes || !fresh) ? ((lo + hi + 1) >> 1) - Q / 2 : 0;
      by = min(31, max(-31, by));
      c.slide(by);
      base += by;
    }
    // (with one lane an extension the fresh ones have theirs already)
    if (move || k != C::kMaxSteps || ((S > 1 || Work::kResumes) && ballot64(fresh))) {
      typename C::Bases b;
      C::bases(it.t, d, base, b);
      c.refill(it.t, d, base, b);
    } else if (!fresh) {
      c.feed(it.t, d, base, ahead);
    }
    // what the next event feeds the windows with, unless it comes early or
    // moves them
    C::look_ahead(it.t, d + C::kMaxSteps, base + C::kMaxSteps / 2, ahead);
    if constexpr (Work::kResumes) {
      // lists are in no order: the wavefronts that may end last go first
      const int32_t ahead_of = active ? 2 * min(it.t.m, it.t.n) - d : 0;
      if (ballot64(ahead_of > 24576))
        __builtin_amdgcn_s_setprio(3);
      else if (ballot64(ahead_of > 16384))
        __builtin_amdgcn_s_setprio(2);
      else if (ballot64(ahead_of > 8192))
        __builtin_amdgcn_s_setprio(1);
      else
        __builtin_amdgcn_s_setprio(0);
    }
    k = 0;
    do {
      c.group(k);
      k += C::kGroup;
    } while (k < C::kMaxSteps && !ballot64(c.edge() != 0));
    int32_t row = c.settle(base);
    row = over_group<S>(row, [](int32_t a, int32_t b) { return min(a, b); });
    if (row < 1 << 30) {
      bi = row;
      dstar = d + c.bk + 1;
    }
    d += k;
    base += k >> 1;
  }
}

}  // namespace lane
}  // namespace xd
