// The lane tier's arithmetic (lane_core.h) run for one lane on the CPU: one
// X-drop extension of a[0..m) against b[0..n), with the same window moves and
// refills as the kernel.  Returns 1, or 0 when the band outgrew the window.
#include <stdint.h>
#include <string.h>

#include <vector>

#include "lane_core.h"

using namespace xd::lane;

static std::vector<Chunk> planar(const uint8_t* s, int32_t len) {
  const int32_t nc = (len + 31) / 32;
  std::vector<Chunk> v((size_t)nc + 2 * kGuard, Chunk{0xdeadbeefu, 0x12345678u});
  for (int32_t c = 0; c < nc; ++c) {
    Chunk w{0, 0};
    for (int t = 0; t < 32 && 32 * c + t < len; ++t) {
      w.p0 |= (uint32_t)(s[32 * c + t] & 1) << t;
      w.p1 |= (uint32_t)(s[32 * c + t] >> 1) << t;
    }
    v[kGuard + c] = w;
  }
  return v;
}

// One window: from the seed, or from the state a narrower one left at state.
// On overflow leaves its own state there.
template <int P, int W>
static int run(const Task& t, std::vector<uint8_t>& state, bool resume, int64_t* out) {
  Core<P, W> c;
  c.clear(0);
  c.start(t.X, 0);
  int32_t d = 0, base = -Core<P, W>::Q / 2, bi = 0, dstar = 0, lo, hi, events = 0;
  bool fresh = true;
  typename Core<P, W>::Ahead ahead;
  if (resume) {
    StateHead h;
    memcpy(&h, state.data(), sizeof(h));
    c.load_words(0, (int32_t)h.words, state.data());
    d = h.d;
    base = h.base;
    bi = h.bi;
    dstar = h.dstar;
    c.thr = h.thr;
    c.cnt = h.cells;
  }
  for (;;) {
    ++events;
    if (!c.extent(lo, hi)) break;
    if (hi - lo > Core<P, W>::kMaxSpan) {
      const StateHead h = {d, base, c.thr, bi, dstar, c.cnt, (uint32_t)W, 0u};
      state.assign(state_bytes(W), 0);
      memcpy(state.data(), &h, sizeof(h));
      c.save_words(0, state.data());
      return 0;
    }
    if (c.edge()) {
      int32_t s = ((lo + hi + 1) >> 1) - Core<P, W>::Q / 2;
      s = s < -31 ? -31 : s > 31 ? 31 : s;
      c.slide(s);
      base += s;
      fresh = true;
    }
    if (fresh) {
      typename Core<P, W>::Bases x;
      c.bases(t, d, base, x);
      c.refill(t, d, base, x);
    } else {
      c.feed(t, d, base, ahead);
    }
    c.look_ahead(t, d + Core<P, W>::kMaxSteps, base + Core<P, W>::kMaxSteps / 2, ahead);
    fresh = false;
    int32_t k = 0;
    do {
      c.group(k);
      k += Core<P, W>::kGroup;
    } while (k < Core<P, W>::kMaxSteps && !c.edge());
    const int32_t row = c.settle(base);
    if (row < 1 << 30) {
      bi = row;
      dstar = d + c.bk + 1;
    }
    d += k;
    base += k >> 1;
  }
  out[0] = c.thr - (d + 1);
  out[1] = bi;
  out[2] = dstar - bi;
  out[3] = c.cnt;
  out[4] = events;
  return 1;
}

// planes 5, 6, 7: windows of 32, 64, 96 rows.  chain: what outgrows the window
// goes on in the 96-row one (out[5]: 1 when it did).
extern "C" int lane_extend(int planes, int chain, const uint8_t* A, int32_t la, const uint8_t* B,
                           int32_t lb, int32_t oa, int32_t ob, int32_t m, int32_t n, int32_t X,
                           uint32_t flags, int64_t* out) {
  std::vector<Chunk> pa = planar(A, la), pb = planar(B, lb);
  const Task t{pa.data() + kGuard, pb.data() + kGuard, (la + 31) / 32, (lb + 31) / 32, oa, ob, m,
               n, X, flags};
  std::vector<uint8_t> state;
  out[5] = 0;
  int ok = planes == 5   ? run<5, 1>(t, state, false, out)
           : planes == 6 ? run<6, 2>(t, state, false, out)
                         : run<7, 3>(t, state, false, out);
  if (!ok && chain && planes < 7) {
    out[5] = 1;
    ok = run<7, 3>(t, state, true, out);
  }
  return ok;
}
