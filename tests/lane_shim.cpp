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

template <int P, int W>
static int run(const uint8_t* A, int32_t la, const uint8_t* B, int32_t lb, int32_t oa, int32_t ob,
               int32_t m, int32_t n, int32_t X, uint32_t flags, int64_t* out) {
  std::vector<Chunk> pa = planar(A, la), pb = planar(B, lb);
  Task t{pa.data() + kGuard, pb.data() + kGuard, (la + 31) / 32, (lb + 31) / 32, oa, ob, m, n, X,
         flags};
  Core<P, W> c;
  c.clear();
  c.start(X);
  int32_t d = 0, base = -Core<P, W>::Q / 2, bi = 0, dstar = 0, lo, hi, events = 0;
  bool fresh = true;
  for (;;) {
    ++events;
    if (!c.extent(lo, hi)) break;
    if (hi - lo > Core<P, W>::kMaxSpan) return 0;
    if (fresh || c.edge()) {
      int32_t s = fresh ? 0 : ((lo + hi + 1) >> 1) - Core<P, W>::Q / 2;
      s = s < -31 ? -31 : s > 31 ? 31 : s;
      c.slide(s);
      base += s;
      c.refill(t, d, base);
    } else {
      c.feed(t, d, base);
    }
    fresh = false;
    int32_t k = 0;
    do {
      c.group(k);
      k += Core<P, W>::kGroup;
    } while (k < Core<P, W>::kMaxSteps && !c.edge());
    c.settle(d, base, bi, dstar);
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

extern "C" int lane_extend(int planes, const uint8_t* A, int32_t la, const uint8_t* B, int32_t lb,
                           int32_t oa, int32_t ob, int32_t m, int32_t n, int32_t X,
                           uint32_t flags, int64_t* out) {
  switch (planes) {
    case 5: return run<5, 1>(A, la, B, lb, oa, ob, m, n, X, flags, out);
    case 6: return run<6, 2>(A, la, B, lb, oa, ob, m, n, X, flags, out);
    case 7: return run<7, 3>(A, la, B, lb, oa, ob, m, n, X, flags, out);
  }
  return -1;
}
