// X-drop extension in bit planes: one extension per lane (the arithmetic of
// the lane tier; the wavefront around it is lane_device.h).
//
// Same rule as xd::extend, for match = 1, mismatch = -1, gap = -1.  A lane
// owns a window of Q = 32*W consecutive rows of the current antidiagonal, one
// bit per row in each 32-bit register: P registers ("planes") per 32 rows hold
// the cells' values, one the live rows, two the bases of a and two those of
// b.  A logical instruction therefore works on 32 rows of 64 extensions, and
// a step of one antidiagonal costs a lane about 57*W + 20 of them (P = 6).
//
// Values.  V = S + d + X mod 2^P (d = antidiagonal): a gap move keeps V, a
// diagonal one adds 3 on a match and 1 on a mismatch.  A cell is live when
// V >= thr = T_{d-1} + d (V(0, 0) = X); live cells lie in [thr, thr + X + 1],
// so P bits tell them apart while X + 2 <= 2^(P-1).  Dead cells keep
// whatever was computed: every choice below is masked with the live rows.
//
// Comparisons.  Two live neighbours A = (i, j-1) and B = (i-1, j) of a cell
// differ by at most 3, and with D = (i-1, j-1) live both lie in [D, D + 3],
// so three bits decide max(A, B) and two decide whether it is above D.
// Proof: let c be live on antidiagonal d, in row i >= 1, and u the cell above
// it; then either u is live with V(u) >= V(c) - 3, or V(c) <= thr_d + 1 (the
// cell to the left of c: likewise).  By induction along c's best path: from u,
// V(u) = V(c); from the diagonal cell w, V(w) >= V(c) - 3 reaches u by a gap
// move; from the left cell l, V(l) = V(c) and l's upper neighbour is w again,
// live with V(w) >= V(l) - 3 or V(l) <= thr_{d-1} + 1.  In each case u was
// offered V(c) - 3, so u is live at that value or V(c) - 3 < thr_{d-1} <=
// thr_d - 1.  Now A and B live: with D live each is at least D (a gap move
// from D) and at most D + 3, or at most thr_d + 1 <= thr_{d-1} + 3 <= D + 3;
// with D dead both lie in [thr_d, thr_d + 1].
//
// Window.  The rows' first index moves one up on every other step, so the
// band stays put while it follows the main diagonal.  Steps come in pairs:
//   "down"  (base + 1): left neighbour one bit up, upper neighbour same bit,
//           a's bits move down one, the next row's base enters at the top;
//   "right" (base):     left neighbour same bit, upper neighbour one bit
//           down, b's bits move up one, the next column's base enters below;
// and the diagonal neighbour, two antidiagonals back, is always the same bit.
// A third plane per sequence says which of its positions exist (rows <= m,
// columns <= n), which keeps cells outside the grid dead.
//
// Wider windows.  S neighbouring lanes (a power of two) may share an extension,
// lane s holding rows base + 32*W*s on; bits cross from lane to lane with one
// more instruction a plane.  Each lane keeps its own base, so everything above
// holds lane by lane.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define XD_HD __host__ __device__ __forceinline__
#else
#define XD_HD inline __attribute__((always_inline))
#endif

namespace xd {
namespace lane {

// ---- word operations ----------------------------------------------------------

// truth table masks of lut's operands: lut<f(kA, kB, kC) & 255>(a, b, c) = f(a, b, c)
constexpr int kA = 0xF0, kB = 0xCC, kC = 0xAA;

template <int T>
XD_HD uint32_t lut(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(a, b, c, T & 255);
#else
  uint32_t r = 0;
  for (int k = 0; k < 8; ++k)
    if ((T >> k) & 1) r |= ((k & 4) ? a : ~a) & ((k & 2) ? b : ~b) & ((k & 1) ? c : ~c);
  return r;
#endif
}
XD_HD uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return lut<kA ^ kB ^ kC>(a, b, c); }
XD_HD uint32_t or3(uint32_t a, uint32_t b, uint32_t c) { return lut<kA | kB | kC>(a, b, c); }
XD_HD uint32_t maj(uint32_t a, uint32_t b, uint32_t c) {
  return lut<(kA & kB) | (kA & kC) | (kB & kC)>(a, b, c);
}
// borrow out of a - b - c
XD_HD uint32_t borrow(uint32_t a, uint32_t b, uint32_t c) {
  return lut<(~kA & kB) | (~kA & kC) | (kB & kC)>(a, b, c);
}
// s ? a : b
XD_HD uint32_t sel(uint32_t s, uint32_t a, uint32_t b) {
  return lut<(kA & kB) | (~kA & kC)>(s, a, b);
}
// low word of {hi, lo} >> (sh & 31)
XD_HD uint32_t alignbit(uint32_t hi, uint32_t lo, uint32_t sh) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_alignbit(hi, lo, sh);
#else
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> (sh & 31));
#endif
}
XD_HD uint32_t reverse(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_bitreverse32(v);
#else
  uint32_t r = 0;
  for (int k = 0; k < 32; ++k) r |= ((v >> k) & 1u) << (31 - k);
  return r;
#endif
}
// all bits equal to bit p of v
template <int p>
XD_HD uint32_t spread(int32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return (uint32_t)__builtin_amdgcn_sbfe(v, p, 1);
#else
  return 0u - (((uint32_t)v >> p) & 1u);
#endif
}
// the n lowest bits set (n clamped to 0..32)
XD_HD uint32_t low_bits(int32_t n) {
  if (n >= 32) return ~0u;
  return (1u << (n < 0 ? 0 : n)) - 1u;
}
XD_HD int32_t lowest(uint32_t v) { return __builtin_ctz(v); }
XD_HD int32_t highest(uint32_t v) { return 31 - __builtin_clz(v); }

// ---- lanes that share an extension ------------------------------------------------

#if defined(__HIP_DEVICE_COMPILE__)
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, kCtrl, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t lane_above(uint32_t v) { return dpp<0x130>(v); }  // wave_shl:1
__device__ __forceinline__ uint32_t lane_below(uint32_t v) { return dpp<0x138>(v); }  // wave_shr:1
// nonzero in every lane of a group of S when any of them is
template <int S>
__device__ __forceinline__ uint32_t any_of(uint32_t v) {
  if constexpr (S >= 2) v |= dpp<0xB1>(v);   // quad_perm 1,0,3,2
  if constexpr (S >= 4) v |= dpp<0x4E>(v);   // quad_perm 2,3,0,1
  if constexpr (S >= 8) v |= dpp<0x141>(v);  // row_half_mirror
  if constexpr (S >= 16) v |= dpp<0x140>(v); // row_mirror
  if constexpr (S >= 32) {
    auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = r[0] | r[1];
  }
  return v;
}
#else
XD_HD uint32_t lane_above(uint32_t) { return 0; }
XD_HD uint32_t lane_below(uint32_t) { return 0; }
template <int S>
XD_HD uint32_t any_of(uint32_t v) { return v; }
template <int kCtrl>
XD_HD uint32_t dpp(uint32_t v) { return v; }
#endif

// ---- the planar read store ------------------------------------------------------

// A read's bases 32 at a time, two words each: bit t of the first (second) word
// is bit 0 (1) of base 32c + t's code.  kGuard chunks lie between reads (and
// before the first and after the last), so a window may start up to
// kMaxReach chunks before a read or end that far past it.
constexpr int kGuard = 8;
constexpr int kMaxReach = 5;  // chunks a window of up to 96 rows plus its feed reads

struct alignas(8) Chunk {
  uint32_t p0, p1;
};

// 32*N positions of a read, element t at position first + t (up) or first - t
// (!up): the chunks that hold them, and the two planes taken from these.
// Elements outside the read are arbitrary.
template <int N>
XD_HD void load_chunks(const Chunk* read, int32_t n_chunks, int32_t first, bool up,
                       Chunk (&w)[N + 1]) {
  static_assert(N + 1 <= kMaxReach, "guard chunks");
  int32_t c = (up ? first : first - (32 * N - 1)) >> 5;
  // a start clamped here has no element inside the read
  c = c < -kMaxReach ? -kMaxReach : c;
  c = c > n_chunks ? n_chunks : c;
#pragma unroll
  for (int k = 0; k <= N; ++k) w[k] = read[c + k];
}

template <int N>
XD_HD void take_planes(const Chunk (&w)[N + 1], int32_t first, bool up, uint32_t (&o0)[N],
                       uint32_t (&o1)[N]) {
  const uint32_t sh = (uint32_t)(up ? first : first - (32 * N - 1)) & 31u;
  uint32_t f0[N], f1[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    f0[k] = alignbit(w[k + 1].p0, w[k].p0, sh);
    f1[k] = alignbit(w[k + 1].p1, w[k].p1, sh);
  }
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const uint32_t r0 = reverse(f0[N - 1 - k]), r1 = reverse(f1[N - 1 - k]);
    o0[k] = up ? f0[k] : r0;
    o1[k] = up ? f1[k] : r1;
  }
}

template <int N>
XD_HD void gather(const Chunk* read, int32_t n_chunks, int32_t first, bool up,
                  uint32_t (&o0)[N], uint32_t (&o1)[N]) {
  Chunk w[N + 1];
  load_chunks<N>(read, n_chunks, first, up, w);
  take_planes<N>(w, first, up, o0, o1);
}

// State of an extension that outgrew its window: the last antidiagonal, the
// window's first row, threshold, arg-max and cells so far, then for each 32
// rows the planes and live rows of the last antidiagonal (U, L) and of the
// one before (D, LD).  Seven planes, whatever the tier's count.
constexpr int kStatePlanes = 7;
struct StateHead {
  int32_t d, base, thr, bi, dstar;
  uint32_t cells, words, cells_high;
};
struct StateWord {
  uint32_t U[kStatePlanes], D[kStatePlanes], L, LD;
};
constexpr uint32_t state_bytes(int words) {
  return (uint32_t)(sizeof(StateHead) + words * sizeof(StateWord));
}
static_assert(sizeof(StateHead) == 32 && sizeof(StateWord) == 64, "state layout");

// Evaluated cells: a lane counts its own in 32 bits (at most 96 rows of 2^23
// antidiagonals), an extension's need 33 in 1,024 rows.  A resumed extension's
// count is spread over its S lanes, lane s's part being count_part, and a group's
// is the sum of its lanes' halves (count_of).  256 and 512 rows need no more
// than 32 bits (kWholeCount: the first lane goes on from the count it resumed
// with); halves cost the lists of 256 rows 3 % and those of 512 rows 5 %, and
// nothing in the narrower ones.
template <int S>
constexpr bool kWholeCount = S == 8 || S == 16;
template <int S>
XD_HD uint32_t count_part(const StateHead& h, int s) {
  const uint64_t cells = (uint64_t)h.cells_high << 32 | h.cells;
  return (uint32_t)(cells / S) + (s == 0 ? (uint32_t)(cells % S) : 0u);
}
XD_HD uint64_t count_of(uint32_t low_sum, uint32_t high_sum) {
  return ((uint64_t)high_sum << 16) + low_sum;
}

// ---- one extension ---------------------------------------------------------------

// Inputs of an extension, in the planar store's terms.
struct Task {
  const Chunk *ra, *rb;  // chunk 0 of the reads
  int32_t ca, cb;        // their chunk counts
  int32_t oa, ob;        // position of a_1 in A, of b_1 in B
  int32_t m, n;
  int32_t X;
  uint32_t flags;        // kBackA, kBackB, kComp
};
constexpr uint32_t kBackA = 1, kBackB = 2, kComp = 4;  // A, B walked backwards; b complemented

// largest X that P planes tell apart
constexpr int32_t x_limit(int P) { return (1 << (P - 1)) - 2; }

// W: words of 32 rows a lane; S: lanes an extension (on the host, 1).
template <int P, int W, int S = 1>
struct Core {
  static constexpr int Q = 32 * W * S;   // window rows
  static constexpr int kLaneRows = 32 * W;
  static constexpr int kGroup = 4;       // steps between edge tests: the band grows by
                                         // kGroup / 2 rows at either end
  static constexpr int kMaxSteps = 64;   // steps between refills of the base windows
  static constexpr uint32_t kLowEdge = 0x3u, kHighEdge = 0xC0000000u;
  // highest minus lowest live row that can be centred clear of both edges
  static constexpr int kMaxSpan = Q - 6;

  uint32_t U[P][W];   // values on the last antidiagonal d
  uint32_t D[P][W];   // and on the one before
  uint32_t L[W], LD[W];          // their live rows
  uint32_t a0[W], a1[W], va[W];  // a's bases and which rows exist
  uint32_t b0[W], b1[W], vb[W];  // b's, by row of the current antidiagonal
  uint32_t fa0, fa1, fva, fb0, fb1, fvb;  // what enters next (a: bit 0 first, b: bit 31)
  int32_t thr;        // threshold of antidiagonal d + 1: T_d + d + 1
  int32_t top;        // X + 1
  uint32_t cnt;       // evaluated cells
  uint32_t bm[W];     // improving rows of the last improving step since the refill
  int32_t bk;         // that step
  uint32_t inner_top, inner_low;  // all ones except in the group's last / first lane (S > 1)

  // the word that borders the lane's last / first one, 0 at the window's ends
  XD_HD uint32_t above(uint32_t first) const {
    return S > 1 ? lane_above(first) & inner_top : 0u;
  }
  XD_HD uint32_t below(uint32_t last) const {
    return S > 1 ? lane_below(last) & inner_low : 0u;
  }
  // the same for the base windows, fed at the window's ends
  XD_HD uint32_t above(uint32_t first, uint32_t feed) const {
    return S > 1 ? sel(inner_top, lane_above(first), feed) : feed;
  }
  XD_HD uint32_t below(uint32_t last, uint32_t feed) const {
    return S > 1 ? sel(inner_low, lane_below(last), feed) : feed;
  }

  // s: this lane's place in its group
  XD_HD void clear(int s) {
    inner_top = s == S - 1 ? 0u : ~0u;
    inner_low = s == 0 ? 0u : ~0u;
#pragma unroll
    for (int w = 0; w < W; ++w) {
#pragma unroll
      for (int p = 0; p < P; ++p) U[p][w] = D[p][w] = 0;
      L[w] = LD[w] = bm[w] = 0;
      a0[w] = a1[w] = va[w] = b0[w] = b1[w] = vb[w] = 0;
    }
    fa0 = fa1 = fva = fb0 = fb1 = fvb = 0;
    thr = 1;
    top = 1;
    cnt = 0;
    bk = 0;
  }

  // the origin alone is live, in the middle of the window (base = -Q / 2);
  // s: this lane's place in its group
  XD_HD void start(int32_t X, int s) {
    constexpr int w0 = S > 1 ? 0 : Q / 2 / 32;
    const uint32_t bit = S > 1 ? (s == S / 2 ? 1u : 0u) : 1u << (Q / 2 % 32);
#pragma unroll
    for (int w = 0; w < W; ++w) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        U[p][w] = w == w0 && ((X >> p) & 1) ? bit : 0u;
        D[p][w] = 0;
      }
      L[w] = w == w0 ? bit : 0u;
      LD[w] = bm[w] = 0;
    }
    thr = 1;
    top = X + 1;
    cnt = 0;
  }

  // plane p: bit p of v in every row
  template <int p = 0>
  static XD_HD void planes(uint32_t (&o)[P], int32_t v) {
    o[p] = spread<p>(v);
    if constexpr (p + 1 < P) planes<p + 1>(o, v);
  }

  // antidiagonal d + 1; k: steps since the refill (even: down, odd: right)
  template <bool DOWN>
  XD_HD void step(int32_t k) {
    if (DOWN) {
      const uint32_t e0 = above(a0[0], fa0), e1 = above(a1[0], fa1), ev = above(va[0], fva);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        a0[w] = alignbit(w + 1 < W ? a0[w + 1] : e0, a0[w], 1);
        a1[w] = alignbit(w + 1 < W ? a1[w + 1] : e1, a1[w], 1);
        va[w] = alignbit(w + 1 < W ? va[w + 1] : ev, va[w], 1);
      }
      fa0 >>= 1;
      fa1 >>= 1;
      fva >>= 1;
    } else {
      const uint32_t e0 = below(b0[W - 1], fb0), e1 = below(b1[W - 1], fb1),
                     ev = below(vb[W - 1], fvb);
#pragma unroll
      for (int w = W - 1; w >= 0; --w) {
        b0[w] = alignbit(b0[w], w > 0 ? b0[w - 1] : e0, 31);
        b1[w] = alignbit(b1[w], w > 0 ? b1[w - 1] : e1, 31);
        vb[w] = alignbit(vb[w], w > 0 ? vb[w - 1] : ev, 31);
      }
      fb0 <<= 1;
      fb1 <<= 1;
      fvb <<= 1;
    }
    // planes of the threshold and of the score that improves on T
    uint32_t t[P], i[P];
    planes(t, thr);
    planes(i, thr + top);
    uint32_t any = 0;
    uint32_t NU[P][W], NL[W], NI[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      // the gap neighbour that is a bit away; at the window's end it is dead,
      // whatever its value planes take from the next group of lanes
      uint32_t N[P];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const uint32_t* x = U[p];
        N[p] = DOWN ? alignbit(w + 1 < W ? x[w + 1] : S > 1 ? lane_above(x[0]) : 0u, x[w], 1)
                    : alignbit(x[w], w > 0 ? x[w - 1] : S > 1 ? lane_below(x[W - 1]) : 0u, 31);
      }
      const uint32_t LN = DOWN ? alignbit(w + 1 < W ? L[w + 1] : above(L[0]), L[w], 1)
                               : alignbit(L[w], w > 0 ? L[w - 1] : below(L[W - 1]), 31);
      const uint32_t LU = L[w], LX = LD[w];
      // M: the larger gap neighbour (three bits decide)
      uint32_t bw = ~U[0][w] & N[0];
      bw = borrow(U[1][w], N[1], bw);
      const uint32_t less = xor3(U[2][w], N[2], bw);
      const uint32_t useN = lut<kA & (~kB | kC)>(LN, LU, less);
      uint32_t M[P];
#pragma unroll
      for (int p = 0; p < P; ++p) M[p] = sel(useN, N[p], U[p][w]);
      // the diagonal move wins on a match, and otherwise unless a live gap
      // neighbour is above D (two bits decide)
      const uint32_t ne = lut<kA | (kB ^ kC)>(M[0] ^ D[0][w], M[1], D[1][w]);
      const uint32_t above = lut<kA & (kB | kC)>(ne, LU, LN);
      const uint32_t eq = lut<~(kA | (kB ^ kC)) & 255>(a0[w] ^ b0[w], a1[w], b1[w]);
      const uint32_t useD = lut<kA & (kB | ~kC)>(LX, eq, above);
      // D + 1 + 2 eq, chosen plane by plane
      uint32_t V[P];
      V[0] = lut<(kA & ~kB) | (~kA & kC)>(useD, D[0][w], M[0]);
      V[1] = sel(useD, xor3(D[1][w], eq, D[0][w]), M[1]);
      uint32_t cy = maj(D[1][w], eq, D[0][w]);
#pragma unroll
      for (int p = 2; p < P; ++p) {
        V[p] = sel(useD, D[p][w] ^ cy, M[p]);
        cy &= D[p][w];
      }
      // evaluated and live cells
      uint32_t ev = or3(LU, LN, LX);
      ev = lut<kA & kB & kC>(ev, va[w], vb[w]);
      bw = ~V[0] & t[0];
#pragma unroll
      for (int p = 1; p < P - 1; ++p) bw = borrow(V[p], t[p], bw);
      // live: V - thr >= 0 as a P-bit signed number
      const uint32_t dead = xor3(V[P - 1], t[P - 1], bw);
      const uint32_t nl = ev & ~dead;
      // improving: V = thr + X + 1 (P - 1 bits decide among live cells)
      uint32_t diff = V[0] ^ i[0];
#pragma unroll
      for (int p = 1; p < P - 1; ++p) diff = lut<kA | (kB ^ kC)>(diff, V[p], i[p]);
      const uint32_t imp = nl & ~diff;
      any |= imp;
#pragma unroll
      for (int p = 0; p < P; ++p) NU[p][w] = V[p];
      NL[w] = nl;
      NI[w] = imp;
      cnt += (uint32_t)__builtin_popcount(ev);
    }
    const bool up = any_of<S>(any) != 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        D[p][w] = U[p][w];
        U[p][w] = NU[p][w];
      }
      LD[w] = L[w];
      L[w] = NL[w];
      bm[w] = up ? NI[w] : bm[w];
    }
    bk = up ? k : bk;
    thr += up ? 2 : 1;
  }

  // kGroup steps from step k of the refill period (k even)
  XD_HD void group(int32_t k) {
    step<true>(k);
    step<false>(k + 1);
    step<true>(k + 2);
    step<false>(k + 3);
  }

  // nonzero: the band reached the margin the next group needs (in one lane)
  XD_HD uint32_t edge() const {
    if (S > 1)
      return ((L[0] | LD[0]) & kLowEdge & ~inner_low) |
             ((L[W - 1] | LD[W - 1]) & kHighEdge & ~inner_top);
    if (W == 1) return (L[0] | LD[0]) & (kLowEdge | kHighEdge);
    return ((L[0] | LD[0]) & kLowEdge) | ((L[W - 1] | LD[W - 1]) & kHighEdge);
  }

  // this lane's lowest and highest live bit of the last two antidiagonals;
  // false: none (lo is then large and hi negative)
  XD_HD bool extent(int32_t& lo, int32_t& hi) const {
    lo = 1 << 20;
    hi = -1;
#pragma unroll
    for (int w = W - 1; w >= 0; --w) {
      const uint32_t m = L[w] | LD[w];
      lo = m ? 32 * w + lowest(m) : lo;
      hi = m && hi < 0 ? 32 * w + highest(m) : hi;
    }
    return hi >= 0;
  }

  // moves the window up by s rows (|s| <= 31; bits that leave are dead)
  XD_HD void slide(int32_t s) {
    const bool neg = s < 0;
    const uint32_t sh = (uint32_t)s & 31u;
    auto mv = [&](uint32_t (&x)[W]) {
      const uint32_t first = below(x[W - 1]), last = above(x[0]);
      uint32_t y[W + 1];
#pragma unroll
      for (int w = 0; w <= W; ++w) {
        const uint32_t under = w > 0 ? x[w - 1] : first, at = w < W ? x[w] : last;
        y[w] = neg ? under : at;
      }
#pragma unroll
      for (int w = 0; w < W; ++w) x[w] = alignbit(y[w + 1], y[w], sh);
    };
#pragma unroll
    for (int p = 0; p < P; ++p) {
      mv(U[p]);
      mv(D[p]);
    }
    mv(L);
    mv(LD);
  }

  // The bases a window needs after antidiagonal d, when the lane's rows start
  // at base: 32 * (W + 1) of each sequence, a's element q being row base + q
  // and b's column d - base + 32 - q.
  struct Bases {
    uint32_t a0[W + 1], a1[W + 1], b0[W + 1], b1[W + 1];
  };
  static XD_HD int32_t a_first(const Task& t, int32_t row) {
    return (t.flags & kBackA) ? t.oa - (row - 1) : t.oa + (row - 1);
  }
  static XD_HD int32_t b_first(const Task& t, int32_t column) {
    return (t.flags & kBackB) ? t.ob - (column - 1) : t.ob + (column - 1);
  }
  static XD_HD void bases(const Task& t, int32_t d, int32_t base, Bases& x) {
    gather<W + 1>(t.ra, t.ca, a_first(t, base), !(t.flags & kBackA), x.a0, x.a1);
    gather<W + 1>(t.rb, t.cb, b_first(t, d - base + 32), (t.flags & kBackB) != 0, x.b0, x.b1);
    const uint32_t cm = (t.flags & kComp) ? ~0u : 0u;
#pragma unroll
    for (int w = 0; w <= W; ++w) {
      x.b0[w] ^= cm;
      x.b1[w] ^= cm;
    }
  }

  // fills the base windows and feeds from them
  XD_HD void refill(const Task& t, int32_t d, int32_t base, const Bases& x) {
    const int32_t na = t.m - base + 1;        // elements of a that exist
    const int32_t nb = d - base + 32 - t.n;   // elements of b that do not
#pragma unroll
    for (int w = 0; w < W; ++w) {
      a0[w] = x.a0[w];
      a1[w] = x.a1[w];
      va[w] = low_bits(na - 32 * w);
      b0[w] = x.b0[w + 1];
      b1[w] = x.b1[w + 1];
      vb[w] = ~low_bits(nb - 32 * (w + 1));
    }
    fa0 = x.a0[W];
    fa1 = x.a1[W];
    fva = low_bits(na - 32 * W);
    fb0 = x.b0[0];
    fb1 = x.b1[0];
    fvb = ~low_bits(nb);
  }

  // The feeds alone, when the windows have moved kMaxSteps steps since the
  // last refill and nowhere else: the chunks they come from, which may be
  // read one period ahead, and the feeds.
  struct Ahead {
    Chunk a[2], b[2];
  };
  static XD_HD void look_ahead(const Task& t, int32_t d, int32_t base, Ahead& x) {
    load_chunks<1>(t.ra, t.ca, a_first(t, base + kLaneRows), !(t.flags & kBackA), x.a);
    load_chunks<1>(t.rb, t.cb, b_first(t, d - base + 32), (t.flags & kBackB) != 0, x.b);
  }
  XD_HD void feed(const Task& t, int32_t d, int32_t base, const Ahead& x) {
    uint32_t x0[1], x1[1], y0[1], y1[1];
    take_planes<1>(x.a, a_first(t, base + kLaneRows), !(t.flags & kBackA), x0, x1);
    take_planes<1>(x.b, b_first(t, d - base + 32), (t.flags & kBackB) != 0, y0, y1);
    const uint32_t cm = (t.flags & kComp) ? ~0u : 0u;
    fa0 = x0[0];
    fa1 = x1[0];
    fva = low_bits(t.m - base - kLaneRows + 1);
    fb0 = y0[0] ^ cm;
    fb1 = y1[0] ^ cm;
    fvb = ~low_bits(d - base + 32 - t.n);
  }

  // this lane's lowest improving row of the last improving step since the
  // refill (step bk), which found the lane's rows at base; none: a large number
  XD_HD int32_t settle(int32_t base) {
    int32_t q = 1 << 30;
#pragma unroll
    for (int w = W - 1; w >= 0; --w)
      q = bm[w] ? base + (bk >> 1) + 1 + 32 * w + lowest(bm[w]) : q;
#pragma unroll
    for (int w = 0; w < W; ++w) bm[w] = 0;
    return q;
  }

  // Planes P and up of the values x[.][w]: a live value is thr plus the signed
  // P-bit difference to it, so it lies in thr's block of 2^P, in the next one
  // (plus) or in the one before (minus).
  XD_HD void save_planes(const uint32_t (&x)[P][W], int w, uint32_t (&o)[kStatePlanes]) const {
    uint32_t t[P];
    planes(t, thr);
    uint32_t bw = ~x[0][w] & t[0];
#pragma unroll
    for (int p = 1; p < P - 1; ++p) bw = borrow(x[p][w], t[p], bw);
    const uint32_t neg = xor3(x[P - 1][w], t[P - 1], bw);      // V - thr < 0
    const uint32_t lower = borrow(x[P - 1][w], t[P - 1], bw);  // V's low bits below thr's
    uint32_t plus = lower & ~neg, minus = neg & ~lower;
#pragma unroll
    for (int p = 0; p < kStatePlanes; ++p) {
      if (p < P) {
        o[p] = x[p < P ? p : 0][w];
        continue;
      }
      const uint32_t b = 0u - (((uint32_t)thr >> p) & 1u);
      o[p] = b ^ (plus | minus);
      plus &= b;
      minus &= ~b;
    }
  }

  // this lane's words (s: its place in the group) of the state at dst
  XD_HD void save_words(int s, uint8_t* dst) const {
    StateWord* out = (StateWord*)(dst + sizeof(StateHead)) + s * W;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      StateWord x;
      save_planes(U, w, x.U);
      save_planes(D, w, x.D);
      x.L = L[w];
      x.LD = LD[w];
      out[w] = x;
    }
  }

  // this lane's rows from a state of `words` words; rows above them are dead
  XD_HD void load_words(int s, int32_t words, const uint8_t* src) {
    static_assert(P <= kStatePlanes, "planes kept");
    const StateWord* in = (const StateWord*)(src + sizeof(StateHead));
#pragma unroll
    for (int w = 0; w < W; ++w) {
      StateWord x = {};
      if (s * W + w < words) x = in[s * W + w];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        U[p][w] = x.U[p];
        D[p][w] = x.D[p];
      }
      L[w] = x.L;
      LD[w] = x.LD;
      bm[w] = 0;
    }
  }
};

}  // namespace lane
}  // namespace xd
