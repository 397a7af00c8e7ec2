// Banded Smith-Waterman, two tasks to a wavefront: one in the low, one in the
// high 16 bits of every lane's value.
//
// A band of half-width w holds at most w + 1 <= 49 rows of an antidiagonal, so
// one task fills the lanes of a wavefront and what bounds the one-task kernel
// is vector issue: 10 to 11 instructions an antidiagonal.  Here an antidiagonal
// of both tasks takes 8: rotate a row, max, add the gap, add the substitution
// (one to join the two tasks' looked-up bytes), max, the band's edge, and the
// running maximum.
//
// Values are H - 32768 in 16 signed bits.  Adding a negative score with
// saturation is then the floor at H = 0, exactly, as long as no H exceeds
// 65,535; tasks that could are left to the one-task code.
//
// Cells outside the grid need no masks.  A row or column outside it never
// matches, so values there come from in-grid cells by mismatches and gaps only,
// which are all negative: they stay below the best, and no path leads back.
// Cells outside the band are cut off by a minimum with -32768, one register a
// step: a group of 16 antidiagonals starts where d + c - w is even and moves the
// window up 8 rows, so the masks of every group are the same.
//
// Positions are not followed.  Every 128 antidiagonals (a block) the two running
// maxima are reduced; when one has passed its task's best, the state in which
// the block began is kept.  The task's end cell lies in the last such block,
// which the one-task code runs again with the best known, at most 128
// antidiagonals of some 20,000.
//
// 50,000 pairs of 10 kbp reads at w = 32: 11.6 -> 6.3 ms against one task to a
// wavefront.
#pragma once

#include "xdrop_device.h"

namespace xd {

typedef int16_t pk16 __attribute__((ext_vector_type(2)));

namespace pair_band {

constexpr int GS = 16;        // antidiagonals a group
constexpr int kGroups = 8;    // groups a block
constexpr int kStep = GS * kGroups;
constexpr int kRows = kStep / 2;  // rows (and columns) a block advances
constexpr int RING = 256, MIR = GS + 1, RA = 128;
constexpr int kHalf = RING + MIR + RA / 4;  // words of one task's rings
constexpr int kNone = 2 * kHalf;            // words that no code matches in
constexpr int kLdsWords = 2 * kHalf + MIR;

constexpr int32_t kMaxH = 65535;

// one task as the wavefront runs it (uniform)
struct Half {
  const uint32_t* wa;
  const uint32_t* wb;
  int32_t la, lb, c, w;
  int32_t d0, base0;      // first antidiagonal (d0 + c - w even), its window
  int32_t aorg, borg;     // ring index 0 is row aorg, column borg
  int32_t first, end;     // blocks it runs: [first, end)
  int32_t best;           // so far, and the block that reached it
  int32_t at;
  int32_t task;           // -1: none
};

__device__ __forceinline__ pk16 splat(int32_t v) { return (pk16){(int16_t)v, (int16_t)v}; }
__device__ __forceinline__ uint32_t bits(pk16 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ pk16 from_bits(uint32_t v) { return __builtin_bit_cast(pk16, v); }

// lane l takes lane l - 1's value, lane 0 lane 63's (never a band row)
__device__ __forceinline__ pk16 rot1(pk16 v) {
  return from_bits((uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)bits(v), 0x13C /* wave_ror:1 */,
                                                         0xF, 0xF, true));
}

}  // namespace pair_band

// Runs the tasks `next(h)` hands out, at most one in each half at a time, and
// gives each one's result to `done(task, out)`.  next fills a Half's reads and
// band (task < 0: nothing left).  lds holds pair_band::kLdsWords words, ring
// what banded_sw takes.
template <bool UNIT, class Next, class Done>
__device__ __forceinline__ void banded_pairs(const Scoring& sc, uint32_t* __restrict__ lds,
                                             uint32_t* __restrict__ ring, Next&& next,
                                             Done&& done) {
  using namespace pair_band;
  const int lane = lane_id();
  const pk16 kFloor = splat(-32768);
  const uint32_t none = 0x01010101u * (uint32_t)(uint8_t)sc.MM;
  const uint32_t swap = (uint32_t)(uint8_t)(sc.M ^ sc.MM);
  const pk16 gap = splat(sc.G);
  if (lane < MIR) lds[kNone + lane] = none;

  Half H[2];
  pk16 cap[GS];  // 32767 in the band, -32768 outside
#pragma unroll
  for (int t = 0; t < GS; ++t) cap[t] = kFloor;
  pk16 U1 = kFloor, Up = kFloor;  // last antidiagonal; the one before, rows up by one
  pk16 S1 = kFloor, Sp = kFloor;  // the same where each task's best block began
  uint32_t pfa[2] = {0, 0}, pfb[2] = {0, 0};
  int32_t blk = 0;  // blocks run so far; ring indices go up by 64 with each

  auto word_of = [&](const uint32_t* wd, int32_t q, int32_t lim) -> uint32_t {
    uint32_t v = 0;
    if (q >= 1 & q <= lim) v = wd[(q - 1) >> 4];
    return v;
  };
  auto put_b = [&](const Half& e, int h, int32_t x0, uint32_t wd) {  // columns x0..x0+63
    const int32_t j = e.borg + x0 + lane;
    uint32_t v = none;
    if (j >= 1 & j <= e.lb) v ^= swap << (8u * ((wd >> (((j - 1) & 15) << 1)) & 3u));
    const int slot = (x0 + lane) & (RING - 1);
    lds[h * kHalf + slot] = v;
    if (slot < MIR) lds[h * kHalf + RING + slot] = v;
  };
  auto put_a = [&](const Half& e, int h, int32_t y0, uint32_t wd) {  // rows y0..y0+63
    const int32_t i = e.aorg + y0 + lane;
    const uint32_t v = (i >= 1 & i <= e.la) ? (wd >> (((i - 1) & 15) << 1)) & 3u : 4u;
    ((uint8_t*)(lds + h * kHalf + RING + MIR))[(y0 + lane) & (RA - 1)] = (uint8_t)v;
  };
  // half h's part of a packed value
  auto put_half = [](pk16 to, pk16 from, int h) {
    return h ? (pk16){to.x, from.y} : (pk16){from.x, to.y};
  };
  auto start = [&](auto h_tag) {
    constexpr int h = decltype(h_tag)::value;
    Half& e = H[h];
    next(e);
    U1 = put_half(U1, kFloor, h);
    Up = put_half(Up, kFloor, h);
    S1 = put_half(S1, kFloor, h);
    Sp = put_half(Sp, kFloor, h);
    e.best = 0;
    e.at = e.first = e.end = blk;
    if (e.task < 0) {
#pragma unroll
      for (int t = 0; t < GS; ++t) cap[t] = put_half(cap[t], kFloor, h);
      return;
    }
    const BandSpan sp = band_span(e.la, e.lb, e.c, e.w);
    e.d0 = sp.d_first - ((sp.d_first + e.c - e.w) & 1);
    e.base0 = ((e.d0 + e.c - e.w) >> 1) - 1;
    e.end = blk + (sp.d_last - e.d0) / kStep + 1;
    // row base0 + lane at y = 64 blk + lane; column d0 - base0 - lane at x = 64 (blk + 1) - lane
    e.aorg = e.base0 - kRows * blk;
    e.borg = e.d0 - e.base0 - kRows * (blk + 1);
#pragma unroll
    for (int t = 0; t < GS; ++t) {
      const int lo = 1 + (t + 1) / 2, n = e.w + 1 - (t & 1);
      const pk16 in = splat((lane >= lo & lane < lo + n) ? 32767 : -32768);
      cap[t] = put_half(cap[t], in, h);
    }
    put_a(e, h, kRows * blk, word_of(e.wa, e.aorg + kRows * blk + lane, e.la));
    for (int q = 0; q < 2; ++q)
      put_b(e, h, kRows * (blk + q), word_of(e.wb, e.borg + kRows * (blk + q) + lane, e.lb));
    pfa[h] = word_of(e.wa, e.aorg + kRows * (blk + 1) + lane, e.la);
    pfb[h] = word_of(e.wb, e.borg + kRows * (blk + 2) + lane, e.lb);
  };
  auto finish = [&](auto h_tag) {
    constexpr int h = decltype(h_tag)::value;
    Half& e = H[h];
    const int32_t g = -sc.G;
    BandStart s;
    s.d = e.d0 + kStep * (e.at - e.first);
    s.base = e.base0 + kRows * (e.at - e.first);
    s.d_stop = s.d + kStep - 1;
    s.U1 = (int32_t)(h ? S1.y : S1.x) + 32768 + g * (s.d - 1) + kBias0;
    s.Up = (int32_t)(h ? Sp.y : Sp.x) + 32768 + g * (s.d - 2) + kBias0;
    s.T = max(e.best - 1, 0);
    BandTask bt{e.wa, e.wb, e.la, e.lb, e.c, e.w};
    ExtOut o;
    banded_sw<UNIT, kNoTrace, true>(bt, sc, ring, o, BandTrace{nullptr}, s);
    done(e.task, o);
  };
  using zero = std::integral_constant<int, 0>;
  using one = std::integral_constant<int, 1>;
  H[0].task = H[1].task = 0;
  H[0].end = H[1].end = 0;
  bool fresh = true;
  while (true) {
    // tasks that ended with the last block (or none yet) make room for new ones
    if (H[0].task >= 0 && H[0].end == blk) {
      if (!fresh) finish(zero{});
      start(zero{});
    }
    if (H[1].task >= 0 && H[1].end == blk) {
      if (!fresh) finish(one{});
      start(one{});
    }
    fresh = false;
    if (H[0].task < 0 && H[1].task < 0) break;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (H[h].task < 0) continue;
      put_a(H[h], h, kRows * (blk + 1), pfa[h]);
      put_b(H[h], h, kRows * (blk + 2), pfb[h]);
      pfa[h] = word_of(H[h].wa, H[h].aorg + kRows * (blk + 2) + lane, H[h].la);
      pfb[h] = word_of(H[h].wb, H[h].borg + kRows * (blk + 3) + lane, H[h].lb);
    }
    wave_lds_fence();
    const pk16 B1 = U1, Bp = Up;
    pk16 run = kFloor;
    const int8_t* lb8 = (const int8_t*)lds;
#pragma unroll 1
    for (int k = 0; k < kGroups; ++k) {
      const int32_t y = (kRows * blk + 8 * k + lane) & (RA - 1);
      const int32_t x = (kRows * (blk + 1) + 8 * k - lane) & (RING - 1);
      uint32_t ad[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t code = ((const uint8_t*)(lds + h * kHalf + RING + MIR))[y];
        ad[h] = code < 4u ? (uint32_t)(h * kHalf + x) * 4u + code : (uint32_t)kNone * 4u;
      }
      pk16 sub[GS];
#pragma unroll
      for (int t = 0; t < GS; ++t)
        sub[t] = (pk16){(int16_t)lb8[ad[0] + 4 * t], (int16_t)lb8[ad[1] + 4 * t]};
#pragma unroll
      for (int t = 0; t < GS; ++t) {
        const pk16 up = rot1(U1);
        pk16 s = __builtin_elementwise_add_sat(__builtin_elementwise_max(up, U1), gap);
        s = __builtin_elementwise_max(s, __builtin_elementwise_add_sat(Up, sub[t]));
        U1 = __builtin_elementwise_min(s, cap[t]);
        run = __builtin_elementwise_max(run, U1);
        Up = up;
      }
      // the window moves up 8 rows (the lanes that wrap hold rows below the band)
      const int src = ((lane + 8) & 63) << 2;
      U1 = from_bits((uint32_t)__builtin_amdgcn_ds_bpermute(src, (int32_t)bits(U1)));
      Up = from_bits((uint32_t)__builtin_amdgcn_ds_bpermute(src, (int32_t)bits(Up)));
    }
    wave_lds_fence();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int32_t m = wave_max_i32((int32_t)(h ? run.y : run.x) + 32768);
      if (m > H[h].best) {
        H[h].best = m;
        H[h].at = blk;
        S1 = put_half(S1, B1, h);
        Sp = put_half(Sp, Bp, h);
      }
    }
    ++blk;
  }
}

}  // namespace xd
