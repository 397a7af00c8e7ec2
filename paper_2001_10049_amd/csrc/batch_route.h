// Which kernels a batch of extensions runs in (host code, no HIP).
#pragma once

#include <stdint.h>

namespace xd {

// what the host knows of a batch
struct BatchShape {
  bool batched;         // the caller asked for the device queue
  bool pair_ok;         // scores of the packed two-extension tiers (match = 1)
  bool lane_ok;         // scores 1/-1/-1, and the store has bit planes
  bool x_known;         // one X for all tasks,
  int32_t x;            // this one
  uint64_t n_ext;       // two a task
  uint32_t mean_len;    // of the store's reads
  int32_t tier1, tier2; // X limits of the 64- and the 128-cell first window
  uint32_t cus;
};

struct Route {
  bool queue;            // the device queue (batched form)
  bool packed;           // two extensions per wavefront in the 64-, 128- and 256-cell windows
  bool solo;             // match = 1, too few extensions for that: one per wavefront
  uint32_t lane_blocks;  // workgroups of single and split lanes (0: no lane tiers)
  uint32_t solo_blocks;  // more for the longest (with 96 rows, lane_blocks less)
  int32_t tier1, tier2;  // X limits of the queue's first windows
};

// Extensions from which the lane tiers run: they hold 65,536 at once, and a
// batch of half as many leaves most of them to wavefronts of their own.  Read
// pairs, ms one per wavefront / packed / in lanes: 12,500 at X = 25 2.4 / 2.9 / 2.6
// (10 kbp), 0.76 / 0.79 / 0.72 (1.3 kbp), 16,000 3.0 / 3.2 / 2.9, 32,000 5.5 / 4.8
// / 3.8; at X = 50 12,500 4.7 / 4.4 / 3.7.
constexpr uint64_t kLaneMin = 24576;
// X up to 14 gains later in long reads, because the narrow windows' lanes run in a
// launch after its longest: 20,000 pairs of 10 kbp at X = 7 3.5 / 3.3 / 3.6, 24,000
// 4.0 / 3.7 / 3.8, 32,000 5.3 / 4.7 / 4.0.
constexpr uint64_t kNarrowMin = 49152;
constexpr int32_t kNarrowX = 14;
// Extensions up to which the lane tiers get a workgroup more per CU for those that
// run one per wavefront: such a batch may run whole so, and the single lanes'
// workgroups leave at once (12,500 pairs of 10 kbp at X = 25 2.99 -> 2.61 ms).
constexpr uint64_t kLaneFill = 65536;
// Extensions up to which the batched form runs one per wavefront: their time
// is the longest one's chain of steps, about 40 ns a step with a wavefront to
// itself and 90 ns in a packed one.  64 pairs at X of 7 and 25: 1.59 -> 1.15 ms
// as a plan.  The packed kernels catch up at 18,000 to 20,000 pairs when all start
// in 64 cells (one per wavefront / packed, X = 25: 16,000 of 10 kbp 3.0 / 3.2, 20,000
// 3.6 / 3.4, of 3.5 kbp 1.38 / 1.42, 1.68 / 1.63), sooner when they start wider (X =
// 50: 12,000 of 10 kbp 4.5 / 4.9, 16,000 5.7 / 5.3, 6,000 of 3.5 kbp 1.18 / 1.26,
// 9,000 1.62 / 1.43); when the host does not know X, at the lane tiers' line.
constexpr uint64_t kSoloMax = kLaneMin - 1, kSoloMaxKnown = 36000, kSoloMaxWide = 15000;

// Whether a plain batch goes through the device queue all the same.  One
// wavefront per extension in task order has two launches and no sort before it;
// the queue runs the longest first, and packed or in lanes.  Times in ms, read
// pairs, without / with the queue:
//   reads of 2,500 bases and more on average, from 6,000 extensions on: X = 25,
//   3.5 kbp, 3,000 pairs 0.62 / 0.53, 10 kbp, 6,000 pairs 2.6 / 2.2; shorter ones
//   have no tail worth it (1.3 kbp, 6,000 pairs 0.40 / 0.45, 12,000 0.63 / 0.75),
//   but from 32,768 on the lane tiers gain (16,000 pairs 0.76 / 0.73, 32,000 1.34
//   / 0.75);
//   fewer extensions when X needs a wider first window than 64 cells, which is
//   else run and given up.  How many outgrow it depends on X: at 1.2 times the limit
//   few (X = 34, 10 kbp, 1,000 pairs 1.9 / 3.1), at 1.5 most, late (X = 52 5.4 /
//   3.2), past twice all, early, so that giving up costs little (X = 80, 1,000
//   pairs 3.2 / 3.2, 2,900 4.0 / 3.2).  Past the 128-cell limit the queue starts in
//   256 cells, the other form works up to them (X = 81, 1,000 pairs 3.2 / 7.7, X
//   = 100 4.9 / 7.7, 4,500 7.7 / 8.2, X = 130 8.1 / 7.7).
inline bool plain_queue(const BatchShape& b) {
  if (b.n_ext >= 6000 && b.mean_len >= 2500) return true;
  if (b.lane_ok && b.n_ext >= 32768) return true;
  if (!b.x_known) return false;
  const int64_t x = b.x, t1 = b.tier1, t2 = b.tier2;
  if (5 * x <= 6 * t1) return false;
  if (10 * x <= 21 * t1) return true;
  if (x <= t2) return b.n_ext >= 2000;
  if (5 * x <= 7 * t2) return b.n_ext >= 6000;
  return true;
}

inline Route batch_route(const BatchShape& b) {
  Route r = {b.batched || plain_queue(b), false, false, 0u, 0u, b.tier1, b.tier2};
  if (!r.queue) return r;
  // a plain batch starts narrower up to 1.2 times the limits, as it would without
  // the queue (X = 34, 10 kbp, 4,500 pairs: 2.4 in 64 cells, 3.3 in 128)
  if (!b.batched) {
    r.tier1 = (int32_t)(6ll * b.tier1 / 5);
    r.tier2 = (int32_t)(6ll * b.tier2 / 5);
  }
  const bool longer = b.mean_len >= 5000;
  const bool narrow = longer && b.x_known && b.x <= kNarrowX;
  if (b.lane_ok && b.n_ext >= (narrow ? kNarrowMin : kLaneMin)) {
    r.lane_blocks = b.cus;
    r.solo_blocks = (b.n_ext < kLaneFill ? 4 : 3) * b.cus;
  }
  if (b.pair_ok) {
    const uint64_t solo_max = !b.x_known ? kSoloMax
                              : b.x <= r.tier1 ? kSoloMaxKnown : longer ? kSoloMax : kSoloMaxWide;
    r.solo = !r.lane_blocks && b.n_ext <= solo_max;
    r.packed = !r.solo;
  }
  return r;
}

}  // namespace xd
