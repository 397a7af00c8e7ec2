// The batched form's queue layout (lane_share.h) on the CPU: the segments of n
// extensions with the given X and estimated antidiagonal counts (X < 0: of an
// invalid task).
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "lane_share.h"

using namespace xd::queue;

extern "C" void queue_segments(const int32_t* X, const uint32_t* cost, uint32_t n, int32_t x_tier1,
                               int32_t x_tier2, int32_t by_cost, uint32_t cus, uint32_t* seg) {
  const BinRule R = {x_tier1, x_tier2, by_cost, cus};
  std::vector<uint32_t> h(kBins, 0);
  for (uint32_t e = 0; e < n; ++e) ++h[X[e] < 0 ? kBins - 1 : bin_key(R, X[e], cost[e])];
  Shares S;
  std::vector<ClassBins> x(kKinds);
  for (int k = 0; k < kKinds && cus; ++k) {
    class_bins(h.data(), k, x[k]);
    if (!x[k].before[kCostBins]) continue;
    uint64_t best = ~0ull;
    for (uint32_t q = 0; q < kCandidates; ++q) best = std::min(best, share_rank(x[k], k, q, cus));
    S.choose(x[k], k, best, cus);
  }
  const bool merged = S.merged();
  std::vector<uint32_t> sum(kBins + 1, 0), slot(kBins, 0);
  for (uint32_t b = 0; b < (uint32_t)kBins; ++b) slot[slot_of(b, S, merged)] += h[b];
  for (int b = 0; b < kBins; ++b) sum[b + 1] = sum[b] + slot[b];
  segments(S, merged, n, cus, [&](uint32_t s) { return sum[s]; }, seg);
}
