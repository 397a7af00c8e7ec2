// The rule that chooses a batch's kernels (batch_route.h) for the tests.
// in: batched, pair_ok, lane_ok, x_known, x, n_ext, mean_len, tier1, tier2, cus;
// out: queue, packed, solo, lane_blocks, solo_blocks, tier1, tier2.
#include <stdint.h>

#include "batch_route.h"

extern "C" void batch_route(const int64_t* in, int64_t* out) {
  const xd::BatchShape b = {in[0] != 0,          in[1] != 0,     in[2] != 0,     in[3] != 0,
                            (int32_t)in[4],      (uint64_t)in[5], (uint32_t)in[6], (int32_t)in[7],
                            (int32_t)in[8],      (uint32_t)in[9]};
  const xd::Route r = xd::batch_route(b);
  const int64_t o[7] = {r.queue, r.packed, r.solo, r.lane_blocks, r.solo_blocks, r.tier1, r.tier2};
  for (int i = 0; i < 7; ++i) out[i] = o[i];
}
