// The lane tiers' count of evaluated cells (lane_core.h) on the CPU: through a
// state's head, spread over the lanes that resume it, each of which then counts
// `own` more, and summed as the wavefront does.
#include <stdint.h>
#include <string.h>

#include "lane_core.h"

using namespace xd::lane;

template <int S>
static uint64_t carry(uint64_t cells, uint32_t own) {
  const StateHead h = {0, 0, 0, 0, 0, (uint32_t)cells, (uint32_t)S, (uint32_t)(cells >> 32)};
  uint32_t low = 0, high = 0;
  for (int s = 0; s < S; ++s) {
    const uint32_t cnt = count_part<S>(h, s) + own;
    low += cnt & 0xffffu;
    high += cnt >> 16;
  }
  return count_of(low, high);
}

extern "C" uint64_t lane_count(int lanes, uint64_t cells, uint32_t own) {
  switch (lanes) {
    case 4: return carry<4>(cells, own);
    case 8: return carry<8>(cells, own);
    case 16: return carry<16>(cells, own);
    default: return carry<32>(cells, own);
  }
}
