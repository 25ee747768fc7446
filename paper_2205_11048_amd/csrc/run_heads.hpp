// Device side of RunHeads: a block's base number from the two levels.
#pragma once

#include "gba_device.hpp"
#include "gba_internal.hpp"

namespace gba {

// The runs before the group that holds `tile`, for a whole block of 256
// threads, in two calls with a block barrier between them: run_base loads and
// adds each wave's share of the earlier groups' counts (or takes the scanned
// value), run_base_sum joins the four waves.  The loads are clamped, not
// branched around or looped over, so that they are in flight together with
// whatever the caller has issued before (a loop made the position pass 16 us
// slower at 400 groups).
__device__ __forceinline__ void run_base(const RunHeads& h, int64_t tile, uint32_t* s_wave) {
  constexpr int kLoads = (int)(kRunFoldGroups / 256);
  const int g = (int)(tile >> h.shift);
  uint32_t s = 0;
  if (h.scanned) {
    s = threadIdx.x == 0 ? h.group[g] : 0u;
  } else {
    uint32_t v[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int i = (int)threadIdx.x + 256 * k;
      v[k] = h.group[i < h.groups ? i : h.groups - 1];
    }
#pragma unroll
    for (int k = 0; k < kLoads; ++k) s += (int)threadIdx.x + 256 * k < g ? v[k] : 0u;
  }
  s = wave_sum(s);
  if (lane_id() == 0) s_wave[threadIdx.x / kWave] = s;
}
__device__ __forceinline__ uint32_t run_base_sum(const uint32_t* s_wave) {
  return s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
}

}  // namespace gba
