// The frontier statistics' per-block results, added up by the kernels that
// publish the control block.
#pragma once

#include <cstddef>

#include "gr_internal.h"
#include "k_common.h"

namespace gr {

constexpr int kPublishBlock = 256;

// m_f and max_deg of one statistics slot as the 32-bit words of the control
// block: low and high word of each.
struct StatsTotal {
  uint32_t w[4];
};

__device__ __forceinline__ int stats_word_at(int slot, int i) {
  constexpr int kM = (int)(offsetof(Ctrl, m_f) / 4), kD = (int)(offsetof(Ctrl, max_deg) / 4);
  return (i < 2 ? kM : kD) + 2 * slot + (i & 1);
}
__device__ __forceinline__ bool stats_word(int slot, int i) {
  return i == stats_word_at(slot, 0) || i == stats_word_at(slot, 1) ||
         i == stats_word_at(slot, 2) || i == stats_word_at(slot, 3);
}

// Sum and maximum of the kStatsGrid packed block results into *t (shared
// memory).  Every thread of the kPublishBlock-thread workgroup calls it; it
// synchronises the workgroup.
__device__ __forceinline__ void stats_total(const StatsSum& s, StatsTotal* t) {
  __shared__ int64_t s_sum[kPublishBlock / kWave];
  __shared__ uint32_t s_max[kPublishBlock / kWave];
  int64_t x[kStatsGrid / kPublishBlock];
#pragma unroll
  for (int r = 0; r < kStatsGrid / kPublishBlock; ++r)
    x[r] = s.block_sums[r * kPublishBlock + threadIdx.x];
  int64_t sum = 0;
  uint32_t mx = 0;
#pragma unroll
  for (int r = 0; r < kStatsGrid / kPublishBlock; ++r) {
    sum += (uint32_t)x[r];
    const uint32_t d = (uint32_t)(x[r] >> 32);
    mx = d > mx ? d : mx;
  }
  sum = wave_sum(sum);
  mx = wave_max(mx);
  if (lane() == 0) {
    s_sum[threadIdx.x / kWave] = sum;
    s_max[threadIdx.x / kWave] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t m = 0;
    uint32_t d = 0;
    for (int i = 0; i < kPublishBlock / kWave; ++i) {
      m += s_sum[i];
      d = s_max[i] > d ? s_max[i] : d;
    }
    t->w[0] = (uint32_t)m;
    t->w[1] = (uint32_t)(m >> 32);
    t->w[2] = d;
    t->w[3] = 0u;
  }
  __syncthreads();
}

}  // namespace gr
