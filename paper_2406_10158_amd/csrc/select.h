// Selection from histograms: shared by submission's most written rows
// (ingest.hip) and the latency percentiles (latency.hip).
#pragma once

#include "device.h"

namespace cce {

__device__ __forceinline__ uint32_t ld_u32(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True in the workgroup that is last to get here (of nb; *done counts up from 0).  What the others left
// for it they wrote with agent-scope atomics, so their completion is enough
// (write-backs of the caches, 2,048 times, took 0.3 ms).
__device__ __forceinline__ bool last_block(uint64_t *done, uint32_t nb) {
  __shared__ uint32_t mine;
  if (nb == 1) {
    __syncthreads();
    return true;
  }
  order_point<false>();
  __syncthreads();
  if (threadIdx.x == 0) mine = (uint32_t)add_word(done, 1);
  __syncthreads();
  return mine + 1 == nb;
}

// First bin (of `bins`, a multiple of 64 up to 64 x 64, in order or from the
// last down) at which the running count reaches `want`, and the count before
// it; the last one tried if it never does.  Wavefront 0 of a workgroup calls it.
__device__ __forceinline__ void find_bin(const uint32_t *h, uint32_t bins, bool down, uint64_t want, uint32_t *bin,
                                         uint64_t *before) {
  const uint32_t lane = __lane_id(), per = bins / 64;
  auto at = [&](uint32_t k) { return h + (down ? bins - 1 - k : k); };
  auto scan = [&](uint64_t v) {  // inclusive, over the lanes
#pragma unroll
    for (uint32_t o = 1; o < 64; o <<= 1) {
      const uint64_t y = (uint64_t)__shfl_up((long long)v, o, 64);
      if (lane >= o) v += y;
    }
    return v;
  };
  uint64_t sum = 0;
  for (uint32_t i = 0; i < per; ++i) sum += ld_u32(at(lane * per + i));
  uint64_t inc = scan(sum);
  uint64_t reach = ballot(inc >= want);
  const int group = reach ? __ffsll((unsigned long long)reach) - 1 : 63;
  const uint64_t base = (uint64_t)__shfl((long long)(inc - sum), group, 64);
  sum = lane < per ? ld_u32(at((uint32_t)group * per + lane)) : 0;
  inc = scan(sum);
  reach = ballot(lane < per && base + inc >= want);
  const int k = reach ? __ffsll((unsigned long long)reach) - 1 : (int)per - 1;
  *before = base + (uint64_t)__shfl((long long)(inc - sum), k, 64);
  const uint32_t found = (uint32_t)group * per + (uint32_t)k;
  *bin = down ? bins - 1 - found : found;
}

}  // namespace cce
