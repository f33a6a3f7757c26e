// Latency percentiles of a run, and the number of K-sets, from its outcome
// records: the value at rank q (n - 1) + 1/2 (rounded down) of the n committed
// transactions' latencies, for q = 0.5 and 0.99, by histograms of 12 bits of
// the latencies' range at a time.
//
// What bounds it: reading the 32-byte records once a level (range, then two or
// three levels).  On the host, which copied every record and selected there, it
// took longer than the run of an uncontended batch: 4.3 ms for 1M transactions
// (run 2.1 ms), 1.2 ms for 2^18 (0.73 ms).  Now the whole call of a 2^18 batch
// takes 0.1 ms more than its run, and a pass of the 1M batch 2.5 instead of
// 6.8 ms.
#include "select.h"

namespace cce {

namespace {

constexpr uint64_t LAT_SIGN = 1ull << 63;  // orders signed values as unsigned ones

// Records from `arrival` on the latency of a served transaction: commit minus arrival.
__device__ __forceinline__ bool lat_value(const LatArgs &a, uint64_t i, uint64_t *v) {
  const DevOutcome o = a.out[i];
  if (o.status != CC_COMMITTED) return false;
  *v = (uint64_t)(a.arrival_ns ? o.commit_ns - a.arrival_ns[i] : o.commit_ns) ^ LAT_SIGN;
  return true;
}

struct LatRange {
  uint64_t n, min, max, ksets;
};

// A workgroup's committed transactions: how many, the range of their
// latencies, the largest serial_hi + 1.  Every thread gets the result.
template <int NT>
__device__ __forceinline__ LatRange lat_range(const LatArgs &a, uint64_t *lds, uint32_t b, uint32_t nb) {
  LatRange r{0, ~0ull, 0, 0};
  for (uint64_t i = (uint64_t)b * NT + threadIdx.x; i < a.n; i += (uint64_t)nb * NT) {
    uint64_t v = 0;
    if (!lat_value(a, i, &v)) continue;
    ++r.n;
    r.min = v < r.min ? v : r.min;
    r.max = v > r.max ? v : r.max;
    if (a.ksets) {
      const uint64_t h = a.out[i].serial_hi + 1;
      r.ksets = h > r.ksets ? h : r.ksets;
    }
  }
  r.n = wave_sum(r.n);
  r.min = ~wave_max(~r.min);
  r.max = wave_max(r.max);
  r.ksets = wave_max(r.ksets);
  const int w = threadIdx.x / 64;
  if (__lane_id() == 0) {
    lds[4 * w] = r.n;
    lds[4 * w + 1] = r.min;
    lds[4 * w + 2] = r.max;
    lds[4 * w + 3] = r.ksets;
  }
  __syncthreads();
  r = LatRange{0, ~0ull, 0, 0};
  for (int i = 0; i < NT / 64; ++i) {
    r.n += lds[4 * i];
    r.min = lds[4 * i + 1] < r.min ? lds[4 * i + 1] : r.min;
    r.max = lds[4 * i + 2] > r.max ? lds[4 * i + 2] : r.max;
    r.ksets = lds[4 * i + 3] > r.ksets ? lds[4 * i + 3] : r.ksets;
  }
  __syncthreads();
  return r;
}

// What is known after some levels: the values at the two ranks lie in
// min + (prefix << shift) + [0, 1 << shift), at `rank` within it.
struct LatLevel {
  uint64_t min, shift, prefix[2], rank[2];
};

__device__ __forceinline__ LatLevel lat_begin(const LatRange &r) {
  LatLevel l{};
  l.min = r.min;
  const uint64_t span = r.n ? r.max - r.min : 0;
  l.shift = span ? 64 - (uint64_t)__clzll((long long)span) : 0;
  // rank q (n - 1) + 1/2, rounded as the two operations are
  const double m = (double)(r.n ? r.n - 1 : 0);
  l.rank[0] = (uint64_t)__dadd_rn(__dmul_rn(0.50, m), 0.5);
  l.rank[1] = (uint64_t)__dadd_rn(__dmul_rn(0.99, m), 0.5);
  return l;
}

__device__ __forceinline__ uint64_t lat_next_shift(uint64_t shift) { return shift > LAT_BITS ? shift - LAT_BITS : 0; }

// One level's histograms (h[0], h[1]: LAT_BINS each, zeroed) of a workgroup's
// share of the records.
template <int NT>
__device__ __forceinline__ void lat_count(const LatArgs &a, const LatLevel &l, uint32_t *h, uint32_t b, uint32_t nb) {
  const uint64_t next = lat_next_shift(l.shift);
  for (uint64_t i = (uint64_t)b * NT + threadIdx.x; i < a.n; i += (uint64_t)nb * NT) {
    uint64_t v = 0;
    if (!lat_value(a, i, &v)) continue;
    const uint64_t d = v - l.min;
    const uint32_t bin = (uint32_t)((d >> next) & (LAT_BINS - 1));
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (l.shift >= 64 || (d >> l.shift) == l.prefix[q]) atomicAdd(&h[q * LAT_BINS + bin], 1u);
  }
}

// Narrows the two ranks by a level's complete histograms (wavefront 0).
__device__ __forceinline__ LatLevel lat_narrow(LatLevel l, const uint32_t *h) {
  const uint64_t next = lat_next_shift(l.shift);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    uint32_t bin = 0;
    uint64_t before = 0;
    find_bin(h + q * LAT_BINS, LAT_BINS, false, l.rank[q] + 1, &bin, &before);
    l.rank[q] -= before;
    l.prefix[q] = (l.prefix[q] << (l.shift - next)) | bin;
  }
  l.shift = next;
  return l;
}

}  // namespace

// A small batch: one workgroup, the histograms in LDS.  Up to LAT_DIRECT
// transactions each value counts the values below it instead, which needs no
// histograms to clear and search (256 transactions: 24
// and 14 us).
constexpr int LAT_DIRECT = 512;
static_assert(LAT_DIRECT <= LAT_BINS, "the values take the histograms' place");
__global__ void __launch_bounds__(1024) latency_small_kernel(LatArgs a) {
  __shared__ __align__(8) uint32_t h[2 * LAT_BINS];
  __shared__ uint64_t value[2];
  __shared__ uint64_t lds[4 * 16];
  __shared__ LatLevel level;
  const LatRange r = lat_range<1024>(a, lds, 0, 1);
  LatLevel l = lat_begin(r);
  if (a.n <= (uint64_t)LAT_DIRECT) {
    uint64_t *vs = (uint64_t *)h;
    uint64_t v = 0;
    const bool have = threadIdx.x < a.n && lat_value(a, threadIdx.x, &v);
    if (threadIdx.x < (uint32_t)LAT_DIRECT) vs[threadIdx.x] = have ? v : ~0ull;
    __syncthreads();
    if (have) {
      uint64_t less = 0, same = 0;
      for (uint32_t i = 0; i < (uint32_t)a.n; ++i) {
        const uint64_t x = vs[i];
        less += x < v;
        same += x == v;
      }
      // (threads with the same value write the same; an uncommitted one's ~0 is above every rank)
      for (int q = 0; q < 2; ++q)
        if (less <= l.rank[q] && l.rank[q] < less + same) value[q] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int q = 0; q < 2; ++q) a.st->value[q] = r.n ? value[q] ^ LAT_SIGN : 0;
      a.st->ksets = r.ksets;
      a.st->shift = 0;
    }
    return;
  }
  while (l.shift) {
    for (uint32_t i = threadIdx.x; i < 2 * LAT_BINS; i += 1024) h[i] = 0;
    __syncthreads();
    lat_count<1024>(a, l, h, 0, 1);
    __syncthreads();
    if (threadIdx.x < 64) {
      l = lat_narrow(l, h);
      if (threadIdx.x == 0) level = l;
    }
    __syncthreads();
    l = level;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.st->value[0] = r.n ? (l.min + l.prefix[0]) ^ LAT_SIGN : 0;
    a.st->value[1] = r.n ? (l.min + l.prefix[1]) ^ LAT_SIGN : 0;
    a.st->ksets = r.ksets;
    a.st->shift = 0;
  }
}

__global__ void __launch_bounds__(1024) latency_range_kernel(LatArgs a) {
  __shared__ uint64_t lds[4 * 16];
  for (uint64_t i = (uint64_t)blockIdx.x * 1024 + threadIdx.x; i < (uint64_t)LAT_LEVELS * 2 * LAT_BINS;
       i += (uint64_t)gridDim.x * 1024)
    a.hist[i] = 0;
  const LatRange r = lat_range<1024>(a, lds, blockIdx.x, gridDim.x);
  if (threadIdx.x == 0) {
    if (r.n) {
      add_word(&a.st->n, r.n);
      atomicMax((unsigned long long *)&a.st->not_min, (unsigned long long)~r.min);
      atomicMax((unsigned long long *)&a.st->max, (unsigned long long)r.max);
    }
    if (r.ksets) atomicMax((unsigned long long *)&a.st->ksets, (unsigned long long)r.ksets);
  }
  if (!last_block(&a.st->done[0], gridDim.x)) return;
  if (threadIdx.x == 0) {
    const LatRange all{ld_word(&a.st->n), ~ld_word(&a.st->not_min), ld_word(&a.st->max), 0};
    const LatLevel l = lat_begin(all);
    a.st->shift = l.shift;
    for (int q = 0; q < 2; ++q) {
      a.st->prefix[q] = 0;
      a.st->rank[q] = l.rank[q];
      a.st->value[q] = all.n ? all.min ^ LAT_SIGN : 0;
    }
  }
}

__global__ void __launch_bounds__(1024) latency_level_kernel(LatArgs a, int level) {
  __shared__ uint32_t h[2 * LAT_BINS];
  if (a.st->shift == 0) return;  // (changed by the last workgroup only, when every other has read it)
  LatLevel l{~a.st->not_min, a.st->shift, {a.st->prefix[0], a.st->prefix[1]}, {a.st->rank[0], a.st->rank[1]}};
  for (uint32_t i = threadIdx.x; i < 2 * LAT_BINS; i += 1024) h[i] = 0;
  __syncthreads();
  lat_count<1024>(a, l, h, blockIdx.x, gridDim.x);
  __syncthreads();
  uint32_t *g = a.hist + (uint64_t)level * 2 * LAT_BINS;
  for (uint32_t i = threadIdx.x; i < 2 * LAT_BINS; i += 1024)
    if (h[i]) atomicAdd(&g[i], h[i]);
  if (!last_block(&a.st->done[1 + level], gridDim.x)) return;
  if (threadIdx.x < 64) {
    l = lat_narrow(l, g);
    if (threadIdx.x == 0) {
      a.st->shift = l.shift;
      for (int q = 0; q < 2; ++q) {
        a.st->prefix[q] = l.prefix[q];
        a.st->rank[q] = l.rank[q];
        a.st->value[q] = (l.min + l.prefix[q]) ^ LAT_SIGN;
      }
    }
  }
}

hipError_t launch_latency(hipStream_t s, const LatArgs &a, int n_cu) {
  if (a.n <= (uint64_t)LAT_SMALL) {
    hipLaunchKernelGGL(latency_small_kernel, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
  }
  const uint64_t need = (a.n + 4095) / 4096;
  const dim3 g((unsigned)(need < (uint64_t)n_cu ? need : (uint64_t)n_cu));
  hipLaunchKernelGGL(latency_range_kernel, g, dim3(1024), 0, s, a);
  for (int i = 0; i < LAT_LEVELS; ++i) hipLaunchKernelGGL(latency_level_kernel, g, dim3(1024), 0, s, a, i);
  return hipGetLastError();
}

}  // namespace cce
