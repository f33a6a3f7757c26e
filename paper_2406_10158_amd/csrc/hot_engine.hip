// OCC's hot-row engine: the transactions of a batch that write one of its hot
// rows run first, in batch order, through the chain scan (chain.hip); the
// rest of the batch then runs in the transaction kernel, where the hot rows
// are only read.
//
// Why: under skew the batch is serialised on its hottest rows.  In the
// transaction kernel each commit on a row takes about 3.6 us (three round trips
// to the coherent level while it is held, and the gap until a contender that
// backed off comes back), so that a row written H times costs at least 3.6 H
// us whatever else runs.  The transactions' operations are known before the run
// and any serial order will do, so the ones on hot rows are given one -- their
// order in the batch -- and executed by it, as the conflict-graph schemes do:
// sorted by cell, every cell's accesses are a prefix sum.  That costs the same
// per operation however hot the row is (the first engine, one workgroup with
// the hot rows in LDS, still took 1.4 us per commit on the hottest row).
//
//   split   which transactions write a hot row (a bit per row, set at
//           submission for every row written more than once, which leaves
//           the rest no write to conflict on; or, where the caller forces the
//           engine on another batch, the rows of its plan); scans give each its place and its operations' places;
//   list    a compact copy of the engine's operations in engine order, with
//           their cells as sort keys;
//   (sort and chain scan)
//   commit  outcome records: ticket = place in the engine's order.
// Serial key (0, ticket), as OCC.  Every engine transaction comes before every
// other one, whose tickets are drawn later, and no word of a row needs a ticket:
// the rest reads words that were cleared with the run.
//
// What bounds it: the sort's passes and the scan's random accesses, about 0.1
// ns an operation, and a dozen launches for a small batch.  Measured, run time:
// 10M rows x 10 fields, 1M transactions x 16 ops, Zipf 0.9: 249 ms with the one
// workgroup, 1.82 ms now; 2^18 transactions on 1M rows, Zipf 0.6: 10.1 ms in
// the transaction kernel as it was, 0.45 ms now; 2^18 transactions on 65,536 rows,
// uniform: 9.3 and 0.41 ms.
#include "opset.h"

namespace cce {

namespace {
constexpr int SPLIT_L = 16;  // lanes per transaction
}

// Per transaction: its operations if it is the engine's, else 0.
template <bool MAP>
__global__ void __launch_bounds__(256) split_flags_kernel(const DevOp *ops, const DevTxn *txns, uint64_t n_txns,
                                                          EngineRows e, const uint32_t *map, uint32_t *flag,
                                                          uint32_t *n_ops, uint64_t *waits) {
  const uint32_t tl = threadIdx.x % SPLIT_L;
  const int tb = __lane_id() - (int)tl;
  uint32_t behind = 0;
  const uint64_t step = (uint64_t)gridDim.x * (256 / SPLIT_L);
  for (uint64_t t0 = (uint64_t)blockIdx.x * (256 / SPLIT_L); t0 < n_txns; t0 += step) {
    const uint64_t t = t0 + threadIdx.x / SPLIT_L;
    DevTxn d{0, 0};
    if (t < n_txns) d = txns[t];
    bool write = false;
    uint32_t touch = 0;
    for (uint32_t j = tl; j < d.n; j += SPLIT_L) {
      const uint32_t rk = ops[d.first + j].rowk, row = op_row(rk);
      bool hot = false;
      if constexpr (MAP) {
        hot = (map[row >> 5] >> (row & 31)) & 1u;
      } else {
#pragma unroll
        for (int k = 0; k < ENG_MAX; ++k) hot |= (uint32_t)k < e.n_rows && e.row[k] == row;
      }
      write |= hot && op_written(rk);
      touch += hot && op_leader(rk);
    }
    const bool mine = ((ballot(write) >> tb) & 0xFFFFull) != 0;
    behind += mine ? touch : 0;
    if (t < n_txns && tl == 0) {
      flag[t] = mine ? 1u : 0u;
      n_ops[t] = mine ? d.n : 0u;
    }
  }
  __shared__ uint32_t sum;
  if (threadIdx.x == 0) sum = 0;
  __syncthreads();
  const uint32_t w = (uint32_t)wave_sum(behind);
  if (__lane_id() == 0 && w) atomicAdd(&sum, w);
  __syncthreads();
  if (threadIdx.x == 0 && sum) add_word(waits, sum);
}

__global__ void __launch_bounds__(64) split_ends_kernel(uint32_t *flag, uint32_t *n_ops, uint64_t n_txns, uint64_t *waits) {
  if (threadIdx.x == 0) {
    flag[n_txns] = n_ops[n_txns] = 0;
    *waits = 0;
  }
}

// Engine transactions first, then the others, each in batch order; `before`
// and `at` are the exclusive scans of the flags and of the operations.
__global__ void __launch_bounds__(256) split_lists_kernel(const DevTxn *txns, uint64_t n_txns, const uint32_t *before,
                                                          const uint32_t *at, uint32_t *part, EngineDesc *desc) {
  const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= n_txns) return;
  const uint32_t k = before[t];
  if (before[t + 1] != k) {
    const DevTxn d = txns[t];
    part[k] = (uint32_t)t;
    desc[k] = EngineDesc{(uint32_t)t, d.first, d.n, at[t]};
  } else {
    part[before[n_txns] + (uint32_t)t - k] = (uint32_t)t;
  }
}

hipError_t launch_split(hipStream_t s, const DevOp *ops, const DevTxn *txns, uint64_t n_txns, const EngineRows &e,
                        const uint32_t *map, uint32_t *scratch, uint32_t *part, EngineDesc *desc, int n_cu) {
  if (n_txns == 0) return hipSuccess;
  uint64_t *waits = (uint64_t *)scratch;
  uint32_t *flag = scratch + 2, *n_ops = flag + n_txns + 1, *partial = n_ops + n_txns + 1;
  const uint64_t blocks = (n_txns + 255) / 256, teams = (n_txns + 256 / SPLIT_L - 1) / (256 / SPLIT_L);
  const uint64_t most = (uint64_t)n_cu * 8;
  const dim3 g((unsigned)(teams < most ? teams : most));
  hipLaunchKernelGGL(split_ends_kernel, dim3(1), dim3(64), 0, s, flag, n_ops, n_txns, waits);
  if (map)
    hipLaunchKernelGGL((split_flags_kernel<true>), g, dim3(256), 0, s, ops, txns, n_txns, e, map, flag, n_ops, waits);
  else
    hipLaunchKernelGGL((split_flags_kernel<false>), g, dim3(256), 0, s, ops, txns, n_txns, e, map, flag, n_ops, waits);
  exclusive_scan_u32(s, flag, n_txns + 1, partial);
  exclusive_scan_u32(s, n_ops, n_txns + 1, partial);
  if (part)
    hipLaunchKernelGGL(split_lists_kernel, dim3((unsigned)blocks), dim3(256), 0, s, txns, n_txns, flag, n_ops, part,
                       desc);
  return hipGetLastError();
}

// The engine's operations in engine order: descriptors whose cell (which the
// sort key carries) is replaced by the operation's index, and the sort's input.
// Clears what the chain kernels count up from zero.
__global__ void __launch_bounds__(256) engine_list_kernel(const DevOp *ops, const EngineDesc *desc, uint64_t n_txns,
                                                          uint64_t n, DevOp *list, uint32_t *keys, uint32_t *vals,
                                                          uint64_t *meta, uint64_t n_tiles, uint32_t *ready,
                                                          uint32_t *txn_first) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n_tiles) meta[i] = 0;
  const uint64_t k = i / SPLIT_L;
  if (k >= n_txns) return;
  const EngineDesc d = desc[k];
  for (uint32_t j = (uint32_t)(i % SPLIT_L); j < d.n; j += SPLIT_L) {
    const uint32_t p = d.at + j;
    if (p >= n) return;
    DevOp o = ops[d.first + j];
    keys[p] = o.elem;
    vals[p] = p;
    o.elem = d.first + j;
    list[p] = o;
    if (ready) ready[p] = 0;
    if (txn_first) txn_first[p] = d.at;
  }
}

// The engine's transactions commit, in their order; a run that stopped leaves
// them pending.  The claim counters go back to 0 for the transaction kernel.
__global__ void __launch_bounds__(256) engine_commit_kernel(const EngineDesc *desc, uint64_t n, DevOutcome *out,
                                                            Ctl *ctl, uint32_t ns_per_tick_q16, uint64_t ticket0) {
  const uint64_t k = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (ld_word(&ctl->stop)) return;
  const uint64_t dt = wall_clock64() - ctl->start_clock;
  if (k < n) {
    DevOutcome o;
    o.status = CC_COMMITTED;
    o.attempts = 1;
    o.serial_hi = 0;
    o.serial_lo = ticket0 + k + 1;
    o.commit_ns = (int64_t)((dt * ns_per_tick_q16) >> 16);
    out[desc[k].txn] = o;
  }
  if (k == 0) {
    ctl->queue = ctl->pending_n = 0;
    ctl->ticket = ticket0 + n;
    ctl->stats[DS_COMMITTED] = ctl->stats[DS_ATTEMPTS] = n;
    ctl->stats[DS_MAX_ATTEMPTS] = 1;
  }
}

size_t engine_scratch_bytes(uint64_t m, bool breaks, bool slots) {
  const uint64_t tiles = chain_tiles(m);
  return m * sizeof(DevOp) + 3 * tiles * 8 + (breaks ? m * 16 : 0) + (slots ? m * 4 : 0) +
         (2 * m + radix_sort_scratch_words(m)) * 4 + 64;
}

hipError_t launch_engine(hipStream_t s, bool strict, const RunArgs &r, const EngineDesc *desc, uint64_t n_txns,
                         uint64_t m, uint64_t n_cells, bool breaks, bool slots, void *scratch, uint64_t ticket0,
                         uint64_t wait_limit_ticks, int n_cu) {
  if (n_txns == 0) return hipSuccess;  // no transaction writes a hot row: the claim counters are at 0 as they are
  const uint64_t tiles = chain_tiles(m);
  ChainArgs a{};
  DevOp *list = (DevOp *)scratch;
  a.ops = list;
  a.n = m;
  a.listed = 1;
  a.data = r.data;
  a.reads = r.reads;
  a.ctl = r.ctl;
  a.wait_limit_ticks = wait_limit_ticks;
  a.meta = (uint64_t *)(list + m);
  a.sum = a.meta + tiles;
  a.total = a.sum + tiles;
  uint32_t *at = (uint32_t *)(a.total + tiles);
  if (breaks) {
    a.result = (uint64_t *)at;
    a.ready = (uint32_t *)(a.result + m);
    a.base = a.ready + m;
    at = a.base + m;
  }
  if (slots) {
    a.txn_first = at;
    at += m;
  }
  uint32_t *keys = at, *vals = keys + m, *sorted_k = nullptr, *sorted_v = nullptr;
  const uint64_t threads = n_txns * SPLIT_L > tiles ? n_txns * SPLIT_L : tiles;
  const uint64_t blocks = (threads + 255) / 256;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(engine_list_kernel, dim3((unsigned)(blocks ? blocks : 1)), dim3(256), 0, s, r.ops, desc, n_txns, m,
                     list, keys, vals, a.meta, tiles, a.ready, a.txn_first);
  int bits = 0;
  while (bits < 32 && ((n_cells - 1) >> bits) != 0) ++bits;
  hipError_t e = radix_sort_pairs(s, keys, vals, m, bits, vals + m, &sorted_k, &sorted_v);
  if (e != hipSuccess) return e;
  a.keys = sorted_k;
  a.vals = sorted_v;
  e = chain_scan(s, strict, a, n_cu);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(engine_commit_kernel, dim3((unsigned)((n_txns + 255) / 256)), dim3(256), 0, s, desc, n_txns, r.out,
                     r.ctl, r.ns_per_tick_q16, ticket0);
  return hipGetLastError();
}

}  // namespace cce
