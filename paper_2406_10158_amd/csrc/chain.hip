// Ordered execution of transactions by cell chains, for a serial order that is
// known before the run (GaccO: transaction ids; GPUTx: its K-sets put
// conflicting transactions in id order too, so the same values result; OCC's
// hot-row engine: batch order, of its share of the batch, hot_engine.hip).
//
// Given the order, what an operation reads depends only on the earlier
// operations of its own cell: a transaction touches a cell at most once, and
// only a slot write takes a value from another cell.  So instead of handing
// every row from transaction to transaction through memory (one round trip to
// the coherent level, 1.5 us, for each access of the hottest row), the
// accesses are sorted by cell -- stable, so that each cell's list is in serial
// order -- and a cell's list is a prefix sum:
//   1. chain_scan: a segmented scan over the sorted list in one pass (tiles
//      of 2,048 accesses; a tile whose first access continues a chain looks
//      back over its predecessors' sums: the published "decoupled look-back" of
//      Merrill and Garland's single-pass prefix scan).  A read adds 0, an add its argument,
//      a slot write that multiplies its source by 0 sets a constant.  Every
//      access gets its pre-image, every chain's last access stores the cell.
//   2. batches with conditional adds or slot writes: such an access is a
//      break, whose result the scan cannot know.  The accesses after it are
//      summed relative to it, and chain_break resolves the breaks in serial
//      order, each from at most one earlier break (the one its own value, or
//      its source's, is relative to): a wavefront takes 64 consecutive
//      operations, resolves what it can from its own lanes, publishes, and
//      waits only for breaks of lower operations, which a wavefront that is
//      already running has taken.  chain_finish then adds the breaks' results.
//   3. chain_outcomes: the outcome records.
// What bounds it: the random accesses -- a 16-byte descriptor and an 8-byte
// read value per operation -- and the sort before it (gacco.hip).  2^18
// transactions x 16 ops, 10M rows, Zipf 0.9: the row-by-row hand-off took
// 132 ms (86k accesses of the hottest row), the sort and the scan take 0.20
// and 0.26 ms.  Order-entry, 8 warehouses, 2^13 transactions: 4.1 ms before,
// now 0.10 ms after 0.1 ms of sorting, 69 us of it the breaks.
#include "opset.h"

namespace cce {

constexpr int CH_THREADS = 256;
constexpr int CH_ITEMS = 8;
constexpr int CH_TILE = CH_THREADS * CH_ITEMS;

// What is known of a cell's value at a place of its chain: v plus the value
// on entry (REL), v itself (ABS), or v plus the result of break `b` (BRK).
enum ChainBase : uint32_t { CH_REL = 0, CH_ABS = 1, CH_BRK = 2 };
struct ChainVal {
  uint64_t v;
  uint32_t f, b;
};
__device__ __forceinline__ ChainVal ch_then(const ChainVal &x, const ChainVal &y) {
  ChainVal r = y;
  if (y.f == CH_REL) {
    r.f = x.f;
    r.b = x.b;
    r.v = x.v + y.v;
  }
  return r;
}
__device__ __forceinline__ ChainVal ch_shfl_up(const ChainVal &x, int o) {
  ChainVal r;
  r.v = (uint64_t)__shfl_up((long long)x.v, o, 64);
  r.f = (uint32_t)__shfl_up((int)x.f, o, 64);
  r.b = (uint32_t)__shfl_up((int)x.b, o, 64);
  return r;
}

// A slot write whose multiplier is 0 stores a constant.
__device__ __forceinline__ bool slot_const(int64_t arg) { return (((uint64_t)arg >> 8) & 0xFFFFFFull) == 0; }
__device__ __forceinline__ bool ch_is_break(uint32_t kind, int64_t arg) {
  return kind == CC_COND_ADD || (kind == CC_WRITE_SLOT && !slot_const(arg));
}

// An access's effect on its cell (op: its operation index, for breaks).
__device__ __forceinline__ ChainVal ch_effect(uint32_t kind, int64_t arg, uint32_t op) {
  ChainVal e{0, CH_REL, 0};
  if (kind == CC_ADD) {
    e.v = (uint64_t)arg;
  } else if (kind != CC_READ) {
    if (ch_is_break(kind, arg)) {
      e.f = CH_BRK;
      e.b = op;
    } else {
      e.f = CH_ABS;
      e.v = (uint64_t)apply_op(CC_WRITE_SLOT, 0, arg, 0);
    }
  }
  return e;
}

// Sort keys: the cell of every operation.  (A gap, which no transaction names,
// sits in cell 0's chain, changes nothing and gets no read value.)  Clears
// what the later kernels of the run count up from zero: the tiles' states and,
// with breaks, the breaks' ready words.
__global__ void __launch_bounds__(256) chain_keys_kernel(const DevOp *ops, uint64_t n, uint32_t *keys, uint32_t *vals,
                                                         uint64_t *meta, uint64_t n_tiles, uint32_t *ready) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_tiles) meta[i] = 0;
  if (i >= n) return;
  keys[i] = ops[i].elem;
  vals[i] = (uint32_t)i;
  if (ready) ready[i] = 0;
}

// Tile states for the look-back: meta is 0 until the tile has published, then
// 1 with its sum relative to its entry in sum[], or 2 | f << 2 | b << 32 with
// its value at the end in total[].  A value is performed before its meta.
// CHM_SETTLED: the chain at the tile's end has its initial value loaded, by a
// tile that the chain begins in.  A constant slot write or a break gives a tile
// its total whatever comes before it, so that a total alone does not say so; a
// workgroup that ends a chain it did not begin stores the cell only once a tile
// before it is settled, or the first tile could load what the last one stored.
constexpr uint64_t CHM_SUM = 1, CHM_TOTAL = 2, CHM_SETTLED = 16;
__device__ __forceinline__ uint64_t chm_total(const ChainVal &x, bool settled) {
  return CHM_TOTAL | (settled ? CHM_SETTLED : 0) | ((uint64_t)x.f << 2) | ((uint64_t)x.b << 32);
}

template <bool BREAKS, bool STRICT>
__global__ void __launch_bounds__(CH_THREADS) chain_scan_kernel(ChainArgs a) {
  __shared__ uint32_t tile_s;
  __shared__ ChainVal wave_s[CH_THREADS / 64];
  __shared__ ChainVal entry_s;
  __shared__ uint32_t mark_s[CH_THREADS / 64];  // 1: a chain begins among the wavefront's accesses, 2: one ends there
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (ld_word(&a.ctl->stop)) return;  // GPUTx: the rank pass was stopped (not changed while this kernel runs)
  // tiles are taken in order, so the tiles a look-back waits for belong to
  // running workgroups or are done
  if (tid == 0) tile_s = (uint32_t)add_word(&a.ctl->queue, 1);
  __syncthreads();
  const uint64_t tile = tile_s;
  const uint64_t p0 = tile * CH_TILE + (uint64_t)tid * CH_ITEMS;
  uint32_t key[CH_ITEMS], op[CH_ITEMS];
#pragma unroll
  for (int j = 0; j < CH_ITEMS; ++j) {
    key[j] = p0 + j < a.n ? a.keys[p0 + j] : 0u;
    op[j] = p0 + j < a.n ? a.vals[p0 + j] : 0u;
  }
  const uint32_t before = p0 > 0 && p0 <= a.n ? a.keys[p0 - 1] : 0u;
  const uint32_t after = p0 + CH_ITEMS < a.n ? a.keys[p0 + CH_ITEMS] : 0u;
  uint32_t kind[CH_ITEMS], read[CH_ITEMS];  // read: where the access's read value goes
  int64_t arg[CH_ITEMS], init[CH_ITEMS];
  bool ok[CH_ITEMS], gap[CH_ITEMS], head[CH_ITEMS], last[CH_ITEMS];
#pragma unroll
  for (int j = 0; j < CH_ITEMS; ++j) {
    ok[j] = p0 + j < a.n;
    head[j] = ok[j] && (p0 + j == 0 || (j ? key[j - 1] : before) != key[j]);
    last[j] = ok[j] && (p0 + j + 1 == a.n || (j + 1 < CH_ITEMS ? key[j + 1] : after) != key[j]);
    kind[j] = CC_READ;
    arg[j] = init[j] = 0;
    gap[j] = true;
    read[j] = op[j];
    if (ok[j]) {
      const DevOp o = a.ops[op[j]];
      gap[j] = o.rowk == GAP_OP;
      if (!gap[j]) kind[j] = op_kind(o.rowk);
      arg[j] = o.arg;
      if (a.listed) read[j] = o.elem;
    }
    if (head[j]) init[j] = a.data[key[j]];
  }
  // the thread's accesses, then the wavefront's and the workgroup's prefix
  bool begins = false, ends = false;
  ChainVal run{0, CH_REL, 0};
#pragma unroll
  for (int j = 0; j < CH_ITEMS; ++j) {
    if (head[j]) run = ChainVal{(uint64_t)init[j], CH_ABS, 0};
    run = ch_then(run, ch_effect(kind[j], arg[j], op[j]));
    begins |= head[j];
    ends |= last[j];
  }
  ChainVal inc = run;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const ChainVal y = ch_shfl_up(inc, o);
    if (lane >= o) inc = ch_then(y, inc);
  }
  ChainVal pre = ch_shfl_up(inc, 1);
  if (lane == 0) pre = ChainVal{0, CH_REL, 0};
  if (lane == 63) wave_s[w] = inc;
  const uint32_t mark = (ballot(begins) ? 1u : 0u) | (ballot(ends) ? 2u : 0u);
  if (lane == 0) mark_s[w] = mark;
  order_point<STRICT>();  // the initial values are in registers before the workgroup publishes (CHM_SETTLED) or stores
  __syncthreads();
  ChainVal all{0, CH_REL, 0}, waves{0, CH_REL, 0};
  uint32_t marks = 0;
#pragma unroll
  for (int i = 0; i < CH_THREADS / 64; ++i) {
    if (i == w) waves = all;
    all = ch_then(all, wave_s[i]);
    marks |= mark_s[i];
  }
  if (w == 0) {
    // (only wavefront 0: lane 0 holds the tile's first access)
    const bool cont = __shfl((int)(ok[0] && !head[0]), 0, 64) != 0;
    if (lane == 0 && (all.f != CH_REL || cont)) {
      if (all.f == CH_REL) st_word(a.sum + tile, all.v);
      else st_word(a.total + tile, all.v);
    }
    order_point<STRICT>();
    if (lane == 0 && (all.f != CH_REL || cont))
      st_word(a.meta + tile, all.f == CH_REL ? CHM_SUM : chm_total(all, marks & 1u));
    ChainVal entry{0, CH_REL, 0};
    if (cont) {
      // look back, 64 tiles at a time, to the nearest one whose value at its
      // end is known; the tiles between give their sums
      int64_t at = (int64_t)tile - 1;
      bool settled = false;
      for (;;) {
        const int64_t t = at - lane;
        const uint64_t m = t >= 0 ? ld_word(a.meta + t) : CHM_TOTAL | CHM_SETTLED;
        const uint64_t done = ballot((m & 3) == CHM_TOTAL), none = ballot((m & 3) == 0);
        const uint64_t upto = done ? (done & -done) | ((done & -done) - 1) : ~0ull;
        if (none & upto) {
          __builtin_amdgcn_s_sleep(1);
          continue;
        }
        order_point<STRICT>();
        uint64_t v = 0;
        if (((upto >> lane) & 1) && t >= 0) v = ld_word(((m & 3) == CHM_TOTAL ? a.total : a.sum) + t);
        entry.v += wave_sum(v);
        if (done) {
          const uint64_t md = readlane64(m, __ffsll((unsigned long long)done) - 1);
          entry.f = (uint32_t)(md >> 2) & 3u;
          entry.b = (uint32_t)(md >> 32);
          settled = (md & CHM_SETTLED) != 0;
          break;
        }
        at -= 64;
      }
      if (all.f == CH_REL) {
        if (lane == 0) st_word(a.total + tile, entry.v + all.v);
        order_point<STRICT>();
        if (lane == 0) st_word(a.meta + tile, chm_total(entry, settled));
      }
      // the chain ends here: on to the nearest settled tile.  Those between
      // belong to the chain, as one that a chain begins in is settled; every
      // tile is, or publishes without a wait, so that this one ends
      at = (int64_t)tile - 1;
      while ((marks & 2u) && !settled) {
        const int64_t t = at - lane;
        const uint64_t m = t >= 0 ? ld_word(a.meta + t) : CHM_SETTLED;
        const uint64_t found = ballot((m & CHM_SETTLED) != 0), none = ballot(m == 0);
        const uint64_t upto = found ? (found & -found) | ((found & -found) - 1) : ~0ull;
        if (none & upto) {
          __builtin_amdgcn_s_sleep(1);
          continue;
        }
        settled = found != 0;
        at -= 64;
      }
      order_point<STRICT>();
    }
    if (lane == 0) entry_s = entry;
  }
  __syncthreads();
  ChainVal st = ch_then(entry_s, ch_then(waves, pre));
#pragma unroll
  for (int j = 0; j < CH_ITEMS; ++j) {
    if (head[j]) st = ChainVal{(uint64_t)init[j], CH_ABS, 0};
    if (ok[j]) {
      if (!gap[j]) __builtin_nontemporal_store((int64_t)st.v, a.reads + read[j]);
      else if (BREAKS) a.result[op[j]] = st.v;  // chain_finish's value of the cell, if the chain ends here
      if (BREAKS) a.base[op[j]] = st.f == CH_BRK ? st.b + 1 : 0u;
    }
    st = ch_then(st, ch_effect(kind[j], arg[j], op[j]));
    // a cell that only one operation reads keeps its value
    if (last[j] && st.f == CH_ABS && !(head[j] && kind[j] == CC_READ)) a.data[key[j]] = (int64_t)st.v;
  }
}

// Breaks, in operation order (the serial order).  A break's result needs the
// value its own pre-image (conditional add) or its source's read value (slot
// write) is relative to: base[] names that earlier break, 0 = none.
template <bool STRICT>
__global__ void __launch_bounds__(256) chain_break_kernel(ChainArgs a) {
  const int lane = __lane_id();
  if (ld_word(&a.ctl->stop)) return;
  for (;;) {
    uint64_t c0 = 0;
    if (lane == 0) c0 = add_word(&a.ctl->pending_n, 64);
    c0 = readlane64(c0, 0);
    if (c0 >= a.n) break;
    const uint64_t i = c0 + lane;
    DevOp o{GAP_OP, 0, 0};
    if (i < a.n) o = a.ops[i];
    const uint32_t kind = op_kind(o.rowk);
    const bool brk = o.rowk != GAP_OP && ch_is_break(kind, o.arg);
    if (ballot(brk) == 0) continue;
    uint32_t dep = 0;   // 1 + the break this one waits for
    uint64_t rel = 0;   // the pre-image / source value, relative to it
    if (brk) {
      const uint64_t from = kind == CC_COND_ADD ? i : (uint64_t)a.txn_first[i] + (uint64_t)(o.arg & 0xFF);
      dep = a.base[from];
      rel = (uint64_t)a.reads[a.listed ? a.ops[from].elem : (uint32_t)from];
    }
    bool done = !brk, told = !brk;
    uint64_t res = 0;
    const int near = dep && (uint64_t)dep - 1 >= c0 ? (int)((uint64_t)dep - 1 - c0) : -1;  // a lane of this wavefront
    const uint64_t began = wall_clock64();
    for (uint32_t polls = 0;; ++polls) {
      uint64_t got = 0;
      bool have = !done && dep == 0;
      if (!done && dep && near < 0 && __hip_atomic_load(a.ready + (dep - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        have = true;
      order_point<STRICT>();  // a ready word before its result
      if (have && dep) got = ld_word(a.result + (dep - 1));
      // then whatever follows inside the wavefront
      for (;;) {
        if (have) {
          const int64_t x = (int64_t)(got + rel);
          res = (uint64_t)(kind == CC_COND_ADD ? apply_op(CC_COND_ADD, x, o.arg, 0)
                                               : apply_op(CC_WRITE_SLOT, 0, o.arg, x));
          done = true;
        }
        const uint64_t r = (uint64_t)__shfl((long long)res, near < 0 ? 0 : near, 64);
        const bool rd = __shfl((int)done, near < 0 ? 0 : near, 64) != 0;
        have = !done && near >= 0 && rd;
        got = r;
        if (ballot(have) == 0) break;
      }
      const bool tell = done && !told;
      if (tell) st_word(a.result + i, res);
      order_point<STRICT>();
      if (tell) __hip_atomic_store(a.ready + i, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      told = told || tell;
      if (ballot(!done) == 0) break;
      // the breaks waited for belong to lower operations, taken by running
      // wavefronts; the limit is a safeguard
      if (wall_clock64() - began > a.wait_limit_ticks) st_word(&a.ctl->stop, 1);
      if ((polls & 63u) == 63u && ld_word(&a.ctl->stop)) return;
      __builtin_amdgcn_s_sleep(1);
    }
  }
}

// Adds the breaks' results to what is relative to them, and stores the cells
// whose chains have a break.
__global__ void __launch_bounds__(256) chain_finish_kernel(ChainArgs a) {
  const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= a.n || ld_word(&a.ctl->stop)) return;
  const uint32_t key = a.keys[p], op = a.vals[p];
  const DevOp o = a.ops[op];
  const bool gap = o.rowk == GAP_OP;
  const uint32_t kind = gap ? (uint32_t)CC_READ : op_kind(o.rowk);
  const uint32_t dep = a.base[op];
  const uint32_t read = a.listed ? o.elem : op;
  uint64_t x = gap ? a.result[op] : (uint64_t)a.reads[read];
  if (dep) {
    x += a.result[dep - 1];
    if (!gap) a.reads[read] = (int64_t)x;
  }
  const bool brk = ch_is_break(kind, o.arg);
  const bool last = p + 1 >= a.n || a.keys[p + 1] != key;
  if (!last || (!dep && !brk)) return;
  if (brk) a.data[key] = (int64_t)a.result[op];
  else a.data[key] = apply_op(kind, (int64_t)x, o.arg, 0);
}

// Every transaction commits with the batch; a run that stopped (the breaks'
// wait limit) leaves them pending.
__global__ void __launch_bounds__(256) chain_outcomes_kernel(DevOutcome *out, uint64_t n, const uint32_t *rank,
                                                             Ctl *ctl, uint32_t ns_per_tick_q16) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool ok = ctl->stop == 0;
  const uint64_t dt = wall_clock64() - ctl->start_clock;
  if (t < n) {
    DevOutcome o;
    o.status = ok ? CC_COMMITTED : CC_PENDING;
    o.attempts = ok ? 1 : 0;
    o.serial_hi = ok && rank ? rank[t] : 0;
    o.serial_lo = ok ? t : 0;
    o.commit_ns = ok ? (int64_t)((dt * ns_per_tick_q16) >> 16) : -1;
    out[t] = o;
  }
  if (t == 0 && ok) {
    ctl->stats[DS_COMMITTED] = n;
    ctl->stats[DS_ATTEMPTS] = n;
    ctl->stats[DS_MAX_ATTEMPTS] = n ? 1 : 0;
  }
}

// First operation of every operation's transaction, for slot sources.
__global__ void __launch_bounds__(256) chain_txn_first_kernel(const DevTxn *txns, uint64_t n_txns, uint32_t *txn_first) {
  const uint64_t t = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / 16;
  if (t >= n_txns) return;
  const DevTxn d = txns[t];
  for (uint32_t j = threadIdx.x & 15; j < d.n; j += 16) txn_first[d.first + j] = d.first;
}

uint64_t chain_tiles(uint64_t n) { return (n + CH_TILE - 1) / CH_TILE; }

hipError_t chain_prepare(hipStream_t s, const ChainArgs &a, uint64_t n_cells, const DevTxn *txns, uint64_t n_txns, uint32_t *keys,
                         uint32_t *vals, uint32_t *sort_scratch, uint32_t **keys_out, uint32_t **vals_out) {
  *keys_out = keys;
  *vals_out = vals;
  if (a.n == 0) return hipSuccess;
  const uint64_t blocks = (a.n + 255) / 256;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(chain_keys_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a.ops, a.n, keys, vals, a.meta,
                     chain_tiles(a.n), a.ready);
  if (a.txn_first && n_txns)
    hipLaunchKernelGGL(chain_txn_first_kernel, dim3((unsigned)((n_txns * 16 + 255) / 256)), dim3(256), 0, s, txns,
                       n_txns, a.txn_first);
  int bits = 0;
  while (bits < 32 && ((n_cells - 1) >> bits) != 0) ++bits;
  return radix_sort_pairs(s, keys, vals, a.n, bits, sort_scratch, keys_out, vals_out);
}

template <bool STRICT>
static void chain_run(hipStream_t s, const ChainArgs &a, int n_cu) {
  const uint64_t tiles = chain_tiles(a.n);
  if (tiles) {
    const unsigned blocks = (unsigned)((a.n + 255) / 256);
    if (!a.base) {
      hipLaunchKernelGGL((chain_scan_kernel<false, STRICT>), dim3((unsigned)tiles), dim3(CH_THREADS), 0, s, a);
    } else {
      hipLaunchKernelGGL((chain_scan_kernel<true, STRICT>), dim3((unsigned)tiles), dim3(CH_THREADS), 0, s, a);
      // 256 consecutive operations per workgroup and round, one workgroup per CU
      const unsigned grid = blocks < (unsigned)n_cu ? blocks : (unsigned)n_cu;
      hipLaunchKernelGGL((chain_break_kernel<STRICT>), dim3(grid), dim3(256), 0, s, a);
      hipLaunchKernelGGL(chain_finish_kernel, dim3(blocks), dim3(256), 0, s, a);
    }
  }
}

hipError_t chain_scan(hipStream_t s, bool strict, const ChainArgs &a, int n_cu) {
  strict ? chain_run<true>(s, a, n_cu) : chain_run<false>(s, a, n_cu);
  return hipGetLastError();
}

hipError_t chain_execute(hipStream_t s, bool strict, const ChainArgs &a, DevOutcome *out, uint64_t n_txns,
                         const uint32_t *rank, uint32_t ns_per_tick_q16, int n_cu, int *grid_used) {
  *grid_used = (int)chain_tiles(a.n);
  const hipError_t e = chain_scan(s, strict, a, n_cu);
  if (e != hipSuccess) return e;
  const uint64_t bt = (n_txns + 255) / 256;
  hipLaunchKernelGGL(chain_outcomes_kernel, dim3((unsigned)(bt ? bt : 1)), dim3(256), 0, s, out, n_txns, rank, a.ctl,
                     ns_per_tick_q16);
  return hipGetLastError();
}

}  // namespace cce
