// GPUTx (conflict-graph ordering by K-sets), a deterministic scheme.  The
// paper's description (Section 2, "Conflict Graph Ordering"): conflicts
// between transactions form a DAG ordered by transaction id; each
// transaction gets a rank from it, transactions of one rank (a K-set) run
// together without concurrency control, and the K-sets run in rank order.
// The rank here is the transaction's level in the DAG: one more than the
// largest rank among the earlier transactions it conflicts with (read-write,
// write-read, write-write on one item), 0 if none -- the rank that makes
// every K-set conflict-free.
//
// gfx950 design (preprocessing shared with GaccO, gacco.hip):
//  1. access table, radix sort by row, lock table: every row gets a turn
//     counter and every row access its place in the row's id-ordered list;
//  2. rank pass (gputx_rank_kernel): persistent teams take transactions in
//     id order; once every row of a transaction has come to it, the team
//     reads each row's state -- the largest rank of any earlier accessor and
//     the rank of the last earlier writer, both kept +1 in one 64-bit word --
//     takes the transaction's rank as the largest "one more than what it
//     conflicts with", updates the rows' states and passes the rows on;
//  3. execution: the chain scan in id order (chain.hip).  Conflicting
//     transactions are in different K-sets, the smaller id in the lower one,
//     so running the K-sets one after another gives every operation the value
//     that id order gives it; the rank is the outcome's serial key.
// Waiting in the rank pass is a state of the team in the persistent loop
// (never a spin) for transactions taken earlier by running wavefronts, so
// the smallest unfinished one can always proceed; a team that sees no
// progress for the wait limit stops the run (a safeguard, as for GaccO).
#include "opset.h"
#include "select.h"
#include "txn_kernel.h"

namespace cce {

__global__ void __launch_bounds__(64) gputx_reset_kernel(Ctl *ctl) {
  if (threadIdx.x == 0) ctl->queue = ctl->pending_n = 0;  // claim counters of the execution
}

__global__ void __launch_bounds__(256) gputx_fill_kernel(uint64_t *p, uint64_t n) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------------------
// rank pass
// ---------------------------------------------------------------------------
// Packed state (PACKED, batches of fewer than 2^20 transactions and 2^24
// operations): a row's word holds its turn and its state together --
// [63:40] sorted position whose turn it is, [39:20] largest rank + 1 of the
// row's accessors so far, [19:0] rank + 1 of its last writer.  The look that
// finds the turn brings the state with it, and one store passes the row on
// with its new state, so neither a separate load of the state nor an
// ordering point before the release is needed.  Otherwise the state lives in
// its own word (kstate) and the turn word holds sorted positions.
//
// What bounds the pass is the hottest row's list: passed from team to team, an
// access costs 1.5 us (the store, and the look that finds it).  So the packed
// form can resolve several at once (AHEAD).  A transaction that waits for one row only
// publishes, at its sorted position (a.known), the rank its other rows give it.
// A row's state after an access is a function of the state before and of that
// rank, so a waiting team that finds every position from the row's turn to its
// own published -- its lanes read the L before it along with the row's word --
// steps through them itself, leaves each the rank it found (GX_FINAL) and moves
// the row past its own.  Turns only grow, and a state belongs to its turn, so
// the word is moved by atomic max; a transaction that is overtaken takes its
// rank from its position.
// Measured, the run of 262,144 transactions x 16 ops, half writes, 10M rows, Zipf
// 0.6: 4.60 ms passed from team to team, 2.06 ms so.  Where a transaction mostly
// waits for several rows nothing is published in time, and the looks only make a
// hand-over longer (Zipf 0.9: the pass 46 ms, and 53 so): gputx_ahead chooses.
// (Ids claimed several at a time by a wavefront, or one ahead by a team, leave
// holes in the lists that every later team waits for: 2.04 and 2.51 ms, and at
// Zipf 0.9 178 ms against 117.)
constexpr uint32_t GX_KNOWN = 1u << 31, GX_FINAL = 1u << 30, GX_WRITE = 1u << 29;
constexpr uint64_t GX_M20 = (1ull << 20) - 1;

// One row group of `lead` is not in `granted`.
template <int NW>
__device__ __forceinline__ bool left_one(const OpSet<NW> &lead, const OpSet<NW> &granted) {
  int n = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) n += __popcll(lead.w[i] & ~granted.w[i]);
  return n == 1;
}

template <int L, int K, bool STRICT, bool PACKED, bool AHEAD>
__global__ void __launch_bounds__(MaxThreads<K>::value) gputx_rank_kernel(GputxArgs a) {
  constexpr int NW = L == 64 ? K : 1;
  static_assert(L == 64 || L * K <= 64, "operation sets of one word");
  using Set = OpSet<NW>;
  Team<L> t;
  int64_t txn = -1;
  bool finished = false;
  uint32_t rowk[K], rk[K];
  uint64_t gst[K];  // PACKED: the row's word as seen when its turn came
  // PACKED, team-uniform: 1 + the sorted position published (0: none), the lane
  // that waits there, whether it writes, and the rank + 1 published
  uint32_t pub = 0, pub_rank = 0;
  int pub_lane = 0;
  bool pub_wr = false;
  Set lead = Set::zero(), granted = Set::zero();
  uint64_t ready_at = 0, progress_at = 0;
  uint32_t idle_polls = 0;

  for (;;) {
    const bool need = txn < 0 && !finished;
    const uint64_t q = t.claim(&a.ctl->queue, need, 1);
    bool fresh = false;
    if (need) {
      if (q < a.n_txns && ld_word(&a.ctl->stop) == 0) {
        txn = (int64_t)q;
        fresh = true;
      } else {
        finished = true;
      }
    }
    if (ballot(txn >= 0) == 0) break;
    const uint64_t now = wall_clock64();
    if (ballot(fresh)) {
      uint32_t first = 0, n = 0;
      if (fresh) {
        const DevTxn d = a.txns[txn];
        first = d.first;
        n = d.n;
      }
      bool ld[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t idx = (uint32_t)t.tl + (uint32_t)(k * L);
        ld[k] = false;
        if (fresh && idx < n) {
          const uint32_t r = a.ops[first + idx].rowk;
          ld[k] = op_leader(r);
          if (ld[k]) {
            rowk[k] = r;
            rk[k] = a.rank[first + idx];
          }
        }
      }
      const Set sl = team_set<L, K, NW>(t, ld);
      if (fresh) {
        lead = sl;
        granted = Set::zero();
        pub = 0;
        ready_at = 0;
        progress_at = now;
        idle_polls = 0;
      }
    }
    const bool act = txn >= 0 && now >= ready_at;
    bool g[K];
    uint64_t ahead = ~0ull;
    uint64_t wait_w = 0;  // PACKED: the word of a row not yet come to this lane
    bool wait_wr = false, waits = false;
    uint32_t wait_at = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t i = (uint32_t)t.tl + (uint32_t)(k * L);
      g[k] = false;
      if (act && lead.test(i) && !granted.test(i)) {
        const uint64_t w = ld_word(a.words + op_row(rowk[k]));
        const uint64_t turn = PACKED ? (w >> 40) : w;
        g[k] = turn == (uint64_t)rk[k];
        if (PACKED && g[k]) gst[k] = w;
        if (PACKED && !g[k]) {
          wait_w = w;
          wait_wr = op_written(rowk[k]);
          wait_at = rk[k];
          waits = true;
        }
        if (!g[k] && (uint64_t)rk[k] > turn) {
          const uint64_t d = (uint64_t)rk[k] - turn;
          ahead = d < ahead ? d : ahead;
        }
      }
    }
    const Set newly = team_set<L, K, NW>(t, g);
    if (act) granted = granted | newly;
    // every row has come to the transaction: its rank, the rows' new states,
    // then the rows move on
    bool ready = act && granted == lead;
    if (PACKED) {
      // a position published before: the row may have been moved past it, or
      // every position from the row's turn on is known
      bool walked = false, overtaken = false;
      uint32_t any1 = 0, w1 = 0;
      const bool look = AHEAD && act && !ready && pub;
      if (ballot(look)) {
        const uint32_t at = pub - 1;
        uint32_t before = 0, mine = 0;
        if (look) {
          if (at + (uint32_t)t.tl >= (uint32_t)L) before = ld_u32(a.known + (at + (uint32_t)t.tl - (uint32_t)L));
          mine = ld_u32(a.known + at);
        }
        const uint32_t turn = (uint32_t)(wait_w >> 40);
        const uint32_t d = (uint32_t)__shfl((int)(waits && turn < wait_at ? wait_at - turn : 0u), pub_lane, 64);
        overtaken = look && (mine & GX_FINAL);
        const bool in = look && d && d <= (uint32_t)L && (uint32_t)t.tl + d >= (uint32_t)L;
        walked = look && !overtaken && d && d <= (uint32_t)L && !t.any(in && !(before & GX_KNOWN));
        if (ballot(walked)) {
          const uint64_t w = (uint64_t)__shfl((long long)wait_w, pub_lane, 64);
          any1 = (uint32_t)((w >> 20) & GX_M20);
          w1 = (uint32_t)(w & GX_M20);
          uint32_t found = 0;
          for (uint32_t s = 0; s < (uint32_t)L; ++s) {
            const bool step = walked && s + d >= (uint32_t)L;
            if (ballot(step) == 0) continue;
            const uint32_t e = (uint32_t)__shfl((int)before, t.tb + (int)s, 64);
            if (step) {
              const uint32_t c = ((e & GX_WRITE) ? any1 : w1) + 1, b = e & (uint32_t)GX_M20, r = c > b ? c : b;
              any1 = any1 > r ? any1 : r;
              if (e & GX_WRITE) w1 = r;
              if ((uint32_t)t.tl == s) found = r;
            }
          }
          if (walked && in && !(before & GX_FINAL))
            st_u32(a.known + (at + (uint32_t)t.tl - (uint32_t)L), (before & (GX_KNOWN | GX_WRITE)) | GX_FINAL | found);
        }
        if (overtaken) {
          pub_rank = mine & (uint32_t)GX_M20;
        } else if (walked) {
          const uint32_t c = (pub_wr ? any1 : w1) + 1;
          pub_rank = c > pub_rank ? c : pub_rank;
        }
      }
      // (a team with one row left has one lane that waits)
      const uint64_t waiting = ballot(waits) & t.tmask;
      const bool single = AHEAD && act && !ready && !pub && __popcll(waiting) == 1 && left_one<NW>(lead, granted);
      uint64_t r1 = 1;  // the transaction's rank + 1: at least 1, else the largest of these
      if (ballot(ready || single)) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const uint32_t i = (uint32_t)t.tl + (uint32_t)(k * L);
          if ((ready || single) && lead.test(i) && granted.test(i)) {
            const uint64_t c = (op_written(rowk[k]) ? (gst[k] >> 20) & GX_M20 : gst[k] & GX_M20) + 1;
            r1 = c > r1 ? c : r1;
          }
        }
        r1 = t.max(r1);
      }
      if (ballot(single)) {
        const int src = single ? __ffsll((unsigned long long)waiting) - 1 : t.lane;
        const uint32_t at = (uint32_t)__shfl((int)wait_at, src, 64);
        const bool wr = __shfl((int)wait_wr, src, 64) != 0;
        if (single) {
          if (t.lane == src) st_u32(a.known + at, GX_KNOWN | (wr ? GX_WRITE : 0u) | (uint32_t)r1);
          pub = at + 1;
          pub_rank = (uint32_t)r1;
          pub_lane = src;
          pub_wr = wr;
        }
      }
      if (walked || overtaken) r1 = pub_rank;
      ready |= walked || overtaken;
      if (ballot(ready)) {
        if (STRICT) order_point<STRICT>();
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const uint32_t i = (uint32_t)t.tl + (uint32_t)(k * L);
          if (ready && lead.test(i) && granted.test(i)) {
            const uint64_t a1 = (gst[k] >> 20) & GX_M20, b1 = gst[k] & GX_M20;
            const uint64_t nany = a1 > r1 ? a1 : r1;
            const uint64_t nw1 = op_written(rowk[k]) ? r1 : b1;
            const uint64_t next = (((uint64_t)rk[k] + 1) << 40) | (nany << 20) | nw1;
            uint64_t *word = a.words + op_row(rowk[k]);
            // (past a published position others move the row too)
            if (pub == rk[k] + 1) max_word(word, next);
            else st_word(word, next);
          } else if (walked && lead.test(i)) {
            const uint64_t nany = any1 > r1 ? any1 : r1, nw1 = pub_wr ? r1 : w1;
            max_word(a.words + op_row(rowk[k]), ((uint64_t)pub << 40) | (nany << 20) | nw1);
          }
        }
        if (ready && t.tl == 0) a.txn_rank[txn] = (uint32_t)(r1 - 1);
      }
    } else if (!PACKED && ballot(ready)) {
      if (STRICT) order_point<STRICT>();
      else asm volatile("" ::: "memory");
      uint64_t st[K];
      uint64_t r1 = 1;  // the transaction's rank + 1: at least 1, else the largest of these
#pragma unroll
      for (int k = 0; k < K; ++k) {
        st[k] = 0;
        if (ready && lead.test((uint32_t)t.tl + (uint32_t)(k * L))) {
          st[k] = ld_word(a.kstate + op_row(rowk[k]));
          const uint64_t c = op_written(rowk[k]) ? (st[k] >> 32) + 1 : (st[k] & 0xFFFFFFFFull) + 1;
          r1 = c > r1 ? c : r1;
        }
      }
      r1 = t.max(r1);  // rank + 1 (at least 1)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (ready && lead.test((uint32_t)t.tl + (uint32_t)(k * L))) {
          const uint64_t any1 = (st[k] >> 32) > r1 ? (st[k] >> 32) : r1;
          const uint64_t w1 = op_written(rowk[k]) ? r1 : (st[k] & 0xFFFFFFFFull);
          st_word(a.kstate + op_row(rowk[k]), (any1 << 32) | w1);
        }
      }
      order_point<STRICT>();  // the rows' states are performed before the rows move on
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (ready && lead.test((uint32_t)t.tl + (uint32_t)(k * L)))
          st_word(a.words + op_row(rowk[k]), (uint64_t)rk[k] + 1);
      if (ready && t.tl == 0) a.txn_rank[txn] = (uint32_t)(r1 - 1);
    }
    if (txn >= 0) {
      const uint64_t after = wall_clock64();
      if (ready) {
        txn = -1;
      } else if (act && !(newly == Set::zero())) {
        progress_at = after;
        idle_polls = 0;
      } else {
        const uint64_t m = ~t.max(~ahead);  // team minimum of `ahead`
        if (act) {
          // (within reach of a published position no nap)
          const uint64_t reach = AHEAD && pub ? (uint64_t)L : 1ull;
          if (m != ~0ull && m > reach) {
            const uint64_t cap = 4096ull * a.poll_ticks;
            const uint64_t nap = (m - reach) * a.poll_ticks;
            ready_at = after + (nap < cap ? nap : cap);
          }
          ++idle_polls;
        }
        if (after - progress_at > a.wait_limit_ticks) {
          st_word(&a.ctl->stop, 1);
          finished = true;
          txn = -1;
        } else if ((idle_polls & 255u) == 255u && ld_word(&a.ctl->stop) != 0) {
          finished = true;
          txn = -1;
        }
      }
    }
    if (ballot(act) == 0) __builtin_amdgcn_s_sleep(2);
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <int L, int K, bool STRICT>
static hipError_t gputx_launch_one(hipStream_t s, int waves_per_wg, int grid, const GputxArgs &a, int n_cu,
                                   int *grid_used) {
  const int block = 64 * waves_per_wg;
  if (block > MaxThreads<K>::value) return hipErrorInvalidConfiguration;
  if (grid <= 0) grid = n_cu;  // one workgroup per compute unit
  const uint64_t teams_per_wg = (uint64_t)waves_per_wg * (64 / L);
  const uint64_t need = (a.n_txns + teams_per_wg - 1) / teams_per_wg;
  if ((uint64_t)grid > need) grid = (int)(need > 0 ? need : 1);
  *grid_used = grid;
  if (a.known)
    hipLaunchKernelGGL((gputx_rank_kernel<L, K, STRICT, true, true>), dim3(grid), dim3(block), 0, s, a);
  else if (a.packed)
    hipLaunchKernelGGL((gputx_rank_kernel<L, K, STRICT, true, false>), dim3(grid), dim3(block), 0, s, a);
  else
    hipLaunchKernelGGL((gputx_rank_kernel<L, K, STRICT, false, false>), dim3(grid), dim3(block), 0, s, a);
  return hipGetLastError();
}

template <bool STRICT>
static hipError_t gputx_dispatch(hipStream_t s, int lanes, int max_ops, int waves_per_wg, int grid,
                                 const GputxArgs &a, int n_cu, int *grid_used) {
  const int need_k = (max_ops + lanes - 1) / lanes;
#define CCE_TRY(LL, KK)             \
  if (lanes == LL && need_k <= KK) \
    return gputx_launch_one<LL, KK, STRICT>(s, waves_per_wg, grid, a, n_cu, grid_used);
  CCE_TRY(1, 4)
  CCE_TRY(1, 16)
  CCE_TRY(4, 4)
  CCE_TRY(4, 16)
  CCE_TRY(16, 1)
  CCE_TRY(16, 4)
  CCE_TRY(64, 1)
  CCE_TRY(64, 4)
#undef CCE_TRY
  return hipErrorInvalidValue;
}

hipError_t launch_gputx_rank(hipStream_t s, int lanes, int max_ops, int waves_per_wg, int grid, bool strict,
                             const GputxArgs &a, int n_cu, int *grid_used) {
  return strict ? gputx_dispatch<true>(s, lanes, max_ops, waves_per_wg, grid, a, n_cu, grid_used)
                : gputx_dispatch<false>(s, lanes, max_ops, waves_per_wg, grid, a, n_cu, grid_used);
}

hipError_t gputx_init_state(hipStream_t s, uint64_t *kstate, uint64_t n_rows) {
  const uint64_t blocks = (n_rows + 255) / 256;
  if (blocks) hipLaunchKernelGGL(gputx_fill_kernel, dim3((unsigned)blocks), dim3(256), 0, s, kstate, n_rows);
  return hipGetLastError();
}

hipError_t gputx_reset(hipStream_t s, Ctl *ctl) {
  hipLaunchKernelGGL(gputx_reset_kernel, dim3(1), dim3(64), 0, s, ctl);
  return hipGetLastError();
}

}  // namespace cce
