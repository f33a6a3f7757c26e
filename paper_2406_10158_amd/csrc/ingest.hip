// Batch submission on the device: validate a batch's transactions and
// operations, pack them into the engine's descriptors, and find the rows the
// batch writes most.  Batches arrive in device memory, or are copied there
// first.  The rules and status codes are cc_check_batch's (api.cpp,
// validate_and_pack), in the same order: per transaction, the first failing
// check in program order; over the batch, the lowest-numbered malformed
// transaction.
//
//   ingest_headers  whether the transactions' operations follow one another
//                   without gaps, as they mostly do; then no operation can
//                   belong to two transactions or to none, and the next two
//                   kernels have nothing to do:
//   ingest_fill     default descriptors (gaps) and the per-op owner;
//   ingest_claim    each transaction records itself as an owner of its ops
//                   (atomic minimum), so that an op named by two
//                   transactions is reported at the later one;
//   ingest_pack     16 lanes per transaction check and pack its ops, 16 at a
//                   time: row groups from ballots, repeated rows by comparing
//                   every two leaders through lane shuffles.  Each written
//                   row access is counted per row, in an LDS cache first (the
//                   hot rows' counts would otherwise serialise on one word);
//                   the op that counts a row first is marked with it (a common
//                   list of the rows would serialise on its length: 65,000
//                   appends took 1.5 ms);
//   plan_counts, plan_ties, plan_pick
//                   the PLAN_CAND most written of the marked rows (ties: lower
//                   row first) by a histogram of the counts, one of the rows
//                   at the cut, and a sort of what is left; the counts go back
//                   to zero for the next batch.
// A batch of at most INGEST_LOCAL ops in a quarter as many transactions is done
// in one workgroup, with the counts in LDS.
//
// What bounds it: reading 16 bytes and writing 16 bytes per op, and one
// random atomic per distinct written row of a workgroup's share.  A thread per
// transaction, each loading its 16-byte ops one after another, took 1.67 ms
// for 2^18 transactions x 16 ops, and the rows' counts were made on the host,
// over every row of the tables: 40 ms more there, and 36 ms for 2^14 uneven
// transactions (540k ops) from the host.  Now 0.46 ms for the whole submission
// of 2^18 x 16 device-resident ops (pack 0.30, counts 0.10, pick 0.07) and
// 0.43 ms for the uneven host batch; 30 us of kernel for 256 transactions x 4.
#include "select.h"

namespace cce {

namespace {

constexpr int IG_L = 16;  // lanes per transaction

// error word: (transaction << 16) | (message << 4) | code, minimum wins
__device__ __forceinline__ void report(const IngestArgs &a, uint64_t t, uint32_t msg, uint32_t code) {
  atomicMin((unsigned long long *)&a.out[INGEST_ERR], (unsigned long long)((t << 16) | (msg << 4) | code));
}

__device__ __forceinline__ bool header_ok(const IngestArgs &a, const cc_txn &x, uint32_t *msg) {
  if (x.reserved != 0) { *msg = INGEST_MSG_RESERVED; return false; }
  if (x.n_ops > CC_MAX_OPS_PER_TXN) { *msg = INGEST_MSG_TOO_MANY; return false; }
  if (x.first_op > a.n_ops || x.n_ops > a.n_ops - x.first_op) { *msg = INGEST_MSG_OP_RANGE; return false; }
  return true;
}

__device__ __forceinline__ uint32_t msg_code(uint32_t msg) {
  if (msg == INGEST_MSG_TABLE || msg == INGEST_MSG_ROW_FIELD) return (uint32_t)-CC_E_RANGE;
  if (msg == INGEST_MSG_DUP_FIELD || msg == INGEST_MSG_DUP_ROW) return (uint32_t)-CC_E_DUPROW;
  return (uint32_t)-CC_E_INVAL;
}

// ---- the parts, over a grid of nb workgroups of nt threads -----------------

__device__ __forceinline__ void part_reset(const IngestArgs &a, uint32_t tid, uint32_t nthr) {
  for (uint32_t i = tid; i < (uint32_t)INGEST_N; i += nthr) a.out[i] = i == INGEST_ERR ? ~0ull : 0ull;
  if (a.hist)
    for (uint32_t i = tid; i < (uint32_t)(PLAN_COUNTS + PLAN_BINS); i += nthr) a.hist[i] = 0;
}

// Whether a thread's share of the transactions is loose.
__device__ __forceinline__ bool part_headers(const IngestArgs &a, uint64_t tid, uint64_t nthr) {
  bool loose = tid == 0 && a.n_txns == 0 && a.n_ops;
  for (uint64_t t = tid; t < a.n_txns; t += nthr) {
    const cc_txn x = a.txns[t];
    uint32_t msg = 0;
    uint64_t at = 0;  // where the transaction's ops have to begin
    if (t) {
      const cc_txn y = a.txns[t - 1];
      at = y.first_op + y.n_ops;
    }
    loose |= !header_ok(a, x, &msg) || x.first_op != at;
    if (t + 1 == a.n_txns) loose |= x.first_op + x.n_ops != a.n_ops;
  }
  return loose;
}

__device__ __forceinline__ void part_fill(const IngestArgs &a, uint64_t tid, uint64_t nthr) {
  for (uint64_t i = tid; i < a.n_ops; i += nthr) {
    DevOp d;
    d.rowk = GAP_OP;
    d.elem = 0;
    d.arg = 0;
    a.dops[i] = d;
    a.owner[i] = 0xFFFFFFFFu;
    if (a.cnt) a.rows[i] = 0xFFFFFFFFu;
    if (a.meta) {
      a.meta[i] = 0;
      a.rows0[i] = a.ops[i].row;
    }
  }
}

__device__ __forceinline__ void part_claim(const IngestArgs &a, uint64_t tid, uint64_t nthr) {
  for (uint64_t g = tid / IG_L; g < a.n_txns; g += nthr / IG_L) {
    const cc_txn x = a.txns[g];
    uint32_t msg = 0;
    if (!header_ok(a, x, &msg)) continue;
    for (uint32_t i = (uint32_t)(tid % IG_L); i < x.n_ops; i += IG_L) atomicMin(&a.owner[x.first_op + i], (uint32_t)g);
  }
}

// A transaction's ops as bit sets (bit i: op i).
struct OpBits {
  uint64_t lead[4], write[4];
};

// Whether a row group writes its row, for the group op i is in.
__device__ __forceinline__ bool group_writes(const OpBits &s, uint32_t i) {
  const int b = (int)(i & 63u);
  uint64_t hit = 0;
  int w = (int)(i >> 6);
  uint64_t m = b == 63 ? ~0ull : (1ull << (b + 1)) - 1ull;
  for (;;) {  // from op i down to its group's leader
    const uint64_t l = s.lead[w] & m;
    if (l) {
      hit |= s.write[w] & m & ~((1ull << (63 - __clzll((long long)l))) - 1ull);
      break;
    }
    hit |= s.write[w] & m;
    if (w == 0) break;
    --w;
    m = ~0ull;
  }
  w = (int)(i >> 6);
  m = b == 63 ? 0ull : ~0ull << (b + 1);
  for (;;) {  // up to the next leader
    const uint64_t l = s.lead[w] & m;
    if (l) {
      hit |= s.write[w] & m & ((l & -l) - 1ull);
      break;
    }
    hit |= s.write[w] & m;
    if (++w == 4) break;
    m = ~0ull;
  }
  return hit != 0;
}

__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Row counts in LDS.  A cache in front of the counts in memory: a row that
// finds its slot taken is counted there.  A batch of at most INGEST_LOCAL ops
// has half as many rows as a table of twice the slots, which then holds every
// count itself (LOCAL).
constexpr uint32_t RC_NONE = 0xFFFFFFFFu;  // (row ids have 28 bits)
template <bool LOCAL>
constexpr uint32_t rc_slots = LOCAL ? 2 * INGEST_LOCAL : 2048;

template <int NT, bool LOCAL>
struct PackLds {
  OpBits bits[NT / IG_L];
  IngestTable tab[CC_MAX_TABLES];  // (indexed by an op's table, the kernel's arguments would be read from memory)
  uint32_t row[rc_slots<LOCAL>], cnt[rc_slots<LOCAL>], op[LOCAL ? 1 : rc_slots<LOCAL>];
};

// Checks and packs the transactions; block b of nb, NT threads.
template <int NT, bool LOCAL>
__device__ __forceinline__ void part_pack(const IngestArgs &a, PackLds<NT, LOCAL> &s, bool loose, uint32_t b,
                                          uint32_t nb) {
  constexpr uint32_t RC_SLOTS = rc_slots<LOCAL>;
  constexpr uint32_t TEAMS = NT / IG_L;
  const uint32_t tid = threadIdx.x, team = tid / IG_L, tl = tid % IG_L;
  const int lane = __lane_id(), tb = lane - (int)tl;
  if (tid < (uint32_t)CC_MAX_TABLES) s.tab[tid] = a.tab[tid];
  if (a.cnt)
    for (uint32_t i = tid; i < RC_SLOTS; i += NT) {
      s.row[i] = RC_NONE;
      s.cnt[i] = 0;
    }
  __syncthreads();
  // tables whose ops name their rows by key (bit t: table t)
  uint32_t indexed = 0;
  if (a.op_keys)
    for (uint32_t t = 0; t < a.n_tables; ++t) indexed |= a.tab[t].indexed ? 1u << t : 0u;
  static_assert(CC_MAX_TABLES <= 32, "a bit per table");
  auto is_keyed = [&](const cc_op &o) { return o.table < 32u && ((indexed >> o.table) & 1u); };
  uint32_t max_ops = 0, kinds = 0;
  bool unordered = false, any_keyed = false;
  OpBits &bits = s.bits[team];
  const uint64_t step = (uint64_t)nb * TEAMS;
  cc_txn ahead{0, 0, 0};  // the next transaction's header, on its way while this one is worked on
  if ((uint64_t)b * TEAMS + team < a.n_txns) ahead = a.txns[(uint64_t)b * TEAMS + team];
  for (uint64_t t0 = (uint64_t)b * TEAMS; t0 < a.n_txns; t0 += step) {
    const uint64_t t = t0 + team;
    const cc_txn x = ahead;
    uint32_t hmsg = 0;
    bool live = t < a.n_txns;
    if (t + step < a.n_txns) ahead = a.txns[t + step];
    if (live) {
      if (!header_ok(a, x, &hmsg)) {
        if (tl == 0) report(a, t, hmsg, (uint32_t)-CC_E_INVAL);
        live = false;
      } else if (tl == 0 && t > 0) {
        unordered |= x.first_op < a.txns[t - 1].first_op;
      }
    }
    const uint32_t n = live ? x.n_ops : 0u;
    const uint64_t f0 = x.first_op;
    uint32_t longest = n;  // of this wavefront's transactions
#pragma unroll
    for (int o = IG_L; o < 64; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_xor((int)longest, o, 64);
      longest = y > longest ? y : longest;
    }
    const uint32_t chunks = (longest + IG_L - 1) / IG_L;
    // an op and its row's identity: its key on an indexed table (keyed batch), else its row
    // (the key is loaded with the op, keyed or not, and selected afterwards)
    auto load = [&](uint32_t i, cc_op *o, int64_t *id) {
      *o = cc_op{0, 0, 0, 0, 0};
      int64_t key = 0;
      if (i < n) {
        *o = a.ops[f0 + i];
        if (indexed) key = a.op_keys[f0 + i];
      }
      *id = is_keyed(*o) ? key : (int64_t)o->row;
    };
    if (tl < 4) bits.lead[tl] = bits.write[tl] = 0;
    wave_lds_order();
    uint32_t err = 0xFFFFFFFFu;  // op << 8 | message, the first op's
    bool shared = false;
    uint32_t ptab = 0;
    int64_t pid = 0;
    cc_op o0{};   // the first 16 ops stay in registers
    int64_t id0 = 0;
    for (uint32_t c = 0; c < chunks; ++c) {
      const uint32_t i = c * IG_L + tl;
      cc_op o;
      int64_t id;
      load(i, &o, &id);
      if (c == 0) {
        o0 = o;
        id0 = id;
      }
      const bool in = i < n;
      if (loose && in) shared |= a.owner[f0 + i] != (uint32_t)t;
      // the op before: the lane below, or the last lane's op of the chunk before
      const uint32_t utab = (uint32_t)__shfl_up((int)(uint32_t)o.table, 1, 64);
      const int64_t uid = __shfl_up((long long)id, 1, 64);
      const uint32_t qtab = tl ? utab : ptab;
      const int64_t qid = tl ? uid : pid;
      ptab = (uint32_t)__shfl((int)(uint32_t)o.table, tb + IG_L - 1, 64);
      pid = __shfl((long long)id, tb + IG_L - 1, 64);
      const bool follower = in && i > 0 && qtab == o.table && qid == id;
      const uint32_t lead16 = (uint32_t)(ballot(in && !follower) >> tb) & 0xFFFFu;
      const uint32_t write16 = (uint32_t)(ballot(in && o.kind != CC_READ) >> tb) & 0xFFFFu;
      if (tl == 0 && n > c * IG_L) {
        bits.lead[c >> 2] |= (uint64_t)lead16 << (16 * (c & 3));
        bits.write[c >> 2] |= (uint64_t)write16 << (16 * (c & 3));
      }
      wave_lds_order();
      if (in) {
        uint32_t msg = 0;
        if (o.table >= a.n_tables) {
          msg = INGEST_MSG_TABLE;
        } else {
          const IngestTable &tb_ = s.tab[o.table];
          const bool kd = is_keyed(o);
          any_keyed |= kd;
          if (kd && o.row != 0) msg = INGEST_MSG_KEYED_ROW;
          else if ((!kd && o.row >= tb_.n_rows) || o.field >= tb_.n_fields) msg = INGEST_MSG_ROW_FIELD;
          else if (o.kind > CC_WRITE_SLOT) msg = INGEST_MSG_KIND;
          else if (o.kind == CC_WRITE_SLOT && (uint32_t)(o.arg & 0xFF) >= i) msg = INGEST_MSG_SLOT_SRC;
        }
        kinds |= (o.kind == CC_WRITE_SLOT ? 1u : 0u) | (o.kind == CC_COND_ADD ? 2u : 0u);
        if (msg == 0 && follower) {
          for (uint32_t j = i; j-- > 0;) {
            if (a.ops[f0 + j].field == o.field) msg = INGEST_MSG_DUP_FIELD;
            if (msg || ((bits.lead[j >> 6] >> (j & 63)) & 1u)) break;
          }
        }
        if (msg) {
          const uint32_t e = (i << 8) | msg;
          err = e < err ? e : err;
        }
      }
    }
    // a (table, row) may start only one row group
    bool dup = false;
    for (uint32_t c = 0; c < chunks; ++c) {
      const uint32_t i = c * IG_L + tl;
      cc_op o = o0;
      int64_t id = id0;
      if (c) load(i, &o, &id);
      const bool lead = i < n && ((bits.lead[i >> 6] >> (i & 63)) & 1u);
      for (uint32_t d = 0; d <= c; ++d) {
        cc_op q = o0;
        int64_t qid = id0;
        if (d == c) {
          q = o;
          qid = id;
        } else if (d) {
          load(d * IG_L + tl, &q, &qid);
        }
        const uint32_t j0 = d * IG_L;
        const uint32_t qlead = (uint32_t)(bits.lead[j0 >> 6] >> (j0 & 63)) & 0xFFFFu;
        const uint32_t most = longest - j0 < (uint32_t)IG_L ? longest - j0 : (uint32_t)IG_L;
        for (uint32_t k = 0; k < most; ++k) {
          const uint32_t jt = (uint32_t)__shfl((int)(uint32_t)q.table, tb + (int)k, 64);
          const int64_t ji = __shfl((long long)qid, tb + (int)k, 64);
          dup |= lead && j0 + k < i && ((qlead >> k) & 1u) && jt == o.table && ji == id;
        }
      }
    }
    // the transaction's first error in the order of the checks
#pragma unroll
    for (int o = 1; o < IG_L; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_xor((int)err, o, 64);
      err = y < err ? y : err;
    }
    const uint64_t tmask = 0xFFFFull << tb;
    const bool any_shared = (ballot(shared) & tmask) != 0, any_dup = (ballot(dup) & tmask) != 0;
    uint32_t msg = any_shared ? (uint32_t)INGEST_MSG_SHARED
                              : (err != 0xFFFFFFFFu ? (err & 0xFFu) : (any_dup ? (uint32_t)INGEST_MSG_DUP_ROW : 0u));
    if (live && msg && tl == 0) report(a, t, msg, msg_code(msg));
    const bool good = live && !msg;
    // the descriptors, and a count for every written row
    for (uint32_t c = 0; c < chunks; ++c) {
      const uint32_t i = c * IG_L + tl;
      cc_op o = o0;
      int64_t id = id0;
      if (c) load(i, &o, &id);
      const bool in = good && i < n;
      uint32_t mark = RC_NONE;
      if (in) {
        const IngestTable &tb_ = s.tab[o.table];
        const bool kd = is_keyed(o);
        const bool lead = (bits.lead[i >> 6] >> (i & 63)) & 1u, wr = group_writes(bits, i);
        const uint32_t grow = kd ? 0u : (uint32_t)(tb_.row_base + o.row);
        DevOp d;
        d.rowk = grow | ((uint32_t)o.kind << KIND_SHIFT) | (lead ? 0u : FOLLOWER_BIT) | (wr ? WRITTEN_BIT : 0u);
        d.elem = kd ? 0u : (uint32_t)(tb_.elem_base + (uint64_t)o.row * tb_.n_fields + o.field);
        d.arg = o.arg;
        a.dops[f0 + i] = d;
        if (a.cnt && lead && wr && !kd) {
          uint32_t h = (grow * 0x9E3779B1u) >> (LOCAL ? 20 : 21);
          static_assert(RC_SLOTS == 1u << (LOCAL ? 12 : 11), "hash to the slots");
          uint32_t seen = atomicCAS(&s.row[h], RC_NONE, grow);
          if constexpr (LOCAL) {
            while (seen != RC_NONE && seen != grow) {  // there are more slots than ops
              h = (h + 1) & (RC_SLOTS - 1);
              seen = atomicCAS(&s.row[h], RC_NONE, grow);
            }
            atomicAdd(&s.cnt[h], 1u);
          } else {
            if (seen == RC_NONE) s.op[h] = (uint32_t)f0 + i;
            if (seen == RC_NONE || seen == grow) atomicAdd(&s.cnt[h], 1u);
            else if (atomicAdd(&a.cnt[grow], 1u) == 0) mark = grow;
          }
        }
        if (a.meta) {
          a.meta[f0 + i] = kd ? META_KEYED | ((uint32_t)o.table << 16) | o.field : 0u;
          a.rows0[f0 + i] = o.row;
        }
      }
      if (!LOCAL && a.cnt && i < n) a.rows[f0 + i] = mark;  // (an op of a malformed transaction: none)
    }
    if (good && tl == 0) a.dtx[t] = DevTxn{(uint32_t)f0, n};
    max_ops = n > max_ops ? n : max_ops;
    wave_lds_order();  // the bits are reused by the next transaction
  }
  __syncthreads();
  if (!LOCAL && a.cnt)
    for (uint32_t i = tid; i < RC_SLOTS; i += NT)
      if (s.cnt[i] && atomicAdd(&a.cnt[s.row[i]], s.cnt[i]) == 0) a.rows[s.op[i]] = s.row[i];
  max_ops = (uint32_t)wave_max(max_ops);
  const uint64_t w_slot = ballot(kinds & 1u), w_cond = ballot(kinds & 2u), w_unord = ballot(unordered),
                 w_keyed = ballot(any_keyed);
  if (lane == 0) {
    if (max_ops) atomicMax((unsigned long long *)&a.out[INGEST_MAX_OPS], (unsigned long long)max_ops);
    if (w_slot || w_cond)
      atomicOr((unsigned long long *)&a.out[INGEST_KINDS], (w_slot ? 1ull : 0ull) | (w_cond ? 2ull : 0ull));
    if (w_unord) atomicOr((unsigned long long *)&a.out[INGEST_UNORDERED], 1ull);
    if (w_keyed) atomicOr((unsigned long long *)&a.out[INGEST_KEYED], 1ull);
  }
}

// ---- the most written rows ---------------------------------------------------

__device__ __forceinline__ uint32_t count_bin(uint32_t c) { return c < (uint32_t)PLAN_COUNTS ? c : (uint32_t)PLAN_COUNTS - 1; }

// A marked row's candidate key, larger for more writes, then for the lower
// row; 0: not marked.
__device__ __forceinline__ uint64_t plan_key(uint32_t row, uint32_t c) { return ((uint64_t)c << 32) | (uint32_t)~row; }
__device__ __forceinline__ uint32_t key_row(uint64_t k) { return ~(uint32_t)k; }

// A workgroup's largest count and its sums of c (c - 1) and of c into out[0], [1]
// and [2], by one thread: atomics of every wavefront on the same words took 10 us
// a word with 8,192 of them.
template <int NT>
__device__ __forceinline__ void add_counts(uint64_t *out, uint32_t top, uint64_t pairs, uint64_t writes) {
  __shared__ uint64_t part[3 * (NT / 64)];
  const int w = threadIdx.x / 64;
  top = (uint32_t)wave_max(top);
  pairs = wave_sum(pairs);
  writes = wave_sum(writes);
  if (__lane_id() == 0) {
    part[3 * w] = top;
    part[3 * w + 1] = pairs;
    part[3 * w + 2] = writes;
  }
  __syncthreads();
  if (threadIdx.x) return;
  for (int i = 1; i < NT / 64; ++i) {
    top = (uint32_t)part[3 * i] > top ? (uint32_t)part[3 * i] : top;
    pairs += part[3 * i + 1];
    writes += part[3 * i + 2];
  }
  if (!writes) return;
  atomicMax((unsigned long long *)&out[0], (unsigned long long)top);
  if (pairs) add_word(&out[1], pairs);
  add_word(&out[2], writes);
}
static_assert(INGEST_PAIRS == INGEST_TOP + 1 && INGEST_WRITES == INGEST_TOP + 2, "the counts' results");

// Four ops a thread and step, so that four rows' counts are on their way at once.
constexpr int PLAN_STEP = 4;

// Every marked row's count becomes its key and goes back to zero; histogram of
// the counts (PLAN_COUNTS - 1 and more in the last bin).  The last workgroup
// finds the cut: the lowest count that a candidate can have, and how many rows
// are above it.
template <int NT>
__device__ __forceinline__ void part_counts(const IngestArgs &a, uint32_t *lds, uint32_t b, uint32_t nb) {
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i < (uint32_t)PLAN_COUNTS; i += NT) lds[i] = 0;
  __syncthreads();
  uint32_t top = 0;
  uint64_t pairs = 0, writes = 0;
  for (uint64_t i0 = (uint64_t)b * NT * PLAN_STEP; i0 < a.n_ops; i0 += (uint64_t)nb * NT * PLAN_STEP) {
    uint32_t row[PLAN_STEP], c[PLAN_STEP];
#pragma unroll
    for (int j = 0; j < PLAN_STEP; ++j) {
      const uint64_t i = i0 + (uint64_t)j * NT + tid;
      row[j] = i < a.n_ops ? a.rows[i] : RC_NONE;
    }
#pragma unroll
    for (int j = 0; j < PLAN_STEP; ++j) c[j] = row[j] != RC_NONE ? ld_u32(a.cnt + row[j]) : 0u;
#pragma unroll
    for (int j = 0; j < PLAN_STEP; ++j) {
      const uint64_t i = i0 + (uint64_t)j * NT + tid;
      if (row[j] != RC_NONE) {
        a.cnt[row[j]] = 0;
        pairs += (uint64_t)c[j] * (c[j] - 1);
        writes += c[j];
        if (a.hot_map && c[j] > 1) atomicOr(&a.hot_map[row[j] >> 5], 1u << (row[j] & 31));
        atomicAdd(&lds[count_bin(c[j])], 1u);
        top = c[j] > top ? c[j] : top;
      }
      if (i < a.n_ops) a.keys[i] = row[j] != RC_NONE ? plan_key(row[j], c[j]) : 0ull;
    }
  }
  __syncthreads();
  for (uint32_t i = tid; i < (uint32_t)PLAN_COUNTS; i += NT)
    if (lds[i]) atomicAdd(&a.hist[i], lds[i]);
  add_counts<NT>(&a.out[INGEST_TOP], top, pairs, writes);
  if (!last_block(&a.out[INGEST_DONE1], nb)) return;
  if (tid < 64) {
    uint32_t cut = 0;
    uint64_t above = 0;
    find_bin(a.hist, PLAN_COUNTS, true, PLAN_CAND, &cut, &above);
    if (tid == 0) {
      a.out[INGEST_CUT] = cut;
      a.out[INGEST_ABOVE] = above;
      // many rows at the cut (the last bin holds different counts: all are candidates)
      a.out[INGEST_TIES] = cut + 1 < (uint32_t)PLAN_COUNTS && ld_u32(a.hist + cut) > (uint32_t)PLAN_SORT / 2 ? 1 : 0;
      a.out[INGEST_ROW_CUT] = PLAN_BINS - 1;
    }
  }
}

// Many rows share the lowest count: a histogram of the rows themselves, and
// the bin up to which they are candidates (lower rows first).
template <int NT>
__device__ __forceinline__ void part_ties(const IngestArgs &a, uint32_t *lds, uint32_t b, uint32_t nb) {
  if (!ld_word(&a.out[INGEST_TIES])) return;  // every workgroup alike
  const uint32_t cut = (uint32_t)ld_word(&a.out[INGEST_CUT]), tid = threadIdx.x;
  for (uint32_t i = tid; i < (uint32_t)PLAN_BINS; i += NT) lds[i] = 0;
  __syncthreads();
  for (uint64_t i = (uint64_t)b * NT + tid; i < a.n_ops; i += (uint64_t)nb * NT) {
    const uint64_t k = a.keys[i];
    if ((uint32_t)(k >> 32) == cut && k) atomicAdd(&lds[key_row(k) >> a.row_shift], 1u);
  }
  __syncthreads();
  uint32_t *h = a.hist + PLAN_COUNTS;
  for (uint32_t i = tid; i < (uint32_t)PLAN_BINS; i += NT)
    if (lds[i]) atomicAdd(&h[i], lds[i]);
  if (!last_block(&a.out[INGEST_DONE2], nb)) return;
  if (tid < 64) {
    uint32_t bin = 0;
    uint64_t before = 0;
    find_bin(h, PLAN_BINS, false, PLAN_CAND - ld_word(&a.out[INGEST_ABOVE]), &bin, &before);
    if (tid == 0) a.out[INGEST_ROW_CUT] = bin;
  }
}

// Sorts n keys in LDS (at most PLAN_SORT), largest first, and reports the
// first PLAN_CAND.
template <int NT>
__device__ __forceinline__ void sort_candidates(const IngestArgs &a, uint64_t *lds, uint32_t n) {
  const uint32_t tid = threadIdx.x;
  if (n <= (uint32_t)PLAN_SORT / 2) {
    // few: a key's place is the number of larger ones (no two are equal)
    __syncthreads();
    if (tid >= n && tid < (uint32_t)PLAN_CAND) a.out[INGEST_CAND + tid] = 0;
    for (uint32_t i = tid; i < n; i += NT) {
      const uint64_t k = lds[i];
      uint32_t at = 0;
      for (uint32_t j = 0; j < n; ++j) at += lds[j] > k;
      if (at < (uint32_t)PLAN_CAND) a.out[INGEST_CAND + at] = k;
    }
    return;
  }
  uint32_t w = 64;
  while (w < n) w <<= 1;
  for (uint32_t i = n + tid; i < w; i += NT) lds[i] = 0;
  for (uint32_t k = 2; k <= w; k <<= 1)  // bitonic
    for (uint32_t j = k >> 1; j > 0; j >>= 1) {
      __syncthreads();
      for (uint32_t i = tid; i < w; i += NT) {
        const uint32_t o = i ^ j;
        if (o > i) {
          const uint64_t x = lds[i], y = lds[o];
          if (((i & k) == 0) == (x < y)) {
            lds[i] = y;
            lds[o] = x;
          }
        }
      }
    }
  __syncthreads();
  if (tid < (uint32_t)PLAN_CAND) a.out[INGEST_CAND + tid] = lds[tid];
}

// Candidates gathered; the last workgroup sorts them.
template <int NT>
__device__ __forceinline__ void part_pick(const IngestArgs &a, uint64_t *lds, uint32_t b, uint32_t nb) {
  const uint32_t cut = (uint32_t)ld_word(&a.out[INGEST_CUT]), row_cut = (uint32_t)ld_word(&a.out[INGEST_ROW_CUT]);
  const uint32_t tid = threadIdx.x;
  for (uint64_t i0 = (uint64_t)b * NT; i0 < a.n_ops; i0 += (uint64_t)nb * NT) {
    const uint64_t i = i0 + tid;
    const uint64_t key = i < a.n_ops ? a.keys[i] : 0ull;
    const uint32_t bin = count_bin((uint32_t)(key >> 32));
    const bool p = key && (bin > cut || (bin == cut && (key_row(key) >> a.row_shift) <= row_cut));
    const uint64_t mask = ballot(p);
    if (mask) {
      const int first = __ffsll((unsigned long long)mask) - 1, lane = __lane_id();
      uint64_t at = 0;
      if (lane == first) at = add_word(&a.out[INGEST_N_CAND], (uint64_t)__popcll(mask));
      at = readlane64(at, first) + (uint64_t)__popcll(mask & ((1ull << lane) - 1ull));
      if (p && at < plan_cand_max(a.n_ops)) st_word(a.cand + at, key);
    }
  }
  if (!last_block(&a.out[INGEST_DONE3], nb)) return;
  const uint64_t n = ld_word(&a.out[INGEST_N_CAND]);
  if (n <= (uint64_t)PLAN_SORT) {
    for (uint32_t i = tid; i < (uint32_t)n; i += NT) lds[i] = ld_word(a.cand + i);
    sort_candidates<NT>(a, lds, (uint32_t)n);
    return;
  }
  // more than fit (rows written PLAN_COUNTS times and more): the largest, time
  // after time; a thread looks through its share again when its own was taken
  uint64_t mine = 0;
  for (uint64_t i = tid; i < n; i += NT) {
    const uint64_t k = ld_word(a.cand + i);
    mine = k > mine ? k : mine;
  }
  for (int r = 0; r < PLAN_CAND; ++r) {
    const uint64_t w = wave_max(mine);
    __syncthreads();
    if (__lane_id() == 0) lds[tid / 64] = w;
    __syncthreads();
    uint64_t best = 0;
    for (int i = 0; i < NT / 64; ++i) best = lds[i] > best ? lds[i] : best;
    if (tid == 0) a.out[INGEST_CAND + r] = best;
    if (best && mine == best) {
      mine = 0;
      for (uint64_t i = tid; i < n; i += NT) {
        const uint64_t k = ld_word(a.cand + i);
        if (k < best && k > mine) mine = k;
      }
    }
  }
}

constexpr int PLAN_LDS_WORDS = PLAN_BINS;  // 32-bit words; PLAN_SORT 64-bit keys fit too
static_assert(PLAN_COUNTS <= PLAN_BINS && 2 * PLAN_SORT <= PLAN_LDS_WORDS, "plan scratch in LDS");

}  // namespace

__global__ void __launch_bounds__(256) ingest_reset_kernel(IngestArgs a) { part_reset(a, threadIdx.x, 256); }

__global__ void __launch_bounds__(256) ingest_headers_kernel(IngestArgs a) {
  if (part_headers(a, (uint64_t)blockIdx.x * 256 + threadIdx.x, (uint64_t)gridDim.x * 256) &&
      ld_word(&a.out[INGEST_LOOSE]) == 0)
    atomicOr((unsigned long long *)&a.out[INGEST_LOOSE], 1ull);
}
__global__ void __launch_bounds__(256) ingest_fill_kernel(IngestArgs a) {
  if (!ld_word(&a.out[INGEST_LOOSE])) return;
  part_fill(a, (uint64_t)blockIdx.x * 256 + threadIdx.x, (uint64_t)gridDim.x * 256);
}
__global__ void __launch_bounds__(256) ingest_claim_kernel(IngestArgs a) {
  if (!ld_word(&a.out[INGEST_LOOSE])) return;
  part_claim(a, (uint64_t)blockIdx.x * 256 + threadIdx.x, (uint64_t)gridDim.x * 256);
}
__global__ void __launch_bounds__(256) ingest_pack_kernel(IngestArgs a) {
  __shared__ PackLds<256, false> s;
  part_pack<256, false>(a, s, ld_word(&a.out[INGEST_LOOSE]) != 0, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(256) plan_counts_kernel(IngestArgs a) {
  __shared__ uint32_t lds[PLAN_LDS_WORDS];
  part_counts<256>(a, lds, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(256) plan_ties_kernel(IngestArgs a) {
  __shared__ uint32_t lds[PLAN_LDS_WORDS];
  part_ties<256>(a, lds, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(256) plan_pick_kernel(IngestArgs a) {
  __shared__ __align__(8) uint32_t lds[PLAN_LDS_WORDS];
  part_pick<256>(a, (uint64_t *)lds, blockIdx.x, gridDim.x);
}

// All of it in one workgroup, for a small batch: one launch instead of eight,
// and the counts never leave LDS.
__global__ void __launch_bounds__(1024) ingest_local_kernel(IngestArgs a) {
  __shared__ PackLds<1024, true> s;
  __shared__ uint64_t keys[INGEST_LOCAL];
  __shared__ uint32_t n_keys;
  __shared__ unsigned long long all_sums;
  const uint32_t tid = threadIdx.x;
  part_reset(a, tid, 1024);
  if (tid == 0) {
    n_keys = 0;
    all_sums = 0;
  }
  const bool loose = __syncthreads_or(part_headers(a, tid, 1024));
  if (loose) {
    part_fill(a, tid, 1024);
    __syncthreads();
    part_claim(a, tid, 1024);
    __syncthreads();
  }
  part_pack<1024, true>(a, s, loose, 0, 1);
  if (!a.cnt) return;
  __syncthreads();
  // (at most INGEST_LOCAL writes: their sum and their pairs' fit one word)
  static_assert((uint64_t)INGEST_LOCAL * INGEST_LOCAL < (1ull << 32), "pairs below bit 32");
  uint64_t sums = 0;
  for (uint32_t i = tid; i < rc_slots<true>; i += 1024)
    if (s.cnt[i]) {
      keys[atomicAdd(&n_keys, 1u)] = plan_key(s.row[i], s.cnt[i]);
      sums += (uint64_t)s.cnt[i] * (s.cnt[i] - 1) + ((uint64_t)s.cnt[i] << 32);
      if (a.hot_map && s.cnt[i] > 1) atomicOr(&a.hot_map[s.row[i] >> 5], 1u << (s.row[i] & 31));
    }
  sums = wave_sum(sums);
  if (__lane_id() == 0 && sums) atomicAdd(&all_sums, (unsigned long long)sums);
  __syncthreads();
  sort_candidates<1024>(a, keys, n_keys);
  __syncthreads();
  if (tid == 0) {
    a.out[INGEST_TOP] = ld_word(&a.out[INGEST_CAND]) >> 32;
    a.out[INGEST_PAIRS] = all_sums & 0xFFFFFFFFull;
    a.out[INGEST_WRITES] = all_sums >> 32;
  }
}

// The counts of a batch whose rows are known only at the run (keyed), or which
// has no submission (cc_run_static): as the pack and count parts above, without
// the candidates.  262,144 x 16 ops, half writes, uniform: 0.1 ms.
__global__ void __launch_bounds__(256) count_mark_kernel(const DevOp *ops, uint64_t n_ops, uint32_t *cnt,
                                                         uint32_t *rows, uint64_t *out, const uint64_t *err) {
  if (err && ld_word(err) != ~0ull) return;  // malformed: the descriptors are not the batch's
  if (blockIdx.x == 0 && threadIdx.x < 3) out[threadIdx.x] = 0;
  const uint64_t step = (uint64_t)gridDim.x * 256;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n_ops; i += step) {
    const uint32_t rk = ops[i].rowk;
    uint32_t mark = RC_NONE;
    if (rk != GAP_OP && op_leader(rk) && op_written(rk) && atomicAdd(&cnt[op_row(rk)], 1u) == 0) mark = op_row(rk);
    rows[i] = mark;
  }
}
__global__ void __launch_bounds__(256) count_sum_kernel(const uint32_t *rows, uint64_t n_ops, uint32_t *cnt,
                                                        uint64_t *out, const uint64_t *err) {
  if (err && ld_word(err) != ~0ull) return;
  uint32_t top = 0;
  uint64_t pairs = 0, writes = 0;
  const uint64_t step = (uint64_t)gridDim.x * 256;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n_ops; i += step) {
    const uint32_t r = rows[i];
    if (r == RC_NONE) continue;
    const uint32_t c = cnt[r];
    cnt[r] = 0;
    pairs += (uint64_t)c * (c - 1);
    writes += c;
    top = c > top ? c : top;
  }
  add_counts<256>(out, top, pairs, writes);
}
hipError_t launch_count_writes(hipStream_t s, const DevOp *ops, uint64_t n_ops, uint32_t *cnt, uint32_t *rows,
                               uint64_t *out, const uint64_t *err, int n_cu) {
  const uint64_t most = (uint64_t)n_cu * 8, b = (n_ops + 255) / 256;
  const dim3 g((unsigned)(b < 1 ? 1 : (b < most ? b : most)));
  hipLaunchKernelGGL(count_mark_kernel, g, dim3(256), 0, s, ops, n_ops, cnt, rows, out, err);
  hipLaunchKernelGGL(count_sum_kernel, g, dim3(256), 0, s, rows, n_ops, cnt, out, err);
  return hipGetLastError();
}

hipError_t launch_ingest(hipStream_t s, const IngestArgs &a, int n_cu) {
  if (a.n_txns <= (uint64_t)INGEST_LOCAL / 4 && a.n_ops <= (uint64_t)INGEST_LOCAL) {
    hipLaunchKernelGGL(ingest_local_kernel, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
  }
  // 8 workgroups of 256 threads on every CU, or as many as there is work for
  const uint64_t most = (uint64_t)n_cu * 8;
  auto blocks = [&](uint64_t items, uint64_t per) {
    const uint64_t b = (items + per - 1) / per;
    return dim3((unsigned)(b < 1 ? 1 : (b < most ? b : most)));
  };
  hipLaunchKernelGGL(ingest_reset_kernel, dim3(1), dim3(256), 0, s, a);
  hipLaunchKernelGGL(ingest_headers_kernel, blocks(a.n_txns, 256), dim3(256), 0, s, a);
  hipLaunchKernelGGL(ingest_fill_kernel, blocks(a.n_ops, 256), dim3(256), 0, s, a);
  hipLaunchKernelGGL(ingest_claim_kernel, blocks(a.n_txns, 256 / IG_L), dim3(256), 0, s, a);
  hipLaunchKernelGGL(ingest_pack_kernel, blocks(a.n_txns, 256 / IG_L), dim3(256), 0, s, a);
  if (a.cnt) {
    const dim3 g = blocks(a.n_ops, 256 * PLAN_STEP);
    hipLaunchKernelGGL(plan_counts_kernel, g, dim3(256), 0, s, a);
    hipLaunchKernelGGL(plan_ties_kernel, g, dim3(256), 0, s, a);
    hipLaunchKernelGGL(plan_pick_kernel, g, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace cce
