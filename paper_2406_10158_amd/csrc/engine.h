// Internal layout shared by the host runtime (api.cpp) and the kernels (kernels.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/cc.h"

namespace cce {

// ---- device operation descriptor (16 B) ------------------------------------
// rowk packs the global row id (row within its table + the table's first row
// in the shared row-id space) with the op kind and two flags computed at
// submission:
//   FOLLOWER  the op touches the same row as the previous op of its txn, so
//             the row's first op ("leader") does the concurrency control;
//   WRITTEN   some op of the row group writes the row.
// elem is the cell index in the value arena (table base + row*fields + field).
struct DevOp {
  uint32_t rowk;
  uint32_t elem;
  int64_t arg;
};
static_assert(sizeof(DevOp) == 16, "DevOp is 16 bytes");

constexpr uint32_t ROW_BITS = 28;
constexpr uint32_t ROW_MASK = (1u << ROW_BITS) - 1u;
constexpr uint32_t KIND_SHIFT = 28;
constexpr uint32_t FOLLOWER_BIT = 1u << 30;
constexpr uint32_t WRITTEN_BIT = 1u << 31;
// rowk of an operation no transaction names: a follower that writes in a row
// group that is not written, which no real operation is
constexpr uint32_t GAP_OP = FOLLOWER_BIT | ((uint32_t)CC_ADD << KIND_SHIFT);

struct DevTxn {
  uint32_t first;  // first op
  uint32_t n;      // op count
};

struct DevOutcome {  // same layout as cc_outcome
  uint32_t status;
  uint32_t attempts;
  uint64_t serial_hi;
  uint64_t serial_lo;
  int64_t commit_ns;
};
static_assert(sizeof(DevOutcome) == sizeof(cc_outcome), "outcome layout");

// ---- device control block, cleared by the init kernel ----------------------
enum DevStat {
  DS_COMMITTED = 0,
  DS_ATTEMPTS = 1,
  DS_ABORT_LOCK = 2,
  DS_ABORT_VALID = 3,
  DS_GAVE_UP = 4,
  DS_MAX_ATTEMPTS = 5,
  DS_TS_OVERFLOW = 6,
  DS_DEFERRED = 7,
  DS_T_USEFUL = 8,  // wall-clock ticks, summed over teams
  DS_T_ABORT = 9,
  DS_T_WAIT = 10,
  DS_ADMIT_WAITS = 11,  // serving: admissions deferred because the byte budget was full
  DS_R1 = 12,           // OCC, committed attempts: ticks in each round (lock / read+ticket /
  DS_R2 = 13,           //   validate+install / release)
  DS_R3 = 14,
  DS_R4 = 15,
  DS_INDEX_MISS = 16,   // keyed operations whose key no row holds
  DS_WD_WAITS = 17,     // 2PL wait-die: times a team kept its locks and waited
  DS_LATCH_STUCK = 18,  // CC_RUN_LATCH: latches not obtained within the spin limit (run invalid)
  DS_HOT_ACQ = 19,      // OCC: acquisitions of the batch's most written row's lock
  DS_HOT_FAILED = 20,   //   of which the attempt then aborted
  DS_HOT_HOLD = 21,     //   ticks the row was held, summed over acquisitions
  DS_BLOCKED_WAITS = 22,// CC_RUN_WAIT_BLOCKER: waits for a held row entered
  DS_VERSION_MISS = 23, // MVCC: old-version reads that found their version's slot reused (attempt aborted)
  DS_N = 24
};

struct Ctl {
  uint64_t queue;        // next transaction index to hand out
  uint64_t ticket;       // serial ticket / timestamp counter (last value drawn)
  uint64_t start_clock;  // device wall clock at CC initialisation
  uint64_t pending_n;    // length of the pending list built between passes
  uint64_t budget_reserved;  // serving: bytes ever reserved (a FIFO position counter)
  uint64_t budget_released;  // serving: bytes ever released
  uint64_t stats[DS_N];
  uint64_t stop;             // set by a team whose wait exceeded its limit (GaccO, GPUTx) or whose latch
                             // was stuck (CC_RUN_LATCH); every team then exits
};

// Kernel arguments for a transaction run.
// Rows a batch's submission singles out as hot (most writes first).
constexpr int HOT_MAX = 8;

struct RunArgs {
  const DevOp *ops;
  const DevTxn *txns;
  const uint32_t *list;  // transactions of this pass (nullptr: 0..n_txns-1)
  uint64_t n_txns;       // transactions in this pass
  int64_t *data;    // value arena
  uint64_t *words;  // one control word per global row
  uint64_t *aux;    // second word per row (MVCC version pointer)
  uint64_t *nodes;  // MVCC version arena: n_nodes slots of 4 words {tag, prev, writer ts | cell << 32, pre-image}
  uint64_t n_nodes;
  uint64_t *node_ring;  // MVCC: slots handed out so far (the arena is a ring; pos -> slot pos % n_nodes)
  DevOutcome *out;
  int64_t *reads;   // per op read value
  Ctl *ctl;
  uint64_t max_attempts;
  uint32_t backoff_ticks;  // wall-clock ticks
  uint32_t ns_per_tick_q16;  // wall-clock tick length in ns, 16.16 fixed point
  uint32_t has_slot;       // batch contains WRITE_SLOT ops
  uint32_t defer_after;    // attempts in this pass before deferring (0: never)
  uint32_t pass;           // 0 for the first pass (attempt counts start at 0)
  uint32_t n_from_ctl;     // take the pass's transaction count from ctl->pending_n
  const int64_t *arrival;  // serving: arrival time of each transaction, wall-clock ticks after start
  uint64_t budget_cap;     // serving: admission cap on reserved bytes (0: no cap)
  uint32_t bytes_per_op;   // serving: log / version bytes one operation reserves
  uint32_t eager_install;  // OCC: store values in the validation round (undo on abort)
  uint32_t chunk;          // queue positions a team claims at a time (set by the launcher)
  uint32_t precheck;       // OCC, TicToc: load-only round before any lock: 0 never, 1 on retries, 2 always
  uint32_t wd_wait_limit;  // 2PL wait-die: waits of one attempt before it dies anyway
  uint32_t node_reuse;     // MVCC: 0 = a slot per op (op i keeps slot i, never reused); 1 = the ring protocol
  uint32_t *latch;         // CC_RUN_LATCH: one 32-bit latch per global row (else unused)
  // OCC: the batch's hottest written rows (most writes first), locked -- or,
  // for a read-only access, looked at -- in a round of their own once every
  // other row of the transaction is held (0 rows: one lock round)
  uint32_t n_late;
  uint32_t late[HOT_MAX];
  uint32_t hot0;           // the batch's most written row (~0u: none), for the hold statistics
  // OCC, TicToc (CC_RUN_WAIT_BLOCKER): in passes that defer, a team that failed
  // on a held row looks at that row's word every ~poll_ticks until it is free
  // or wait_max_ticks have passed, then retries after a random jitter below
  // jitter_ticks, instead of backing off
  uint32_t wait_blocker;
  uint32_t poll_ticks;
  uint32_t jitter_ticks;
  uint32_t backoff_cap;    // doublings of the back-off at most, in passes that defer
  uint64_t wait_max_ticks;
};

// A table's index on the device (index.hip): the table's keys sorted, with
// their rows, and a static 16-way search tree over them.  Level 0 is the
// sorted keys, padded with INT64_MAX to a multiple of 16; level l+1 holds the
// largest key of each 16-key node of level l, padded the same way; the top
// level is one node.
constexpr int INDEX_MAX_LEVELS = 8;
struct IndexDesc {
  const int64_t *keys;   // level 0
  const uint32_t *rows;  // row of each sorted key
  const int64_t *tree;   // levels 1..levels, level l at level_off[l]
  uint64_t n;            // keys (rows of the table)
  uint64_t level_off[INDEX_MAX_LEVELS + 1];
  uint64_t row_base;     // the table's first global row
  uint64_t elem_base;    // the table's first cell
  uint32_t n_fields;
  uint32_t levels;       // tree levels above level 0
};

// OCC's hot-row engine (hot_engine.hip).  Its plan: at most ENG_MAX rows of at
// most ENG_FIELDS fields, ENG_VALS cells in all.
constexpr int ENG_MAX = 32;
constexpr int ENG_FIELDS = 64;
constexpr int ENG_VALS = 1024;
struct EngineRows {
  uint32_t n_rows;            // 0: no engine
  uint32_t row[ENG_MAX];      // global rows
};
struct EngineDesc {           // one engine transaction: its id, first op, op count, and its first op's
  uint32_t txn, first, n, at; // place among the engine's ops
};
// Per-op metadata of a keyed batch: bit 31 keyed, bits 16-23 table, 0-7 field.
constexpr uint32_t META_KEYED = 1u << 31;

// Resolve the keys of a keyed batch: patch each keyed op's row and cell in
// `ops`, record its row (within its table) in rows_out, count misses in
// ctl->stats[DS_INDEX_MISS].  tree = false: binary search of the sorted keys;
// true: descent of the 16-way tree.  One lane per op either way.
hipError_t launch_index_lookup(hipStream_t s, bool tree, const int64_t *op_keys, const uint32_t *meta, DevOp *ops,
                               uint32_t *rows_out, uint64_t n_ops, const IndexDesc *idx, Ctl *ctl);

// Kernel arguments for a GaccO execution (gacco_exec.hip).
struct GaccoArgs {
  const DevOp *ops;
  const DevTxn *txns;
  uint64_t n_txns;
  const uint32_t *rank;  // per row-group leader: its position in the sorted access table
  int64_t *data;
  uint64_t *words;       // per row: the position whose turn it is
  DevOutcome *out;
  int64_t *reads;
  Ctl *ctl;
  uint64_t wait_limit_ticks;  // a team waiting longer than this without progress stops the run
  uint32_t poll_ticks;        // sleep per access queued ahead of the team on a row, wall-clock ticks
  uint32_t ns_per_tick_q16;
  uint32_t has_slot;
  uint32_t shared;            // CC_RUN_SHARED_READS: counters instead of turns (see gacco_prepare)
};

// GaccO preprocessing (gacco.hip): clears ctl->stop, then builds the access
// table, sorts it stably by row (radix sort) and writes the lock table (turn
// counters in `words`, per-leader ranks).  `scratch` holds
// gacco_scratch_words(n_ops) 32-bit words.
uint64_t gacco_scratch_words(uint64_t n_ops);
// Stable LSD radix sort (8-bit digits) of n (key, value) pairs on their low
// `bits` key bits.  keys/vals are sorted through `scratch`
// (radix_sort_scratch_words(n) words); *keys_out / *vals_out point at the
// result (the input arrays or the first 2n words of scratch).
uint64_t radix_sort_scratch_words(uint64_t n);
hipError_t radix_sort_pairs(hipStream_t s, uint32_t *keys, uint32_t *vals, uint64_t n, int bits, uint32_t *scratch,
                            uint32_t **keys_out, uint32_t **vals_out);
// Modes:
//  PREP_TURNS   each accessed row's word is the sorted position of its first
//               access, and a leader's rank is its own sorted position (the
//               turn it waits for);
//  PREP_SHARED  the words hold (accesses done, writes done) counters and a
//               leader's rank is its threshold: accesses before it in its row
//               for a write, writes before it for a read (reads between two
//               writes share the row);
//  PREP_HIGH    as PREP_TURNS, in the word's bits from PREP_HIGH_SHIFT on
constexpr int PREP_HIGH_SHIFT = 40;
enum PrepMode { PREP_TURNS = 0, PREP_SHARED = 1, PREP_HIGH = 2 };
hipError_t gacco_prepare(hipStream_t s, const DevOp *ops, uint64_t n_ops, uint32_t sentinel, uint64_t *words,
                         uint32_t *rank, uint32_t *scratch, Ctl *ctl, int mode);
// GaccO execution; hipErrorInvalidValue for an unsupported (lanes, ops per txn).
hipError_t launch_gacco(hipStream_t s, int lanes, int max_ops, int waves_per_wg, int grid, bool strict,
                        const GaccoArgs &a, int n_cu, int *grid_used);

// Ordered execution by cell chains (chain.hip): arguments of its kernels.
struct ChainArgs {
  const DevOp *ops;         // in serial order
  uint64_t n;
  uint32_t listed;          // ops is a list of its own: an entry's elem is the index of its read value
  uint32_t pad;
  const uint32_t *keys;     // sorted by cell ...
  const uint32_t *vals;     // ... the entries of ops, in serial order within a cell
  int64_t *data;
  int64_t *reads;
  uint64_t *meta, *sum, *total;  // per tile: look-back state (meta is cleared by chain_prepare)
  uint32_t *base;           // batches with breaks: per operation, 1 + the break its value is relative to (else nullptr)
  uint64_t *result;         //   per break: the value it leaves
  uint32_t *ready;          //   per break: its result is there (cleared by chain_prepare)
  uint32_t *txn_first;      // batches with slot writes: the first operation of an operation's transaction
  Ctl *ctl;                 // queue and pending_n are counted up from 0
  uint64_t wait_limit_ticks;
};
uint64_t chain_tiles(uint64_t n);
// Builds and sorts the list of accesses by cell (ids below n_cells): keys and vals hold n words
// each, sort_scratch radix_sort_scratch_words(n); *keys_out and *vals_out are
// the sorted list for chain_execute.
hipError_t chain_prepare(hipStream_t s, const ChainArgs &a, uint64_t n_cells, const DevTxn *txns, uint64_t n_txns,
                         uint32_t *keys, uint32_t *vals, uint32_t *sort_scratch, uint32_t **keys_out, uint32_t **vals_out);
// The scan alone.
hipError_t chain_scan(hipStream_t s, bool strict, const ChainArgs &a, int n_cu);
// Runs the batch and writes its outcome records: serial key (rank, id), rank 0
// where rank is nullptr.  Does nothing but mark them pending if ctl->stop is set.
hipError_t chain_execute(hipStream_t s, bool strict, const ChainArgs &a, DevOutcome *out, uint64_t n_txns,
                         const uint32_t *rank, uint32_t ns_per_tick_q16, int n_cu, int *grid_used);

// Kernel arguments for GPUTx's rank pass (gputx.hip).
struct GputxArgs {
  const DevOp *ops;
  const DevTxn *txns;
  uint64_t n_txns;
  const uint32_t *rank;       // per row-group leader: its sorted position (the turn it waits for)
  uint64_t *words;            // per row: the turn
  uint64_t *kstate;           // per row: (largest rank + 1 of its accessors so far) << 32 | (last writer's rank + 1)
  uint32_t *txn_rank;         // output: per transaction
  Ctl *ctl;
  uint64_t wait_limit_ticks;
  uint32_t poll_ticks;
  uint32_t packed;            // turn and rank state share the row's word (see gputx.hip)
  uint32_t *known;            // packed: per sorted position, what is known of the access before its turn, 0 at
                              // first (nullptr: rows pass from team to team)
};
hipError_t launch_gputx_rank(hipStream_t s, int lanes, int max_ops, int waves_per_wg, int grid, bool strict,
                             const GputxArgs &a, int n_cu, int *grid_used);
hipError_t gputx_init_state(hipStream_t s, uint64_t *kstate, uint64_t n_rows);
// Claim counters back to 0, after the rank pass.
hipError_t gputx_reset(hipStream_t s, Ctl *ctl);

// Device-side ingest of a batch already in device memory (ingest.hip).
struct IngestTable {
  uint64_t n_rows;
  uint64_t row_base;   // first global row
  uint64_t elem_base;  // first cell
  uint32_t n_fields;
  uint32_t indexed;    // keyed batches: the table has an index (its ops name rows by key)
};
// reduced results in IngestArgs::out
constexpr int PLAN_CAND = 48;         // candidates for hot rows and engine rows: more than both take
constexpr int PLAN_COUNTS = 2048;     // bins of the histogram of row counts
constexpr int PLAN_BINS = 4096;       // bins of the histogram of rows
constexpr int PLAN_SORT = 2048;       // candidates sorted in LDS
constexpr int INGEST_LOCAL = 2048;    // ops that one workgroup takes in
// Rows gathered for the sort: those above the cut (fewer than PLAN_CAND), and
// at the cut at most PLAN_SORT / 2 rows, or one bin of rows more than the
// PLAN_CAND needed (2^16 rows), or all that are written PLAN_COUNTS - 1 times
// and more.
constexpr uint64_t plan_cand_max(uint64_t n_ops) {
  const uint64_t m = 2 * PLAN_CAND + PLAN_SORT + (1u << 16) + n_ops / (PLAN_COUNTS - 1);
  return m < n_ops ? m : n_ops;
}
enum IngestOut {
  INGEST_ERR = 0,
  INGEST_MAX_OPS,
  INGEST_KINDS,      // bit 0 a WRITE_SLOT, bit 1 a COND_ADD
  INGEST_UNORDERED,
  INGEST_KEYED,
  INGEST_LOOSE,      // the transactions' ops do not simply follow one another
  INGEST_DONE1,      // workgroups done with a part
  INGEST_DONE2,
  INGEST_DONE3,
  INGEST_CUT,        // lowest count of a candidate, and the rows above it
  INGEST_ABOVE,
  INGEST_TIES,
  INGEST_ROW_CUT,
  INGEST_N_CAND,
  INGEST_TOP,        // writes to the most written row
  INGEST_PAIRS,      // sum over the rows of c (c - 1), c writes: ordered pairs of writes that meet
  INGEST_WRITES,     // sum over the rows of c
  INGEST_CAND,       // PLAN_CAND x (count << 32 | ~row), most written first, 0: none
  INGEST_N = INGEST_CAND + PLAN_CAND
};
// what failed (bits 4-15 of the error word); the host turns it into a message
enum IngestMsg {
  INGEST_MSG_RESERVED = 1,
  INGEST_MSG_TOO_MANY,
  INGEST_MSG_OP_RANGE,
  INGEST_MSG_SHARED,
  INGEST_MSG_TABLE,
  INGEST_MSG_KEYED_ROW,
  INGEST_MSG_ROW_FIELD,
  INGEST_MSG_KIND,
  INGEST_MSG_SLOT_SRC,
  INGEST_MSG_DUP_FIELD,
  INGEST_MSG_DUP_ROW
};
struct IngestArgs {
  const cc_txn *txns;     // caller's device arrays
  const cc_op *ops;
  const int64_t *op_keys; // keyed batches (else nullptr)
  uint64_t n_txns, n_ops;
  IngestTable tab[CC_MAX_TABLES];
  uint32_t n_tables;
  uint32_t row_shift;     // rows per bin of the histogram of rows: 1 << row_shift, PLAN_BINS bins cover every row
  DevOp *dops;            // packed descriptors (the batch's own buffers)
  DevTxn *dtx;
  uint32_t *owner;        // n_ops scratch words: lowest transaction naming each op
  uint32_t *meta;         // keyed batches: per-op keyed flag, table, field (else nullptr)
  uint32_t *rows0;        // keyed batches: per-op row as submitted
  uint64_t *out;          // INGEST_N words
  // rows the batch writes most (cnt nullptr: not looked for)
  uint32_t *cnt;          // per global row; 0 before and, if the batch is well formed, after
                          // (ops named by two transactions may leave counts behind)
  uint32_t *rows;         // n_ops scratch words
  uint64_t *keys;         // n_ops scratch words
  uint64_t *cand;         // plan_cand_max(n_ops) scratch words
  uint32_t *hist;         // PLAN_COUNTS + PLAN_BINS scratch words
  uint32_t *hot_map;      // a bit per global row, cleared: set for rows written more than once (nullptr: no)
};
// Resets out, then validates and packs; the host reads `out` afterwards.
hipError_t launch_ingest(hipStream_t s, const IngestArgs &a, int n_cu);

// Counts a batch's writes per global row from its descriptors: out[0] = the most
// written row's, out[1] = sum of c (c - 1) over the rows, out[2] = sum of c.  cnt: a count per
// global row, 0 before and after; rows: n_ops scratch words; err: nothing is
// counted unless it holds ~0 (nullptr: well formed).
hipError_t launch_count_writes(hipStream_t s, const DevOp *ops, uint64_t n_ops, uint32_t *cnt, uint32_t *rows,
                               uint64_t *out, const uint64_t *err, int n_cu);

// The transactions that write one of the engine's rows -- those of `map` (a bit
// per global row), or e's where map is nullptr -- in batch order: part (n_txns
// entries; nullptr: only count) lists them and then the others, desc describes
// them.  Afterwards scratch (split_scratch_words(n_txns) words) holds a 64-bit
// count of accesses to engine rows, then their number at [2 + n_txns] and their
// ops' at [2 + n_txns + 1 + n_txns].
constexpr uint64_t split_scratch_words(uint64_t n_txns) { return 2 + 2 * (n_txns + 1) + (n_txns + 1) / 4096 + 2; }
hipError_t launch_split(hipStream_t s, const DevOp *ops, const DevTxn *txns, uint64_t n_txns, const EngineRows &e,
                        const uint32_t *map, uint32_t *scratch, uint32_t *part, EngineDesc *desc, int n_cu);
// The engine over n_txns transactions of m ops, in desc's order (tickets
// ticket0 + 1, ...); leaves the claim counters at 0.  breaks: the batch has
// conditional adds or slot writes; slots: slot writes.
size_t engine_scratch_bytes(uint64_t m, bool breaks, bool slots);
hipError_t launch_engine(hipStream_t s, bool strict, const RunArgs &r, const EngineDesc *desc, uint64_t n_txns,
                         uint64_t m, uint64_t n_cells, bool breaks, bool slots, void *scratch, uint64_t ticket0,
                         uint64_t wait_limit_ticks, int n_cu);
// Exclusive scan of m 32-bit values in place (partial: (m + 4095) / 4096 + 1 words).
void exclusive_scan_u32(hipStream_t s, uint32_t *data, uint64_t m, uint32_t *partial);

// Latency percentiles of a run (latency.hip).
constexpr uint64_t LAT_BITS = 12;  // of the latencies' range, a level
constexpr int LAT_BINS = 1 << LAT_BITS;
constexpr int LAT_LEVELS = 3;      // up to 2^36 ns of range
constexpr int LAT_SMALL = 8192;    // transactions that one workgroup looks at
struct LatState {                  // zeroed by the init kernel
  uint64_t n, not_min, max, ksets;
  uint64_t done[1 + LAT_LEVELS];
  uint64_t shift;                  // 0: value[] is exact; else they need more levels than LAT_LEVELS
  uint64_t prefix[2], rank[2], value[2];
};
struct LatArgs {
  const DevOutcome *out;
  uint64_t n;
  const int64_t *arrival_ns;       // served batches: latencies count from here (else nullptr)
  LatState *st;
  uint32_t *hist;                  // LAT_LEVELS x 2 x LAT_BINS words
  uint32_t ksets;                  // also find the largest serial_hi + 1
  uint32_t pad;
};
hipError_t launch_latency(hipStream_t s, const LatArgs &a, int n_cu);

// Host-side launchers (kernels.hip).  lat: the latency state to zero.
hipError_t launch_init(hipStream_t s, uint64_t *words, uint64_t n_words, uint64_t *aux, uint64_t n_aux,
                       DevOutcome *out, uint64_t n_out, Ctl *ctl, LatState *lat, uint64_t ticket_start);

// Between passes: list the transactions neither committed nor given up, and
// reset the claim counter.  ctl->pending_n receives the count.
hipError_t launch_compact(hipStream_t s, const DevOutcome *out, uint64_t n_txns, uint64_t max_attempts,
                          uint32_t *list, Ctl *ctl);

// Runs one plain batch: returns hipErrorInvalidValue for an unsupported
// (lanes, ops-per-lane) combination.
hipError_t launch_txn(hipStream_t s, int scheme, int lanes, int max_ops, int waves_per_wg, int grid,
                      bool strict, bool latch, const RunArgs &a, int n_cu, int *grid_used);

// Per-scheme launchers (txn_<scheme>.hip).
#define CCE_DECLARE_LAUNCH(NAME)                                                                    \
  hipError_t NAME(hipStream_t s, int lanes, int max_ops, int waves_per_wg, int grid, bool strict, bool latch, \
                  const RunArgs &a, int n_cu, int *grid_used);
CCE_DECLARE_LAUNCH(launch_txn_occ)
CCE_DECLARE_LAUNCH(launch_txn_2pl)
CCE_DECLARE_LAUNCH(launch_txn_to)
CCE_DECLARE_LAUNCH(launch_txn_mvcc)
CCE_DECLARE_LAUNCH(launch_txn_tictoc)
CCE_DECLARE_LAUNCH(launch_txn_2plwd)
#undef CCE_DECLARE_LAUNCH

// The allocation-free run's device buffers (static_run.hip): one file-scope
// array per device, carved into the regions below.  Sizes follow
// CC_STATIC_MAX_TXNS and CC_STATIC_MAX_OPS (cc.h).
constexpr uint64_t STATIC_OFF_OPS = 0;
constexpr uint64_t STATIC_OFF_TXNS = STATIC_OFF_OPS + (uint64_t)CC_STATIC_MAX_OPS * sizeof(DevOp);
constexpr uint64_t STATIC_OFF_LIST = STATIC_OFF_TXNS + (uint64_t)CC_STATIC_MAX_TXNS * sizeof(DevTxn);
constexpr uint64_t STATIC_OFF_OWNER = STATIC_OFF_LIST + (uint64_t)CC_STATIC_MAX_TXNS * sizeof(uint32_t);
constexpr uint64_t STATIC_OFF_INGEST = STATIC_OFF_OWNER + (uint64_t)CC_STATIC_MAX_OPS * sizeof(uint32_t);
constexpr uint64_t STATIC_SCRATCH_BYTES = STATIC_OFF_INGEST + 1024;
static_assert(STATIC_OFF_TXNS % 256 == 0 && STATIC_OFF_LIST % 256 == 0 && STATIC_OFF_OWNER % 256 == 0 &&
                  STATIC_OFF_INGEST % 256 == 0 && INGEST_N * sizeof(uint64_t) <= 1024,
              "static scratch regions are 256-byte aligned");
// Device address of `device`'s array; `device` must be current.  Resolved
// with hipGetSymbolAddress on a device's first call, then kept.
constexpr int STATIC_MAX_DEVICES = 64;
hipError_t static_scratch_address(int device, void **ptr);
// Clears n int64 words with a fill kernel.
hipError_t launch_fill_zero(hipStream_t s, int64_t *p, uint64_t n);

// Memory micro-benchmarks (roofline.hip); see cc_probe in cc.h.
hipError_t run_probe(hipStream_t s, int kind, uint64_t footprint_bytes, uint64_t n_ops, int peer,
                     const uint64_t *host_idx, double *ms_out, uint64_t *err_out, int n_cu);

}  // namespace cce
