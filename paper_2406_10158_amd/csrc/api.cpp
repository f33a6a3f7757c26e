// C-ABI of the batch transaction engine: context, tables, batches, runs.
// Declarations and the contract of every call are in include/cc.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cmath>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "engine.h"

using namespace cce;

namespace {

struct Table {
  uint64_t n_rows;
  uint32_t n_fields;
  uint64_t row_base;   // first global row id
  uint64_t elem_base;  // first cell in the value arena
};

struct Batch {
  int scheme = 0;
  uint64_t n_txns = 0, n_ops = 0;
  uint32_t max_ops = 0;
  bool has_slot = false, has_cond = false;
  DevOp *d_ops = nullptr;
  DevTxn *d_txns = nullptr;
  DevOutcome *d_out = nullptr;
  int64_t *d_reads = nullptr;
  uint32_t *d_list = nullptr;  // pending transactions between passes
  void *arena = nullptr;       // one allocation for the buffers whose sizes the counts give
  size_t arena_bytes = 0;
  uint64_t *d_nodes = nullptr; // MVCC version arena: a 32-byte header (the ring counter), then node_slots x 4 words
  uint64_t node_slots = 0;
  bool keyed = false;            // some ops name their row by key (cc_submit_batch_keyed)
  int64_t *d_opkeys = nullptr;   // keyed batches: per-op key
  uint32_t *d_meta = nullptr;    // keyed batches: per-op keyed flag, table, field
  uint32_t *d_rows = nullptr;    // keyed batches: per-op row found by the last run's lookups
  uint32_t *d_rank = nullptr;    // GaccO: per row-group leader, its position in the sorted access table
  uint32_t *d_gscratch = nullptr;// GaccO, GPUTx: access-table and sort buffers
  uint32_t *d_tscratch = nullptr;// GPUTx: per-transaction ranks
  uint64_t *d_chain = nullptr;   // GaccO, GPUTx: the chain scan's tile states, 3 words per tile
  uint64_t *d_breaks = nullptr;  //   with conditional adds or slot writes: results, ready words, transactions' first ops
  int64_t *d_arrival = nullptr;           // serving: arrival ticks per transaction, then nanoseconds
  std::vector<int64_t> arrival_ns;        // host copy, for latency statistics
  hipGraphExec_t epoch_graph = nullptr;  // captured epochs for the last epoch-mode parameters
  uint64_t epoch_key[4] = {0, 0, 0, 0};
  int epoch_grid = 0;
  bool ran = false;
  uint64_t stats[CC_N_STATS] = {};
  // counted at submission (plan_hot_rows): writes to the most written row,
  // and the most written rows (most first); hot_known is false for a batch
  // without a submission by row (cc_run_static, keyed)
  bool hot_known = false;
  uint64_t hot_writes = 0;
  // what the launch shape goes by: writes of the most written row, and whether
  // they are known (of a keyed batch from its first plain run on)
  bool shape_known = false;
  uint64_t shape_writes = 0;
  double meet = 0;   // expected writes of one transaction to rows another one writes, for a random pair
  double clash = 0;  // meet, raised where there are more reads than writes, which meet writes too
  double rest_clash = 0;  // the same of the transactions that the hot-row engine leaves: their reads and writes
  uint32_t n_hot = 0;
  uint32_t hot_rows[HOT_MAX] = {};
  // OCC's hot-row engine (hot_engine.hip): the plan's rows, and whether the
  // batch's hot rows are worth it (decided at submission).  d_part, from the
  // split (split_batch): the engine's transactions (n_eng_txns), then the
  // others; d_eng_desc: the engine's.  plan_txns: the transactions that write one
  // of the plan's rows (~0: not counted yet, cc_engine_plan)
  EngineRows eng{};
  bool eng_default = false;
  uint64_t plan_txns = ~0ull;
  uint64_t n_eng_txns = 0, n_eng_ops = 0, eng_behind = 0;
  uint32_t *d_part = nullptr;
  EngineDesc *d_eng_desc = nullptr;
};

}  // namespace

struct DevIndex {
  int64_t *keys = nullptr;
  uint32_t *rows = nullptr;
  int64_t *tree = nullptr;
  IndexDesc desc{};
};

// Pinned host memory of a context: a batch's host arrays up to this size go to
// the device in one copy from here (a pageable copy costs about 10 us more).
constexpr size_t PIN_BYTES = 1u << 20;

struct cc_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  int n_cu = 0;
  uint32_t wallclock_khz = 0;
  std::vector<Table> tables;
  bool frozen = false;
  uint64_t total_rows = 0, total_cells = 0;
  int64_t *d_data = nullptr;
  uint64_t *d_words = nullptr;
  uint64_t *d_aux = nullptr;
  Ctl *d_ctl = nullptr;
  std::vector<DevIndex> indexes;      // per table (empty entries: no index)
  IndexDesc *d_idx = nullptr;         // device copy of every table's IndexDesc
  uint32_t *d_latch = nullptr;        // CC_RUN_LATCH: one latch per global row
  uint64_t *d_kstate = nullptr;       // GPUTx: per-row rank state
  uint64_t *d_ingest = nullptr;       // batch submission: reduced results, then histograms
  uint32_t *d_hot = nullptr;          //   a bit per global row: hot in the batch being submitted
  uint32_t *d_cnt = nullptr;          //   a count per global row, 0 between submissions
  unsigned char *d_sub = nullptr;     //   scratch, grown to the largest batch's need
  size_t sub_bytes = 0;
  LatState *d_lat = nullptr;          // latency percentiles: state, then histograms
  unsigned char *h_pin = nullptr;     // PIN_BYTES of pinned host memory: small arrays on their way to or from the device
  std::vector<std::pair<void *, size_t>> pool;  // released batches' arenas (see release_arena)
  unsigned char *d_static = nullptr;  // cc_run_static: this device's static scratch (never freed)
  std::map<uint64_t, Batch> batches;
  uint64_t next_batch = 1;
  hipEvent_t ev[8] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  std::string err;
};

namespace {

thread_local std::string g_init_err;

cc_status fail(cc_ctx *c, cc_status st, const std::string &msg) {
  if (c) c->err = msg;
  return st;
}

// (a launch asks for the thread's last error: one that has been reported is not left for the next call to find)
cc_status hip_fail(cc_ctx *c, hipError_t e, const char *what) {
  (void)hipGetLastError();
  std::string m = std::string(what) + ": " + hipGetErrorString(e);
  if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) return fail(c, CC_E_NOMEM, m);
  return fail(c, CC_E_HIP, m);
}

#define HIP_OR(ctx, call)                              \
  do {                                                 \
    hipError_t e_ = (call);                            \
    if (e_ != hipSuccess) return hip_fail(ctx, e_, #call); \
  } while (0)

bool activate(cc_ctx *c) { return hipSetDevice(c->device) == hipSuccess; }

// Device memory for a context.  Out of memory, what the context only keeps for
// later is given back first: the released batches' arenas and, where the caller
// does not need it now, the submission scratch.
hipError_t dev_malloc(cc_ctx *c, void **p, size_t bytes, bool keep_scratch) {
  hipError_t e = hipMalloc(p, bytes);
  const bool scratch = c->d_sub && !keep_scratch;
  if (e != hipErrorOutOfMemory || (c->pool.empty() && !scratch)) return e;
  (void)hipGetLastError();
  for (auto &a : c->pool) (void)hipFree(a.first);
  c->pool.clear();
  if (scratch) {
    (void)hipFree(c->d_sub);
    c->d_sub = nullptr;
    c->sub_bytes = 0;
  }
  return hipMalloc(p, bytes);
}
template <class T>
hipError_t dev_malloc(cc_ctx *c, T **p, size_t bytes, bool keep_scratch = false) {
  return dev_malloc(c, (void **)p, bytes, keep_scratch);
}

cc_status freeze(cc_ctx *c) {
  if (c->frozen) return CC_OK;
  if (c->tables.empty()) return fail(c, CC_E_STATE, "no tables declared");
  uint64_t rows = 0, cells = 0;
  for (auto &t : c->tables) {
    t.row_base = rows;
    t.elem_base = cells;
    rows += t.n_rows;
    cells += t.n_rows * t.n_fields;
  }
  if (rows > CC_MAX_TOTAL_ROWS || cells > CC_MAX_TOTAL_CELLS) return fail(c, CC_E_RANGE, "tables too large");
  c->total_rows = rows;
  c->total_cells = cells;
  // all or nothing: a failed step frees what it allocated, so a later call can try again
  int64_t *data = nullptr;
  uint64_t *words = nullptr;
  hipError_t e = hipMalloc(&data, std::max<uint64_t>(cells, 1) * sizeof(int64_t));
  if (e == hipSuccess) e = hipMalloc(&words, std::max<uint64_t>(rows, 1) * sizeof(uint64_t));
  if (e == hipSuccess) e = hipMemsetAsync(data, 0, std::max<uint64_t>(cells, 1) * sizeof(int64_t), c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    if (data) (void)hipFree(data);
    if (words) (void)hipFree(words);
    return hip_fail(c, e, "table allocation");
  }
  c->d_data = data;
  c->d_words = words;
  // the counts per row, here for cc_run_static, which does not allocate (without
  // them it uses the shape for unknown rows, and a submission tries again)
  if (c->d_static) {
    const size_t bytes = std::max<uint64_t>(rows, 1) * sizeof(uint32_t);
    e = hipMalloc(&c->d_cnt, bytes);
    if (e == hipSuccess) e = hipMemsetAsync(c->d_cnt, 0, bytes, c->stream);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      (void)hipFree(c->d_cnt);
      c->d_cnt = nullptr;
    }
  }
  c->frozen = true;
  return CC_OK;
}

static hipError_t need_sub(cc_ctx *c, size_t bytes);
static void trim_sub(cc_ctx *c);

cc_status launch_error(cc_ctx *c, hipError_t e) {
  if (e == hipErrorInvalidValue) return fail(c, CC_E_INVAL, "scheme or (lanes_per_txn, ops per txn) not supported");
  if (e == hipErrorInvalidConfiguration)
    return fail(c, CC_E_INVAL, "waves_per_wg too large for the register slots this lanes_per_txn needs");
  return hip_fail(c, e, "transaction kernel launch");
}

// Resolve a keyed batch's keys on the device, after CC initialisation and
// inside the run's window; *ms receives the lookup kernel's time.
cc_status resolve_keys(cc_ctx *c, Batch &b, const cc_run_params &p, float *ms) {
  HIP_OR(c, hipEventRecord(c->ev[6], c->stream));
  HIP_OR(c, launch_index_lookup(c->stream, (p.flags & CC_RUN_INDEX_TREE) != 0, b.d_opkeys, b.d_meta, b.d_ops,
                                b.d_rows, b.n_ops, c->d_idx, c->d_ctl));
  HIP_OR(c, hipEventRecord(c->ev[7], c->stream));
  uint64_t miss = 0;
  HIP_OR(c, hipMemcpyAsync(&miss, &c->d_ctl->stats[DS_INDEX_MISS], sizeof miss, hipMemcpyDeviceToHost, c->stream));
  HIP_OR(c, hipStreamSynchronize(c->stream));
  HIP_OR(c, hipEventElapsedTime(ms, c->ev[6], c->ev[7]));
  if (miss) return fail(c, CC_E_RANGE, std::to_string(miss) + " keys name no row of their table's index");
  return CC_OK;
}

// What the counted rows say of the batch's conflicts.  Reads are not counted per
// row: they are taken to be distributed as the writes are, so that a row has as
// many reads a write as the batch (the pairs of a read and a write, counted, were
// within 2% of this on Zipf 0.3 and 0.6, half and a tenth writes).  clash is meet
// up to as many reads as writes, for which the rules below were measured, and
// grows with the pairs beyond (but not for short transactions of a skewed batch:
// 16 ops, Zipf 0.8 on 2M rows, a tenth writes, 2PL 0.75 ms with 1024 in flight, 0.80
// with 256).  Behind the hot-row engine no two write one row: what is left is the
// reads of rows written once, few where the batch is skewed (32 ops, Zipf 0.8 on
// 2M rows, OCC 0.23 ms with all of it in flight, 0.25 with 1024; 64 ops, Zipf 0.3
// on 262,144 rows, share 0.0013, 0.36 with all of it, 0.23 with 256).
void set_conflicts(Batch &b, uint64_t top, uint64_t pairs, uint64_t writes) {
  const double n = std::max(1.0, (double)b.n_txns), w = (double)writes, r = (double)b.n_ops - w;
  b.shape_known = true;
  b.shape_writes = top;
  b.meet = (double)pairs / (n * n);
  const double share = (double)top / n;
  b.clash = b.meet;
  if (writes && (b.max_ops > 16 || share < 0.001)) b.clash *= std::max(1.0, (1.0 + 2.0 * r / w) / 3.0);
  b.rest_clash = writes && share < 0.002 ? b.meet * 2.0 * r / w / 3.0 : 0.0;
}

// Counts the writes of a keyed batch's rows, which its first lookup found, for
// the launch shape.  The counts per row are the submissions' (0 in between).
cc_status count_keyed(cc_ctx *c, Batch &b) {
  if (!c->d_cnt || need_sub(c, b.n_ops * sizeof(uint32_t)) != hipSuccess) {
    (void)hipGetLastError();
    return CC_OK;  // the shape for unknown rows will do
  }
  uint64_t res[3] = {};
  HIP_OR(c, launch_count_writes(c->stream, b.d_ops, b.n_ops, c->d_cnt, (uint32_t *)c->d_sub, c->d_ingest, nullptr,
                                c->n_cu));
  HIP_OR(c, hipMemcpyAsync(res, c->d_ingest, sizeof res, hipMemcpyDeviceToHost, c->stream));
  HIP_OR(c, hipStreamSynchronize(c->stream));
  trim_sub(c);
  set_conflicts(b, res[0], res[1], res[2]);
  return CC_OK;
}

// Arenas of released batches are kept for the next ones of about their size,
// so that a stream of batches does not allocate (a 0.3 GB arena cost 0.4 ms a
// batch): at most POOL_ARENAS of at most POOL_BYTES in all, given back with the
// context or when an allocation fails.  The caller has waited for the context's
// stream.
constexpr size_t POOL_ARENAS = 4, POOL_BYTES = 512u << 20;

void free_batch(cc_ctx *c, Batch &b) {
  if (b.arena) {
    size_t kept = b.arena_bytes;
    for (auto &a : c->pool) kept += a.second;
    if (kept <= POOL_BYTES && c->pool.size() < POOL_ARENAS) c->pool.emplace_back(b.arena, b.arena_bytes);
    else (void)hipFree(b.arena);
  }
  if (b.d_part) (void)hipFree(b.d_part);
  if (b.d_eng_desc) (void)hipFree(b.d_eng_desc);
  if (b.d_nodes) (void)hipFree(b.d_nodes);
  if (b.d_breaks) (void)hipFree(b.d_breaks);
  if (b.epoch_graph) (void)hipGraphExecDestroy(b.epoch_graph);
  if (b.d_arrival) (void)hipFree(b.d_arrival);
  b = Batch{};
}

// Queues the copy of the control block and, if wanted, the latency percentiles
// and their copy; both arrive in pinned memory (RunTail) with the next
// synchronisation.
struct RunTail {
  Ctl ctl;
  LatState lat;
};
static_assert(sizeof(RunTail) <= PIN_BYTES, "a run's tail fits the pinned memory");

hipError_t queue_tail(cc_ctx *c, const Batch &b, const int64_t *arrival_ns, bool latency) {
  RunTail *t = (RunTail *)c->h_pin;
  hipError_t e = hipSuccess;
  if (latency) {
    LatArgs a{};
    a.out = b.d_out;
    a.n = b.n_txns;
    a.arrival_ns = arrival_ns;
    a.st = c->d_lat;
    a.hist = (uint32_t *)(c->d_lat + 1);
    a.ksets = b.scheme == CC_GPUTX ? 1u : 0u;
    e = launch_latency(c->stream, a, c->n_cu);
    if (e == hipSuccess) e = hipMemcpyAsync(&t->lat, c->d_lat, sizeof(LatState), hipMemcpyDeviceToHost, c->stream);
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&t->ctl, c->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, c->stream);
  return e;
}

// The latency statistics that came with a tail.  Latencies further apart than
// the levels resolve (68 s) are selected from the records here.
cc_status take_latency(cc_ctx *c, Batch &b, bool serve) {
  const LatState &l = ((RunTail *)c->h_pin)->lat;
  b.stats[CC_STAT_LAT_P50_NS] = l.value[0];
  b.stats[CC_STAT_LAT_P99_NS] = l.value[1];
  if (b.scheme == CC_GPUTX) b.stats[CC_STAT_KSETS] = l.ksets;
  if (l.shift == 0) return CC_OK;
  std::vector<cc_outcome> o(b.n_txns);
  HIP_OR(c, hipMemcpy(o.data(), b.d_out, b.n_txns * sizeof(cc_outcome), hipMemcpyDeviceToHost));
  std::vector<int64_t> lat;
  lat.reserve(o.size());
  for (uint64_t t = 0; t < b.n_txns; ++t)
    if (o[t].status == CC_COMMITTED) lat.push_back(o[t].commit_ns - (serve ? b.arrival_ns[t] : 0));
  auto pick = [&](double q) {
    const size_t i = (size_t)(q * (double)(lat.size() - 1) + 0.5);
    std::nth_element(lat.begin(), lat.begin() + i, lat.end());
    return (uint64_t)lat[i];
  };
  b.stats[CC_STAT_LAT_P50_NS] = pick(0.50);
  b.stats[CC_STAT_LAT_P99_NS] = pick(0.99);
  return CC_OK;
}

}  // namespace

extern "C" {

const char *cc_version(void) { return "cc-gfx950 0.1"; }

const char *cc_strerror(cc_status s) {
  switch (s) {
    case CC_OK: return "ok";
    case CC_E_INVAL: return "invalid argument";
    case CC_E_RANGE: return "out of range";
    case CC_E_DUPROW: return "duplicate row access within a transaction";
    case CC_E_NOMEM: return "out of memory";
    case CC_E_TS_OVERFLOW: return "timestamp overflow";
    case CC_E_LIVELOCK: return "transactions still pending (attempt or epoch limit reached)";
    case CC_E_HIP: return "HIP runtime error";
    case CC_E_NODEV: return "no usable gfx950 device";
    case CC_E_STATE: return "call out of order";
    case CC_E_NOBATCH: return "unknown batch";
    default: return "unknown status";
  }
}

const char *cc_last_error(const cc_ctx *ctx) { return ctx ? ctx->err.c_str() : g_init_err.c_str(); }

cc_status cc_init(cc_ctx **out, const cc_config *cfg) {
  if (!out) return CC_E_INVAL;
  *out = nullptr;
  g_init_err.clear();
  int dev = cfg ? cfg->device : 0;
  if (cfg && cfg->flags != 0) {
    g_init_err = "cc_config.flags must be 0";
    return CC_E_INVAL;
  }
  int n = 0;
  if (hipGetDeviceCount(&n) != hipSuccess || n <= 0) {
    g_init_err = "no HIP device";
    return CC_E_NODEV;
  }
  if (dev < 0 || dev >= n) {
    g_init_err = "device ordinal out of range";
    return CC_E_NODEV;
  }
  hipDeviceProp_t p;
  if (hipGetDeviceProperties(&p, dev) != hipSuccess) {
    g_init_err = "hipGetDeviceProperties failed";
    return CC_E_NODEV;
  }
  if (std::strncmp(p.gcnArchName, "gfx950", 6) != 0) {
    g_init_err = std::string("device is ") + p.gcnArchName + ", the engine is built for gfx950";
    return CC_E_NODEV;
  }
  cc_ctx *c = new (std::nothrow) cc_ctx();
  if (!c) return CC_E_NOMEM;
  c->device = dev;
  c->stream = cfg ? (hipStream_t)cfg->stream : nullptr;
  c->n_cu = p.multiProcessorCount;
  if (!c->stream) {
    // a stream of our own (default priority), so that runs can be captured
    if (hipSetDevice(dev) != hipSuccess || hipStreamCreate(&c->stream) != hipSuccess) {
      delete c;
      g_init_err = "hipStreamCreate failed";
      return CC_E_HIP;
    }
    c->own_stream = true;
  }
  int khz = 0;
  if (hipSetDevice(dev) != hipSuccess ||
      hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0) {
    delete c;
    g_init_err = "cannot read the device wall-clock rate";
    return CC_E_HIP;
  }
  c->wallclock_khz = (uint32_t)khz;
  if (hipMalloc(&c->d_ctl, sizeof(Ctl)) != hipSuccess ||
      hipMalloc(&c->d_lat, sizeof(LatState) + LAT_LEVELS * 2 * LAT_BINS * sizeof(uint32_t)) != hipSuccess ||
      hipHostMalloc((void **)&c->h_pin, PIN_BYTES, hipHostMallocDefault) != hipSuccess) {
    if (c->d_ctl) (void)hipFree(c->d_ctl);
    if (c->d_lat) (void)hipFree(c->d_lat);
    delete c;
    g_init_err = "allocation of the control block failed";
    return CC_E_NOMEM;
  }
  for (auto &e : c->ev) {
    if (hipEventCreate(&e) != hipSuccess) {
      cc_destroy(c);
      g_init_err = "hipEventCreate failed";
      return CC_E_HIP;
    }
  }
  // the allocation-free run's scratch on this device (the device is current)
  void *sp = nullptr;
  const hipError_t se = static_scratch_address(dev, &sp);
  if (se != hipSuccess) {
    cc_destroy(c);
    g_init_err = std::string("device address of the static scratch: ") + hipGetErrorString(se);
    return CC_E_HIP;
  }
  c->d_static = (unsigned char *)sp;
  *out = c;
  return CC_OK;
}

cc_status cc_destroy(cc_ctx *c) {
  if (!c) return CC_OK;
  activate(c);
  (void)hipStreamSynchronize(c->stream);
  for (auto &kv : c->batches) free_batch(c, kv.second);
  for (auto &a : c->pool) (void)hipFree(a.first);
  for (auto &ix : c->indexes) {
    if (ix.keys) (void)hipFree(ix.keys);
    if (ix.rows) (void)hipFree(ix.rows);
    if (ix.tree) (void)hipFree(ix.tree);
  }
  if (c->d_idx) (void)hipFree(c->d_idx);
  if (c->d_latch) (void)hipFree(c->d_latch);
  if (c->d_kstate) (void)hipFree(c->d_kstate);
  if (c->d_ingest) (void)hipFree(c->d_ingest);
  if (c->d_cnt) (void)hipFree(c->d_cnt);
  if (c->d_hot) (void)hipFree(c->d_hot);
  if (c->d_sub) (void)hipFree(c->d_sub);
  if (c->d_lat) (void)hipFree(c->d_lat);
  if (c->h_pin) (void)hipHostFree(c->h_pin);
  if (c->d_data) (void)hipFree(c->d_data);
  if (c->d_words) (void)hipFree(c->d_words);
  if (c->d_aux) (void)hipFree(c->d_aux);
  if (c->d_ctl) (void)hipFree(c->d_ctl);
  for (auto &e : c->ev)
    if (e) (void)hipEventDestroy(e);
  if (c->own_stream) (void)hipStreamDestroy(c->stream);
  delete c;
  return CC_OK;
}

cc_status cc_probe(cc_ctx *c, int kind, uint64_t footprint_bytes, uint64_t n_ops, int peer, double *ms) {
  if (!c || !ms) return CC_E_INVAL;
  if (kind < CC_PROBE_STREAM || kind > CC_PROBE_ENGINE_HANDOFF) return fail(c, CC_E_INVAL, "unknown probe");
  const bool pair = kind == CC_PROBE_HANDOFF || kind == CC_PROBE_COMMIT_HANDOFF;
  if (footprint_bytes < 4096 || (pair && (peer < 0 || peer > 64)))
    return fail(c, CC_E_INVAL, "bad probe size or peer");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  uint64_t err = 0;
  hipError_t e = run_probe(c->stream, kind, footprint_bytes, n_ops, peer, nullptr, ms, &err, c->n_cu);
  if (e != hipSuccess) return hip_fail(c, e, "probe");
  if (err) return fail(c, CC_E_LIVELOCK, "hand-off turn exceeded its bounded wait");
  return CC_OK;
}

cc_status cc_probe_indices(cc_ctx *c, int kind, uint64_t footprint_bytes, const uint64_t *indices, uint64_t n,
                           double *ms) {
  if (!c || !ms || (n && !indices)) return CC_E_INVAL;
  if (kind != CC_PROBE_GATHER && kind != CC_PROBE_GATHER_PLAIN && kind != CC_PROBE_SCATTER && kind != CC_PROBE_ATOMIC)
    return fail(c, CC_E_INVAL, "cc_probe_indices runs the gather, scatter and atomic probes");
  if (footprint_bytes < 4096) return fail(c, CC_E_INVAL, "bad probe size");
  const uint64_t words = footprint_bytes / sizeof(uint64_t) / 4 * 4;
  for (uint64_t i = 0; i < n; ++i)
    if (indices[i] >= words) return fail(c, CC_E_RANGE, "index beyond the probe's footprint");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  uint64_t err = 0;
  hipError_t e = run_probe(c->stream, kind, footprint_bytes, n, 1, indices, ms, &err, c->n_cu);
  if (e != hipSuccess) return hip_fail(c, e, "probe");
  return CC_OK;
}

cc_status cc_device_info(cc_ctx *c, uint32_t *n_cu, uint32_t *khz) {
  if (!c) return CC_E_INVAL;
  if (n_cu) *n_cu = (uint32_t)c->n_cu;
  if (khz) *khz = c->wallclock_khz;
  return CC_OK;
}

cc_status cc_create_table(cc_ctx *c, uint64_t n_rows, uint32_t n_fields, uint32_t *table_id) {
  if (!c || !table_id) return CC_E_INVAL;
  if (c->frozen) return fail(c, CC_E_STATE, "tables must be declared before the first cc_load");
  if (n_rows == 0 || n_fields == 0 || n_fields > 256) return fail(c, CC_E_INVAL, "bad table shape");
  if (c->tables.size() >= CC_MAX_TABLES) return fail(c, CC_E_RANGE, "too many tables");
  c->tables.push_back(Table{n_rows, n_fields, 0, 0});
  *table_id = (uint32_t)(c->tables.size() - 1);
  return CC_OK;
}

cc_status cc_load(cc_ctx *c, uint32_t tid, const int64_t *rows, uint64_t n_rows, int on_device) {
  if (!c || !rows) return CC_E_INVAL;
  if (tid >= c->tables.size()) return fail(c, CC_E_RANGE, "unknown table");
  if (n_rows != c->tables[tid].n_rows) return fail(c, CC_E_INVAL, "row count differs from the table's");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  cc_status st = freeze(c);
  if (st) return st;
  const Table &t = c->tables[tid];
  HIP_OR(c, hipMemcpyAsync(c->d_data + t.elem_base, rows, t.n_rows * t.n_fields * sizeof(int64_t),
                           on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, c->stream));
  HIP_OR(c, hipStreamSynchronize(c->stream));
  return CC_OK;
}

cc_status cc_read_table(cc_ctx *c, uint32_t tid, int64_t *out, int on_device) {
  if (!c || !out) return CC_E_INVAL;
  if (tid >= c->tables.size()) return fail(c, CC_E_RANGE, "unknown table");
  if (!c->frozen) return fail(c, CC_E_STATE, "table not loaded");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  const Table &t = c->tables[tid];
  HIP_OR(c, hipMemcpyAsync(out, c->d_data + t.elem_base, t.n_rows * t.n_fields * sizeof(int64_t),
                           on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, c->stream));
  HIP_OR(c, hipStreamSynchronize(c->stream));
  return CC_OK;
}

}  // extern "C"

namespace {

// Validate a batch against table shapes and build its device descriptors.
cc_status validate_and_pack(cc_ctx *c, const std::vector<Table> &tables, const cc_txn *txns, uint64_t n_txns,
                            const cc_op *ops, uint64_t n_ops, std::vector<DevOp> *dops_out,
                            std::vector<DevTxn> *dtx_out, uint32_t *max_ops_out, bool *has_slot_out,
                            bool *has_cond_out, bool *txn_ordered_out, const int64_t *op_keys = nullptr,
                            const std::vector<bool> *indexed = nullptr) {
  if ((n_txns && !txns) || (n_ops && !ops)) return fail(c, CC_E_INVAL, "null array");
  if (n_txns > 0xFFFFFFFFull || n_ops > 0xFFFFFFFFull) return fail(c, CC_E_RANGE, "batch too large");
  std::vector<DevOp> dummy_ops;
  std::vector<DevTxn> dummy_tx;
  std::vector<DevOp> &dops = dops_out ? *dops_out : dummy_ops;
  std::vector<DevTxn> &dtx = dtx_out ? *dtx_out : dummy_tx;
  // operations no transaction refers to are marked as gaps: they never enter
  // an access table
  dops.assign(n_ops, DevOp{GAP_OP, 0, 0});
  bool txn_ordered = true;  // every transaction's ops come after the previous one's
  dtx.assign(n_txns, DevTxn{0, 0});
  std::vector<uint8_t> used(n_ops, 0);  // every op belongs to at most one transaction
  std::vector<std::pair<uint32_t, int64_t>> keys;  // (table, row or key) of row leaders, for the duplicate check
  uint32_t max_ops = 0;
  bool has_slot = false, has_cond = false;
  for (uint64_t t = 0; t < n_txns; ++t) {
    const cc_txn &x = txns[t];
    if (x.reserved != 0) return fail(c, CC_E_INVAL, "cc_txn.reserved must be 0");
    if (x.n_ops > CC_MAX_OPS_PER_TXN) return fail(c, CC_E_INVAL, "transaction has too many ops");
    if (x.first_op > n_ops || x.n_ops > n_ops - x.first_op) return fail(c, CC_E_INVAL, "op range outside ops");
    if (t > 0 && x.first_op < txns[t - 1].first_op) txn_ordered = false;
    for (uint32_t i = 0; i < x.n_ops; ++i) {
      if (used[x.first_op + i]) return fail(c, CC_E_INVAL, "transactions share operations");
      used[x.first_op + i] = 1;
    }
    max_ops = std::max(max_ops, x.n_ops);
    keys.clear();
    uint32_t group_start = 0;
    bool group_written = false;
    // an op's row identity: its key on a table with an index (keyed batch), else its row
    auto keyed = [&](const cc_op &o) { return op_keys && indexed && o.table < indexed->size() && (*indexed)[o.table]; };
    auto ident = [&](uint32_t k) -> int64_t {
      const cc_op &o = ops[x.first_op + k];
      return keyed(o) ? op_keys[x.first_op + k] : (int64_t)o.row;
    };
    for (uint32_t i = 0; i < x.n_ops; ++i) {
      const cc_op &o = ops[x.first_op + i];
      if (o.table >= tables.size()) return fail(c, CC_E_RANGE, "op table out of range");
      const Table &tb = tables[o.table];
      const bool kd = keyed(o);
      if (kd && o.row != 0) return fail(c, CC_E_INVAL, "an op on an indexed table names its row by key; row must be 0");
      if ((!kd && o.row >= tb.n_rows) || o.field >= tb.n_fields) return fail(c, CC_E_RANGE, "op row/field out of range");
      if (o.kind > CC_WRITE_SLOT) return fail(c, CC_E_INVAL, "unknown op kind");
      if (o.kind == CC_WRITE_SLOT) {
        has_slot = true;
        if ((uint32_t)(o.arg & 0xFF) >= i) return fail(c, CC_E_INVAL, "WRITE_SLOT source is not an earlier op");
      }
      has_cond |= o.kind == CC_COND_ADD;
      const bool follower = i > 0 && ops[x.first_op + i - 1].table == o.table && ident(i - 1) == ident(i);
      if (!follower) {
        for (uint32_t j = group_start; j < i; ++j)
          if (group_written) dops[x.first_op + j].rowk |= WRITTEN_BIT;
        group_start = i;
        group_written = false;
        keys.emplace_back((uint32_t)o.table, ident(i));
      } else {
        for (uint32_t j = group_start; j < i; ++j)
          if (ops[x.first_op + j].field == o.field) return fail(c, CC_E_DUPROW, "field repeated within a txn");
      }
      group_written |= o.kind != CC_READ;
      // keyed ops get their row and cell from the lookup at the start of each run
      const uint64_t grow = kd ? 0 : tb.row_base + o.row;
      DevOp d;
      d.rowk = (uint32_t)grow | ((uint32_t)o.kind << KIND_SHIFT) | (follower ? FOLLOWER_BIT : 0u);
      d.elem = kd ? 0u : (uint32_t)(tb.elem_base + (uint64_t)o.row * tb.n_fields + o.field);
      d.arg = o.arg;
      dops[x.first_op + i] = d;
    }
    for (uint32_t j = group_start; j < x.n_ops; ++j)
      if (group_written) dops[x.first_op + j].rowk |= WRITTEN_BIT;
    std::sort(keys.begin(), keys.end());
    if (std::adjacent_find(keys.begin(), keys.end()) != keys.end())
      return fail(c, CC_E_DUPROW, "row accessed twice (non-adjacent) within a txn");
    dtx[t].first = (uint32_t)x.first_op;
    dtx[t].n = x.n_ops;
  }
  if (max_ops_out) *max_ops_out = max_ops;
  if (has_slot_out) *has_slot_out = has_slot;
  if (has_cond_out) *has_cond_out = has_cond;
  if (txn_ordered_out) *txn_ordered_out = txn_ordered;
  return CC_OK;
}

std::vector<Table> layout_tables(uint32_t n_tables, const uint64_t *n_rows, const uint32_t *n_fields) {
  std::vector<Table> v;
  uint64_t rows = 0, cells = 0;
  for (uint32_t t = 0; t < n_tables; ++t) {
    v.push_back(Table{n_rows[t], n_fields[t], rows, cells});
    rows += n_rows[t];
    cells += n_rows[t] * n_fields[t];
  }
  return v;
}

constexpr uint64_t GACCO_WAIT_LIMIT_MS = 4000;

// Wall-clock ticks a waiting team may go without progress before it stops
// the run (cc_run_params.wait_limit_us; 0 = GACCO_WAIT_LIMIT_MS).
uint64_t wait_limit_ticks(const cc_ctx *c, const cc_run_params &p) {
  if (p.wait_limit_us == 0) return (uint64_t)c->wallclock_khz * GACCO_WAIT_LIMIT_MS;
  return std::max<uint64_t>(1, p.wait_limit_us * c->wallclock_khz / 1000ull);
}

// Whether a launch shape exists: the kernels' variants hold 1, 4 or 16 operations
// a lane in registers, with room for fewer wavefronts the more they hold.  (The
// ordered schemes' chain scan has one shape and takes every batch, but refuses
// what their hand-off kernels refuse.)
hipError_t shape_exists(uint32_t lanes, uint32_t max_ops, uint32_t wpw) {
  const uint32_t k = (max_ops + lanes - 1) / lanes;
  const uint32_t most = lanes <= 4 ? 16u : 4u;
  if (k > most) return hipErrorInvalidValue;
  const uint32_t threads = lanes >= 16 && k <= 1 ? 1024u : (k <= 4 ? 512u : 256u);
  return 64 * wpw > threads ? hipErrorInvalidConfiguration : hipSuccess;
}

// The chain scan's arguments for a batch of an ordered scheme.
ChainArgs chain_args(const cc_ctx *c, const Batch &b, const cc_run_params &p) {
  ChainArgs a{};
  const uint64_t tiles = chain_tiles(b.n_ops);
  a.ops = b.d_ops;
  a.n = b.n_ops;
  a.data = c->d_data;
  a.reads = b.d_reads;
  a.meta = b.d_chain;
  a.sum = a.meta + tiles;
  a.total = a.sum + tiles;
  if (b.d_breaks) {
    a.base = b.d_rank;
    a.result = b.d_breaks;
    a.ready = (uint32_t *)(a.result + b.n_ops);
    if (b.has_slot) a.txn_first = a.ready + b.n_ops;
  }
  a.ctl = c->d_ctl;
  a.wait_limit_ticks = wait_limit_ticks(c, p);
  return a;
}

// What an ordered run reports, from the control block and the events of its parts.
cc_status ordered_stats(cc_ctx *c, Batch &b, bool chain, int grid_used, float ms_index, Ctl *h) {
  HIP_OR(c, queue_tail(c, b, nullptr, b.n_txns != 0));
  HIP_OR(c, hipStreamSynchronize(c->stream));
  *h = ((RunTail *)c->h_pin)->ctl;
  float ms_run = 0, ms_prep = 0, ms_kernel = 0;
  HIP_OR(c, hipEventElapsedTime(&ms_run, c->ev[0], c->ev[3]));
  HIP_OR(c, hipEventElapsedTime(&ms_prep, c->ev[4], c->ev[5]));
  HIP_OR(c, hipEventElapsedTime(&ms_kernel, c->ev[1], c->ev[2]));
  std::memset(b.stats, 0, sizeof(b.stats));
  b.stats[CC_STAT_COMMITTED] = h->stats[DS_COMMITTED];
  b.stats[CC_STAT_ATTEMPTS] = h->stats[DS_ATTEMPTS];
  b.stats[CC_STAT_KERNEL_NS] = (uint64_t)((double)ms_kernel * 1e6);
  b.stats[CC_STAT_RUN_NS] = (uint64_t)((double)ms_run * 1e6);
  b.stats[CC_STAT_PREP_NS] = (uint64_t)((double)ms_prep * 1e6);
  b.stats[CC_STAT_INDEX_NS] = (uint64_t)((double)ms_index * 1e6);
  b.stats[CC_STAT_MAX_ATTEMPTS] = h->stats[DS_MAX_ATTEMPTS];
  b.stats[CC_STAT_PASSES] = b.n_txns ? 1 : 0;
  b.stats[CC_STAT_GRID] = (uint64_t)grid_used;
  const double ns_per_tick = 1e6 / (double)c->wallclock_khz;
  b.stats[CC_STAT_T_USEFUL_NS] =
      chain ? b.stats[CC_STAT_KERNEL_NS] : (uint64_t)((double)h->stats[DS_T_USEFUL] * ns_per_tick);
  b.stats[CC_STAT_T_WAIT_NS] = (uint64_t)((double)h->stats[DS_T_WAIT] * ns_per_tick);
  b.ran = true;
  return b.n_txns ? take_latency(c, b, false) : CC_OK;
}

// GaccO run: CC initialisation, preprocessing, execution.  Every transaction
// runs exactly once.  By default the preprocessing sorts the accesses by cell
// and the execution is the chain scan (chain.hip), whose work does not depend
// on contention; a caller that bounds the waits for a row's turn
// (wait_limit_us) gets the hand-off kernel, whose waits those are, with the
// paper's lock table.  Both sides at 2^18 transactions x 16 ops, 10M rows: see
// chain.hip.
// (mode and flags were checked by check_run_params)
cc_status run_gacco(cc_ctx *c, Batch &b, const cc_run_params &p, uint32_t lanes, uint32_t wpw) {
  const bool strict = (p.flags & CC_RUN_STRICT_FENCES) != 0;
  const bool chain = p.wait_limit_us == 0;
  const hipError_t shape = b.n_txns ? shape_exists(lanes, b.max_ops, wpw) : hipSuccess;
  if (shape != hipSuccess) return launch_error(c, shape);
  const uint32_t ns_per_tick_q16 = (uint32_t)((1000000ull << 16) / c->wallclock_khz);

  HIP_OR(c, hipEventRecord(c->ev[0], c->stream));
  // no word is cleared: the chain scan uses none, the lock table sets those of every accessed row
  HIP_OR(c, launch_init(c->stream, c->d_words, 0, nullptr, 0, b.d_out, chain && !b.keyed ? 0 : b.n_txns, c->d_ctl,
                        c->d_lat, p.ts_start));
  float ms_index = 0;
  if (b.keyed) {
    cc_status st = resolve_keys(c, b, p, &ms_index);
    if (st) return st;
  }
  HIP_OR(c, hipEventRecord(c->ev[4], c->stream));
  int grid_used = 0;
  if (chain) {
    ChainArgs a = chain_args(c, b, p);
    uint32_t *keys = nullptr, *vals = nullptr;
    HIP_OR(c, chain_prepare(c->stream, a, c->total_cells, b.d_txns, b.n_txns, b.d_gscratch, b.d_gscratch + b.n_ops,
                            b.d_gscratch + 2 * b.n_ops, &keys, &vals));
    a.keys = keys;
    a.vals = vals;
    HIP_OR(c, hipEventRecord(c->ev[5], c->stream));
    HIP_OR(c, hipEventRecord(c->ev[1], c->stream));
    HIP_OR(c, chain_execute(c->stream, strict, a, b.d_out, b.n_txns, nullptr, ns_per_tick_q16, c->n_cu, &grid_used));
  } else {
    GaccoArgs a{};
    a.ops = b.d_ops;
    a.txns = b.d_txns;
    a.n_txns = b.n_txns;
    a.rank = b.d_rank;
    a.data = c->d_data;
    a.words = c->d_words;
    a.out = b.d_out;
    a.reads = b.d_reads;
    a.ctl = c->d_ctl;
    a.wait_limit_ticks = wait_limit_ticks(c, p);
    const uint64_t poll_ns = p.backoff_ns ? p.backoff_ns : 200;
    a.poll_ticks = (uint32_t)std::max<uint64_t>(1, poll_ns * c->wallclock_khz / 1000000ull);
    a.ns_per_tick_q16 = ns_per_tick_q16;
    a.has_slot = b.has_slot ? 1u : 0u;
    a.shared = (p.flags & CC_RUN_SHARED_READS) ? 1u : 0u;
    HIP_OR(c, gacco_prepare(c->stream, b.d_ops, b.n_ops, (uint32_t)c->total_rows, c->d_words, b.d_rank, b.d_gscratch,
                            c->d_ctl, a.shared ? PREP_SHARED : PREP_TURNS));
    HIP_OR(c, hipEventRecord(c->ev[5], c->stream));
    HIP_OR(c, hipEventRecord(c->ev[1], c->stream));
    if (b.n_txns) {
      hipError_t e = launch_gacco(c->stream, (int)lanes, (int)b.max_ops, (int)wpw, (int)p.grid, strict, a, c->n_cu,
                                  &grid_used);
      if (e != hipSuccess) return launch_error(c, e);
    }
  }
  HIP_OR(c, hipEventRecord(c->ev[2], c->stream));
  HIP_OR(c, hipEventRecord(c->ev[3], c->stream));
  Ctl h{};
  const cc_status st = ordered_stats(c, b, chain, grid_used, ms_index, &h);
  if (st) return st;
  if (h.stop) return fail(c, CC_E_LIVELOCK, "CC_GACCO: a transaction waited past the limit for its turn on a row");
  if (h.stats[DS_COMMITTED] != b.n_txns) return fail(c, CC_E_LIVELOCK, "CC_GACCO: not every transaction ran");
  return CC_OK;
}

// GPUTx run: CC initialisation, [index lookups], the lock table and the rank
// pass, then the execution.  The K-sets put conflicting transactions in id
// order, so the values are those of the chain scan in id order (chain.hip);
// the ranks are the outcomes' serial keys.  Running the K-sets one after
// another paid a hand-off of a done counter for each: 12.7 of 16.9 ms at 2^18
// transactions x 16 ops, 10M rows, Zipf 0.6.  Every transaction runs exactly once.
// (mode and flags were checked by check_run_params)
// Whether GPUTx's rank pass resolves rows ahead of their turns (gputx.hip): where
// a transaction waits for one row at a time.  Either few of the thousand or so
// in flight meet, or the most written row is most of what they meet.  Measured,
// the pass with and without (ms; 1024 x meet, share of the most written row): 16
// ops, half writes, Zipf 0.6 on 10M rows 1.74, 4.0 (0.1, 0.005); Zipf 0.7 3.1, 5.4
// (1, 0.02); Zipf 0.8 7.2, 8.4 (9, 0.06); Zipf 0.9 53, 46 (59, 0.17); uniform on
// 65,536 rows 1.40, 1.0 (1, < 0.001); 4 ops on 1,024 rows 2.8, 2.1 (4, 0.002).
static bool gputx_ahead(const Batch &b) {
  if (!b.shape_known || !b.n_txns) return false;
  const double x = b.meet * 1024.0, share = (double)b.shape_writes / (double)b.n_txns;
  return x <= 0.5 || (share >= 0.01 && x <= 10.0);
}

cc_status run_gputx(cc_ctx *c, Batch &b, const cc_run_params &p, uint32_t lanes, uint32_t wpw) {
  if (!c->d_kstate) HIP_OR(c, dev_malloc(c, &c->d_kstate, std::max<uint64_t>(c->total_rows, 1) * sizeof(uint64_t)));
  const uint64_t n = b.n_txns;
  GputxArgs a{};
  a.ops = b.d_ops;
  a.txns = b.d_txns;
  a.n_txns = n;
  a.rank = b.d_rank;
  a.words = c->d_words;
  a.kstate = c->d_kstate;
  a.txn_rank = b.d_tscratch;
  a.ctl = c->d_ctl;
  a.wait_limit_ticks = wait_limit_ticks(c, p);
  const uint64_t poll_ns = p.backoff_ns ? p.backoff_ns : 200;
  a.poll_ticks = (uint32_t)std::max<uint64_t>(1, poll_ns * c->wallclock_khz / 1000000ull);
  // the rank pass keeps each row's rank state in its turn word when both fit
  // (rank + 1 in 20 bits, a sorted position in 24)
  const bool packed = n < (1ull << 20) && b.n_ops < (1ull << 24);
  a.packed = packed ? 1u : 0u;
  const bool strict = (p.flags & CC_RUN_STRICT_FENCES) != 0;

  HIP_OR(c, hipEventRecord(c->ev[0], c->stream));
  HIP_OR(c, launch_init(c->stream, c->d_words, 0, nullptr, 0, b.d_out, b.keyed ? n : 0, c->d_ctl, c->d_lat, 0));
  float ms_index = 0;
  if (b.keyed) {
    cc_status st = resolve_keys(c, b, p, &ms_index);
    if (st) return st;
  }
  HIP_OR(c, hipEventRecord(c->ev[4], c->stream));
  HIP_OR(c, gacco_prepare(c->stream, b.d_ops, b.n_ops, (uint32_t)c->total_rows, c->d_words, b.d_rank, b.d_gscratch,
                          c->d_ctl, packed ? PREP_HIGH : PREP_TURNS));
  int grid_used = 0;
  if (n) {
    // (the sort's buffers are free again)
    if (packed && gputx_ahead(b)) {
      a.known = b.d_gscratch;
      HIP_OR(c, gputx_init_state(c->stream, (uint64_t *)a.known, (b.n_ops + 1) / 2));
    }
    if (!packed) HIP_OR(c, gputx_init_state(c->stream, c->d_kstate, c->total_rows));
    hipError_t e = launch_gputx_rank(c->stream, (int)lanes, (int)b.max_ops, (int)wpw, (int)p.grid, strict, a, c->n_cu,
                                     &grid_used);
    if (e != hipSuccess) return launch_error(c, e);
    HIP_OR(c, gputx_reset(c->stream, c->d_ctl));
  }
  ChainArgs ca = chain_args(c, b, p);  // (its breaks' bases take the place of the ranks in the rows' lists)
  uint32_t *keys = nullptr, *vals = nullptr;
  HIP_OR(c, chain_prepare(c->stream, ca, c->total_cells, b.d_txns, n, b.d_gscratch, b.d_gscratch + b.n_ops,
                          b.d_gscratch + 2 * b.n_ops, &keys, &vals));
  ca.keys = keys;
  ca.vals = vals;
  HIP_OR(c, hipEventRecord(c->ev[5], c->stream));
  HIP_OR(c, hipEventRecord(c->ev[1], c->stream));
  HIP_OR(c, chain_execute(c->stream, strict, ca, b.d_out, n, b.d_tscratch,
                          (uint32_t)((1000000ull << 16) / c->wallclock_khz), c->n_cu, &grid_used));
  HIP_OR(c, hipEventRecord(c->ev[2], c->stream));
  HIP_OR(c, hipEventRecord(c->ev[3], c->stream));
  Ctl h{};
  const cc_status st = ordered_stats(c, b, true, grid_used, ms_index, &h);
  if (st) return st;
  b.stats[CC_STAT_PACKED_STATE] = packed ? 1 : 0;
  if (h.stop) return fail(c, CC_E_LIVELOCK, "CC_GPUTX: a transaction waited past the limit");
  if (h.stats[DS_COMMITTED] != n) return fail(c, CC_E_LIVELOCK, "CC_GPUTX: not every transaction ran");
  return CC_OK;
}

// The hot-row engine's plan from the most written rows, most first: at most
// ENG_MAX of them, each written at least max(2, n_txns / 4096) times, of at
// most ENG_FIELDS fields and ENG_VALS cells in all.
static void plan_engine(const uint64_t *cand, int nc, const std::vector<Table> &tables, Batch &b) {
  b.eng = EngineRows{};
  const uint32_t thr = (uint32_t)std::max<uint64_t>(2, b.n_txns / 4096);
  uint32_t cells = 0;
  for (int i = 0; i < nc && b.eng.n_rows < (uint32_t)ENG_MAX; ++i) {
    const uint32_t r = ~(uint32_t)cand[i], writes = (uint32_t)(cand[i] >> 32);
    const Table *tb = nullptr;
    for (const Table &t : tables)
      if (r >= t.row_base && r < t.row_base + t.n_rows) tb = &t;
    if (writes < thr || !tb || tb->n_fields > (uint32_t)ENG_FIELDS || cells + tb->n_fields > (uint32_t)ENG_VALS) continue;
    b.eng.row[b.eng.n_rows++] = r;
    cells += tb->n_fields;
  }
}

// Launch shape of a plain run's transaction kernel where the caller leaves it
// to the library: lanes per transaction, wavefronts per workgroup, workgroups
// (0: one per compute unit).  A transaction's attempt takes 2-4 us of round
// trips, so that the transactions in flight, T, are the throughput until they
// conflict.  share: of the batch's transactions, those that write its most
// written row; clash: the expected conflicts of a random pair (Batch::clash), so
// that T of them have T x clash each.  known: false where the rows were not
// counted (a keyed batch of few transactions).
//
// Measured with 256 compute units, run time in ms at T = 256 (64 lanes),
// 512, 1024 (16 lanes), 4096 (4 lanes), 16384 (4 lanes, 4 wavefronts), OCC's
// kernel / TicToc / MVCC, 16 ops:
//   Zipf 0.8 (share 0.06), 65,536 txns: 12.7/15.4/16.9  14.1/15.8/18.9
//     14.1/15.8/19.3  31/39/45  39/46/54
//   Zipf 0.6 (0.005, clash 1.4e-4), 65,536: 1.13/1.19/1.43  0.96/1.16/1.59
//     1.09/1.24/1.56  1.63/2.35/3.37  2.3/3.4/4.2
//   Zipf 0.6, a tenth writes (0.001, 4e-5), 262,144: 4.0/4.0/4.2  2.4/2.4/2.9
//     1.5/1.6/2.0  1.6/2.3/3.8  2.6/3.3/4.5
//   uniform, 65,536 rows (< 0.001, 1e-3), 65,536: 1.22/1.38/1.35
//     1.05/1.16/1.09  0.89/1.03/0.83  1.6/2.3/1.4  3.0/3.6/2.4
//   uniform, 1M rows (6e-5): 1.03/1.03/1.06  0.59/0.57/0.63  0.45/0.46/0.45
//     0.22/0.26/0.28  0.51/0.55/0.38
//   uniform, 4M rows (1.5e-5), OCC: 0.45 at T = 1024, 0.27 at 16384
//   Zipf 0.3 on 65,536 rows, a tenth writes (< 0.001, 3e-4), 16,384:
//     0.21/0.22/0.24  0.12/0.13/0.16  0.12/0.13/0.12  0.13/0.20/0.16
// and 4,096 txns of 4 ops on 1,024 rows (clash 3.9e-3), OCC's kernel: 0.27 at
// 128, 0.22 at 256, 0.29 at 512, 0.41 at 4096; 8,192 of 16 ops on 4,096 rows
// (1.6e-2) 1.51 at 64, 1.42 at 256, 2.0 at 1024, on 1,024 rows (6e-2) 4.4 at
// 64, 6.0 at 256, 6.6 at 1024 (MVCC 3.6, 3.8, 4.1).
//
// Where few are in flight they have 64 lanes each, rather than 16 on a quarter
// of the compute units (but not the shortest: 4,096 txns of 1 op on 300 rows, OCC
// 0.12 with 16 lanes and 0.15 with 64); those of more than 16 ops, which 16 lanes
// hold in four slots with longer attempts, up to where 900 could be.
// T = 256 with 64 lanes, 256 and 1024 with 16; OCC's kernel / TicToc / wait-die / TO:
//   16 ops, uniform on 16,384 rows (4e-3), 16,384 txns: 0.72/0.93/0.62/0.60
//     0.84/0.98/0.82/0.68  0.79/1.02/0.80/0.59
//   64 ops, Zipf 0.3 on 262,144 rows, a tenth writes (1.2e-3), 8,192:
//     0.27/0.27/0.26/0.25  0.39/0.50/0.37/0.32  0.35/0.46/0.37/0.20
//   33-64 ops, half writes (2.7e-3): 0.27/0.41/0.28/0.25  0.47/0.69/0.60/0.27
//     0.45/0.72/0.67/0.24
//   64 ops, Zipf 0.3 on 2M rows, half writes (6e-4): 0.23/0.24/0.21/0.23
//     0.30/0.37/0.26/0.25  0.17/0.22/0.16/0.13
// Timestamp ordering, whose rows are held shortest, prefers more in flight.
// Transactions of at most 4 ops use 4 lanes with one slot each: uniform on 4M
// rows, 2^14 txns 60 us with 4096 in flight and 106 with 16384, 2^18 443 and
// 499, 2^20 1661 and 1733.
struct Shape {
  uint32_t lanes, waves;
  int grid;
};
static Shape plain_shape(int scheme, uint32_t max_ops, bool known, double share, double clash, int n_cu) {
  if (max_ops > 64) return {64, 1, 0};
  // no more in flight than conflict about once; but 256, or what conflict four
  // times, or 64
  auto limited = [&]() -> Shape {
    const double t = clash > 0 ? std::max({64.0, std::min(256.0, 4.0 / clash), 1.0 / clash}) : 1e9;
    const double few = max_ops <= 4 ? 0.0 : max_ops <= 16 ? 256.0 : scheme == CC_TO ? 400.0 : 900.0;
    if (t <= few) return {64, 1, t >= (double)n_cu ? 0 : (int)t};
    return {16, 1, t / 4 >= (double)n_cu ? 0 : (int)(t / 4)};
  };
  if (!known) {
    uint32_t lanes = 1;
    while (lanes < 64 && lanes < max_ops) lanes *= 4;
    return {lanes, 1, 0};
  }
  if (share >= 0.02) return {64, 1, 0};
  if (share >= 0.001) return limited();
  if (clash * (double)n_cu * 64 <= 0.3) return {4, max_ops <= 4 ? 1u : 4u, 0};
  if (clash * (double)n_cu * 16 <= 0.75) return {4, 1, 0};
  return limited();
}

// Whether OCC's hot-row engine is worth it, from estimates in us.  The engine
// takes 110 and 0.1 ns an op whatever the contention, and the rest of the batch
// -- the transactions none of whose writes meets another one's, e^-(meet x n) of
// them -- 2.2 ns each.  The transaction kernel takes 2.9 a write of the most
// written row, or, with T in flight in its shape, (n / T) times the attempts,
// 1 + 1.4 meet x T, times an attempt: 5 with 16 or 64 lanes, 7.5 with 4, 35
// with 4 wavefronts a workgroup.  Measured, the run with the kernel alone and
// with the engine (meet): 16 ops, 2^20 on 4M rows 2423, 1776 (1.5e-5); 2^18 on
// 4M rows 710, 570; on 1M rows 752, 470 (6e-5); on 65,536 rows 3154, 427 (1e-3);
// Zipf 0.6 on 1M rows 9402, 480; 2^16 on 4M rows 271, 326; 2^12 on 65,536 rows
// 101, 132; on 16,384 rows 228, 110 (4e-3); 4 ops, 2^16 on 262,144 rows 146, 198
// (1.5e-5); on 65,536 rows 181, 146 (6e-5); 2^14 on 65,536 rows 74, 135.  Where
// not one of 4096 in flight in twenty meets another the batch stays optimistic.
static bool engine_pays(const Batch &b, int n_cu) {
  const double n = (double)b.n_txns;
  if (b.meet * std::min(n, 4096.0) < 0.05) return false;
  const double share = (double)b.hot_writes / n;
  const Shape s = plain_shape(b.scheme, b.max_ops, true, share, b.clash, n_cu);
  const double t = std::min(n, (double)(s.grid ? s.grid : n_cu) * s.waves * (64.0 / s.lanes));
  const double attempt = s.waves > 1 ? 35.0 : s.lanes == 4 ? 7.5 : 5.0;
  const double kernel = 25.0 + std::max(n / t * (1.0 + 1.4 * b.meet * t) * attempt, 2.9 * (double)b.hot_writes);
  const double engine = 110.0 + 1e-4 * (double)b.n_ops + 2.2e-3 * n * std::exp(-b.meet * n);
  return engine < kernel;
}

// The batch's most written rows, counted at submission (write accesses per
// global row; ingest.hip): the most written row, and every row written at least
// a quarter as often, at most HOT_MAX of them, most written first (ties: lower
// row first).  With them, OCC's engine plan.
static void plan_hot_rows(const uint64_t *res, const std::vector<Table> &tables, Batch &b, int n_cu) {
  const uint64_t *cand = res + INGEST_CAND;
  int nc = 0;
  while (nc < PLAN_CAND && cand[nc]) ++nc;
  const uint32_t top = (uint32_t)res[INGEST_TOP];
  b.hot_known = true;
  b.hot_writes = top;
  set_conflicts(b, top, res[INGEST_PAIRS], res[INGEST_WRITES]);
  if (b.scheme == CC_OCC && !b.keyed) {
    plan_engine(cand, nc, tables, b);
    b.eng_default = engine_pays(b, n_cu);
  }
  b.n_hot = 0;
  const uint32_t thr = std::max<uint32_t>(1u, (top + 3) / 4);
  for (int i = 0; i < nc && i < HOT_MAX && (uint32_t)(cand[i] >> 32) >= thr; ++i) b.hot_rows[b.n_hot++] = ~(uint32_t)cand[i];
}

// At least `bytes` of submission scratch, which the hot-row engine uses too.  It
// grows to the largest batch's need; a very large one is given back when the
// submission is over, and the engine's, which a batch that runs again needs
// again, when a batch is released (trim_sub).
static hipError_t need_sub(cc_ctx *c, size_t bytes) {
  if (bytes <= c->sub_bytes) return hipSuccess;
  if (c->d_sub) (void)hipFree(c->d_sub);
  c->d_sub = nullptr;
  c->sub_bytes = 0;
  const hipError_t e = dev_malloc(c, &c->d_sub, bytes);
  if (e == hipSuccess) c->sub_bytes = bytes;
  return e;
}
static void trim_sub(cc_ctx *c) {
  constexpr size_t KEEP = 1u << 30;
  if (c->sub_bytes <= KEEP) return;
  (void)hipFree(c->d_sub);
  c->d_sub = nullptr;
  c->sub_bytes = 0;
}

// Splits the batch into the engine's transactions and the others, on the
// device (once): by `map`, the rows found hot at submission, or, without it, by
// the plan's rows.
static hipError_t split_batch(cc_ctx *c, Batch &b, const uint32_t *map) {
  if (b.d_part || b.n_txns == 0) return hipSuccess;
  uint32_t *part = nullptr, n_eng = 0, n_ops = 0;
  uint64_t behind = 0;
  EngineDesc *desc = nullptr;
  hipError_t e = need_sub(c, split_scratch_words(b.n_txns) * sizeof(uint32_t));
  uint32_t *w = (uint32_t *)c->d_sub;
  if (e == hipSuccess) e = dev_malloc(c, &part, b.n_txns * sizeof(uint32_t), true);
  if (e == hipSuccess) e = dev_malloc(c, &desc, b.n_txns * sizeof(EngineDesc), true);
  if (e == hipSuccess) e = launch_split(c->stream, b.d_ops, b.d_txns, b.n_txns, b.eng, map, w, part, desc, c->n_cu);
  if (e == hipSuccess) e = hipMemcpyAsync(&behind, w, sizeof behind, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(&n_eng, w + 2 + b.n_txns, sizeof n_eng, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(&n_ops, w + 2 + 2 * b.n_txns + 1, sizeof n_ops, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    if (part) (void)hipFree(part);
    if (desc) (void)hipFree(desc);
    return e;
  }
  b.d_part = part;
  b.d_eng_desc = desc;
  b.n_eng_txns = n_eng;
  b.n_eng_ops = n_ops;
  b.eng_behind = behind;
  return hipSuccess;
}

// Run parameters against the scheme, before anything touches the device
// (cc_check_run_params and cc_run).  c may be NULL (no message kept).
cc_status check_run_params(cc_ctx *c, int scheme, const cc_run_params &p) {
  if (scheme < 0 || scheme >= CC_N_SCHEMES) return fail(c, CC_E_INVAL, "unknown scheme");
  if (p.mode != CC_MODE_PLAIN && p.mode != CC_MODE_EPOCH && p.mode != CC_MODE_SERVE)
    return fail(c, CC_E_INVAL, "unknown mode");
  const uint32_t lanes = p.lanes_per_txn;
  if (lanes != 0 && lanes != 1 && lanes != 4 && lanes != 16 && lanes != 64)
    return fail(c, CC_E_INVAL, "lanes_per_txn must be 1, 4, 16 or 64");
  if (p.waves_per_wg > 16) return fail(c, CC_E_INVAL, "waves_per_wg must be 1..16");
  if (p.flags & ~(CC_RUN_STRICT_FENCES | CC_RUN_EAGER_INSTALL | CC_RUN_WAIT_UNLOCK | CC_RUN_PRECHECK |
                  CC_RUN_NO_PRECHECK | CC_RUN_INDEX_TREE | CC_RUN_LATCH | CC_RUN_SHARED_READS | CC_RUN_HOT_LAST |
                  CC_RUN_NO_HOT_LAST | CC_RUN_WAIT_BLOCKER | CC_RUN_HOT_ENGINE | CC_RUN_NO_HOT_ENGINE))
    return fail(c, CC_E_INVAL, "unknown run flag");
  if ((p.flags & CC_RUN_SHARED_READS) && scheme != CC_GACCO)
    return fail(c, CC_E_INVAL, "CC_RUN_SHARED_READS is a CC_GACCO option");
  if (p.wait_limit_us && scheme != CC_GACCO && scheme != CC_GPUTX)
    return fail(c, CC_E_INVAL, "wait_limit_us applies to CC_GACCO and CC_GPUTX only");
  if (p.flags & CC_RUN_WAIT_UNLOCK)
    // Switched off: two teams of one wavefront that block each other both see
    // the row free on their next loop iteration (each attempt releases its
    // locks before returning) and retry together, so in the final
    // single-wavefront pass, which never defers, they can conflict forever.
    return fail(c, CC_E_INVAL, "CC_RUN_WAIT_UNLOCK is disabled (same-wavefront retries can livelock)");
  if (scheme == CC_GACCO) {
    if (p.mode != CC_MODE_PLAIN)
      return fail(c, CC_E_INVAL,
                  "CC_GACCO runs in CC_MODE_PLAIN only: it never aborts, so epochs have nothing to retry, and it "
                  "orders the whole batch before running it");
    if (p.flags & ~(CC_RUN_STRICT_FENCES | CC_RUN_INDEX_TREE | CC_RUN_SHARED_READS))
      return fail(c, CC_E_INVAL, "CC_GACCO accepts only CC_RUN_STRICT_FENCES, CC_RUN_INDEX_TREE and CC_RUN_SHARED_READS");
    return CC_OK;
  }
  if (scheme == CC_GPUTX) {
    if (p.mode != CC_MODE_PLAIN)
      return fail(c, CC_E_INVAL, "CC_GPUTX runs in CC_MODE_PLAIN only: it orders the whole batch before running it");
    if (p.flags & ~(CC_RUN_STRICT_FENCES | CC_RUN_INDEX_TREE))
      return fail(c, CC_E_INVAL, "CC_GPUTX accepts only CC_RUN_STRICT_FENCES and CC_RUN_INDEX_TREE");
    return CC_OK;
  }
  const uint32_t pre = CC_RUN_PRECHECK | CC_RUN_NO_PRECHECK;
  if ((p.flags & pre) == pre) return fail(c, CC_E_INVAL, "CC_RUN_PRECHECK and CC_RUN_NO_PRECHECK exclude each other");
  if ((p.flags & pre) && scheme != CC_OCC && scheme != CC_TICTOC && scheme != CC_TO && scheme != CC_MVCC)
    return fail(c, CC_E_INVAL, "the pre-check round exists for CC_OCC, CC_TICTOC, CC_TO and CC_MVCC only");
  if ((p.flags & CC_RUN_EAGER_INSTALL) && scheme != CC_OCC)
    return fail(c, CC_E_INVAL, "CC_RUN_EAGER_INSTALL is a CC_OCC option");
  const uint32_t hot = CC_RUN_HOT_LAST | CC_RUN_NO_HOT_LAST;
  if ((p.flags & hot) == hot) return fail(c, CC_E_INVAL, "CC_RUN_HOT_LAST and CC_RUN_NO_HOT_LAST exclude each other");
  if ((p.flags & hot) && scheme != CC_OCC) return fail(c, CC_E_INVAL, "CC_RUN_HOT_LAST is a CC_OCC option");
  if ((p.flags & CC_RUN_WAIT_BLOCKER) && scheme != CC_OCC && scheme != CC_TICTOC)
    return fail(c, CC_E_INVAL, "CC_RUN_WAIT_BLOCKER is a CC_OCC and CC_TICTOC option");
  const uint32_t eng = CC_RUN_HOT_ENGINE | CC_RUN_NO_HOT_ENGINE;
  if ((p.flags & eng) == eng) return fail(c, CC_E_INVAL, "CC_RUN_HOT_ENGINE and CC_RUN_NO_HOT_ENGINE exclude each other");
  if ((p.flags & eng) && scheme != CC_OCC) return fail(c, CC_E_INVAL, "CC_RUN_HOT_ENGINE is a CC_OCC option");
  if ((p.flags & CC_RUN_HOT_ENGINE) && p.mode != CC_MODE_PLAIN)
    return fail(c, CC_E_INVAL, "CC_RUN_HOT_ENGINE runs in CC_MODE_PLAIN only");
  if ((p.flags & CC_RUN_HOT_ENGINE) && (p.flags & CC_RUN_LATCH))
    return fail(c, CC_E_INVAL, "CC_RUN_HOT_ENGINE does not take CC_RUN_LATCH");
  return CC_OK;
}

}  // namespace

extern "C" {

cc_status cc_check_batch(uint32_t n_tables, const uint64_t *n_rows, const uint32_t *n_fields, const cc_txn *txns,
                         uint64_t n_txns, const cc_op *ops, uint64_t n_ops, int scheme) {
  if (n_tables > CC_MAX_TABLES || (n_tables && (!n_rows || !n_fields))) return CC_E_INVAL;
  if (scheme < 0 || scheme >= CC_N_SCHEMES) return CC_E_INVAL;
  uint64_t rows = 0, cells = 0;
  for (uint32_t t = 0; t < n_tables; ++t) {
    if (n_rows[t] == 0 || n_fields[t] == 0 || n_fields[t] > 256) return CC_E_INVAL;
    rows += n_rows[t];
    cells += n_rows[t] * n_fields[t];
  }
  if (rows > CC_MAX_TOTAL_ROWS || cells > CC_MAX_TOTAL_CELLS) return CC_E_RANGE;
  bool ordered = true;
  const cc_status st = validate_and_pack(nullptr, layout_tables(n_tables, n_rows, n_fields), txns, n_txns, ops, n_ops,
                                         nullptr, nullptr, nullptr, nullptr, nullptr, &ordered);
  if (st == CC_OK && (scheme == CC_GACCO || scheme == CC_GPUTX) && !ordered) return CC_E_INVAL;
  return st;
}

// Device buffers of a batch: descriptors, outcomes, read values, pending
// list, and the scheme's extras, in one allocation.  All or nothing.
static hipError_t alloc_batch(cc_ctx *c, Batch &b, bool keyed) {
  const bool ordered_scheme = b.scheme == CC_GACCO || b.scheme == CC_GPUTX;
  const uint64_t n_ops = b.n_ops, n_txns = b.n_txns;
  size_t bytes = 0;
  auto carve = [&](unsigned char *base) {
    bytes = 0;
    auto take = [&](auto **p, bool want, uint64_t n) {
      if (!want) return;
      if (base) *p = reinterpret_cast<std::remove_reference_t<decltype(*p)>>(base + bytes);
      bytes += (std::max<uint64_t>(n, 1) * sizeof(**p) + 255) / 256 * 256;
    };
    take(&b.d_ops, true, n_ops);
    take(&b.d_txns, true, n_txns);
    take(&b.d_out, true, n_txns);
    take(&b.d_reads, true, n_ops);
    take(&b.d_list, true, n_txns);
    take(&b.d_rank, ordered_scheme, n_ops);
    take(&b.d_gscratch, ordered_scheme, gacco_scratch_words(n_ops));
    take(&b.d_chain, ordered_scheme, 3 * chain_tiles(n_ops));
    take(&b.d_tscratch, b.scheme == CC_GPUTX, n_txns);
    take(&b.d_opkeys, keyed, n_ops);
    take(&b.d_meta, keyed, n_ops);
    take(&b.d_rows, keyed, n_ops);
  };
  carve(nullptr);
  auto best = c->pool.end();
  for (auto it = c->pool.begin(); it != c->pool.end(); ++it)
    if (it->second >= bytes && it->second / 4 <= bytes && (best == c->pool.end() || it->second < best->second)) best = it;
  if (best != c->pool.end()) {
    b.arena = best->first;
    b.arena_bytes = best->second;
    c->pool.erase(best);
  } else {
    const hipError_t e = dev_malloc(c, &b.arena, bytes, true);
    if (e != hipSuccess) {
      b.arena = nullptr;
      return e;
    }
    b.arena_bytes = bytes;
  }
  carve((unsigned char *)b.arena);
  return hipSuccess;
}

// The buffers of an ordered batch's breaks (chain.hip), once its kinds of operations are known.
static hipError_t alloc_breaks(cc_ctx *c, Batch &b) {
  const bool ordered_scheme = b.scheme == CC_GACCO || b.scheme == CC_GPUTX;
  if (!ordered_scheme || !(b.has_slot || b.has_cond) || b.n_ops == 0) return hipSuccess;
  return dev_malloc(c, &b.d_breaks, b.n_ops * (sizeof(uint64_t) + 2 * sizeof(uint32_t)));
}

// True if [p, p + bytes) lies inside one allocation of the context's device.
static bool device_range(const cc_ctx *c, const void *p, uint64_t bytes) {
  if (bytes == 0) return true;
  if (!p) return false;
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (at.type != hipMemoryTypeDevice || at.device != c->device) return false;
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const uintptr_t lo = (uintptr_t)base, q = (uintptr_t)p;
  return q >= lo && bytes <= size && q - lo <= size - bytes;
}

static const char *ingest_message(uint32_t m) {
  switch (m) {
    case INGEST_MSG_RESERVED: return "cc_txn.reserved must be 0";
    case INGEST_MSG_TOO_MANY: return "transaction has too many ops";
    case INGEST_MSG_OP_RANGE: return "op range outside ops";
    case INGEST_MSG_SHARED: return "transactions share operations";
    case INGEST_MSG_TABLE: return "op table out of range";
    case INGEST_MSG_KEYED_ROW: return "an op on an indexed table names its row by key; row must be 0";
    case INGEST_MSG_ROW_FIELD: return "op row/field out of range";
    case INGEST_MSG_KIND: return "unknown op kind";
    case INGEST_MSG_SLOT_SRC: return "WRITE_SLOT source is not an earlier op";
    case INGEST_MSG_DUP_FIELD: return "field repeated within a txn";
    case INGEST_MSG_DUP_ROW: return "row accessed twice (non-adjacent) within a txn";
    default: return "malformed batch";
  }
}

// The ingest kernels' view of the tables and of a batch's arrays on the device.
static IngestArgs ingest_args(const cc_ctx *c, const cc_txn *txns, uint64_t n_txns, const cc_op *ops, uint64_t n_ops) {
  IngestArgs ia{};
  ia.txns = txns;
  ia.ops = ops;
  ia.n_txns = n_txns;
  ia.n_ops = n_ops;
  ia.n_tables = (uint32_t)c->tables.size();
  for (uint32_t t = 0; t < ia.n_tables; ++t) {
    const Table &tb = c->tables[t];
    const bool indexed = t < c->indexes.size() && c->indexes[t].keys != nullptr;
    ia.tab[t] = IngestTable{tb.n_rows, tb.row_base, tb.elem_base, tb.n_fields, indexed ? 1u : 0u};
  }
  return ia;
}

// Device arrays are taken where they are; host arrays are copied into the
// submission scratch first.  Either way the ingest kernels validate, pack and
// count, and one copy brings back what the host needs.
static cc_status submit_impl(cc_ctx *c, const cc_txn *txns, uint64_t n_txns, const cc_op *ops, uint64_t n_ops,
                             const int64_t *op_keys, int scheme, int on_device, uint64_t *batch_id) {
  if (!c || !batch_id) return CC_E_INVAL;
  *batch_id = 0;
  if (scheme < 0 || scheme >= CC_N_SCHEMES) return fail(c, CC_E_INVAL, "unknown scheme");
  if (!c->frozen) return fail(c, CC_E_STATE, "load the tables before submitting a batch");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  if ((n_txns && !txns) || (n_ops && !ops)) return fail(c, CC_E_INVAL, "null array");
  if (n_txns > 0xFFFFFFFFull || n_ops > 0xFFFFFFFFull) return fail(c, CC_E_RANGE, "batch too large");
  if (on_device &&
      (!device_range(c, txns, n_txns * sizeof(cc_txn)) || !device_range(c, ops, n_ops * sizeof(cc_op)) ||
       (op_keys && !device_range(c, op_keys, n_ops * sizeof(int64_t)))))
    return fail(c, CC_E_INVAL, "on_device arrays must lie in device memory of the context's device");
  bool any_index = false;
  for (const DevIndex &x : c->indexes) any_index |= x.keys != nullptr;
  const bool maybe_keyed = op_keys && any_index;
  const bool ordered_scheme = scheme == CC_GACCO || scheme == CC_GPUTX;
  Batch b;
  b.scheme = scheme;
  b.n_txns = n_txns;
  b.n_ops = n_ops;
  if (!c->d_ingest)
    HIP_OR(c, dev_malloc(c, &c->d_ingest, INGEST_N * sizeof(uint64_t) + (PLAN_COUNTS + PLAN_BINS) * sizeof(uint32_t)));
  const uint64_t n_rows = std::max<uint64_t>(c->total_rows, 1);
  if (!c->d_cnt) {
    HIP_OR(c, dev_malloc(c, &c->d_cnt, n_rows * sizeof(uint32_t)));
    HIP_OR(c, hipMemsetAsync(c->d_cnt, 0, n_rows * sizeof(uint32_t), c->stream));
  }
  // scratch: [the host's arrays], keys, candidates, marked rows, owners
  const uint64_t staged = on_device ? 0 : n_ops * sizeof(cc_op) + n_txns * sizeof(cc_txn);
  hipError_t e = need_sub(c, staged + n_ops * 16 + plan_cand_max(n_ops) * 8 + 256);
  if (e == hipSuccess) e = alloc_batch(c, b, maybe_keyed);
  if (e != hipSuccess) return hip_fail(c, e, "batch allocation");
  if (!on_device) {
    cc_op *s_ops = (cc_op *)c->d_sub;
    cc_txn *s_txns = (cc_txn *)(s_ops + n_ops);
    if (staged && staged <= PIN_BYTES) {
      if (n_ops) std::memcpy(c->h_pin, ops, n_ops * sizeof(cc_op));
      if (n_txns) std::memcpy(c->h_pin + n_ops * sizeof(cc_op), txns, n_txns * sizeof(cc_txn));
      e = hipMemcpyAsync(c->d_sub, c->h_pin, staged, hipMemcpyHostToDevice, c->stream);
    } else {
      if (n_ops) e = hipMemcpyAsync(s_ops, ops, n_ops * sizeof(cc_op), hipMemcpyHostToDevice, c->stream);
      if (e == hipSuccess && n_txns)
        e = hipMemcpyAsync(s_txns, txns, n_txns * sizeof(cc_txn), hipMemcpyHostToDevice, c->stream);
    }
    ops = s_ops;
    txns = s_txns;
  }
  if (e == hipSuccess && maybe_keyed && n_ops)
    e = hipMemcpyAsync(b.d_opkeys, op_keys, n_ops * sizeof(int64_t),
                       on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, c->stream);
  IngestArgs ia = ingest_args(c, txns, n_txns, ops, n_ops);
  ia.op_keys = maybe_keyed ? b.d_opkeys : nullptr;
  while (((n_rows - 1) >> ia.row_shift) >= (uint64_t)PLAN_BINS) ++ia.row_shift;
  ia.dops = b.d_ops;
  ia.dtx = b.d_txns;
  ia.meta = maybe_keyed ? b.d_meta : nullptr;
  ia.rows0 = maybe_keyed ? b.d_rows : nullptr;
  ia.out = c->d_ingest;
  ia.cnt = c->d_cnt;
  ia.keys = (uint64_t *)(c->d_sub + staged);
  ia.cand = ia.keys + n_ops;
  ia.rows = (uint32_t *)(ia.cand + plan_cand_max(n_ops));
  ia.owner = ia.rows + n_ops;
  ia.hist = (uint32_t *)(c->d_ingest + INGEST_N);
  if (scheme == CC_OCC) {
    // (with keys too: a batch none of whose ops is on an indexed table is one by row)
    const size_t words = (n_rows + 31) / 32;
    if (e == hipSuccess && !c->d_hot) e = dev_malloc(c, &c->d_hot, words * sizeof(uint32_t), true);
    if (e == hipSuccess) e = hipMemsetAsync(c->d_hot, 0, words * sizeof(uint32_t), c->stream);
    ia.hot_map = c->d_hot;
  }
  uint64_t res[INGEST_N] = {};
  if (e == hipSuccess) e = launch_ingest(c->stream, ia, c->n_cu);
  if (e == hipSuccess && n_ops) e = hipMemsetAsync(b.d_reads, 0, n_ops * sizeof(int64_t), c->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(c->h_pin, c->d_ingest, sizeof res, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e == hipSuccess) std::memcpy(res, c->h_pin, sizeof res);
  auto drop = [&]() {
    free_batch(c, b);
    trim_sub(c);
  };
  if (e != hipSuccess) {
    (void)hipStreamSynchronize(c->stream);
    drop();
    // the counts may be anything now
    (void)hipFree(c->d_cnt);
    c->d_cnt = nullptr;
    return hip_fail(c, e, "batch submission");
  }
  if (res[INGEST_ERR] != ~0ull) {
    drop();
    HIP_OR(c, hipMemsetAsync(c->d_cnt, 0, n_rows * sizeof(uint32_t), c->stream));
    const uint64_t w = res[INGEST_ERR];
    const cc_status code = -(cc_status)(w & 15u);
    std::string msg = ingest_message((uint32_t)((w >> 4) & 0xFFFu));
    if (on_device) msg += " (transaction " + std::to_string(w >> 16) + ")";
    return fail(c, code, msg);
  }
  if (ordered_scheme && res[INGEST_UNORDERED]) {
    drop();
    return fail(c, CC_E_INVAL,
                "CC_GACCO and CC_GPUTX need each transaction's ops after the previous transaction's (first_op "
                "nondecreasing)");
  }
  b.max_ops = (uint32_t)res[INGEST_MAX_OPS];
  b.has_slot = (res[INGEST_KINDS] & 1) != 0;
  b.has_cond = (res[INGEST_KINDS] & 2) != 0;
  b.keyed = res[INGEST_KEYED] != 0;
  if (!b.keyed) {
    b.d_opkeys = nullptr;
    b.d_meta = nullptr;
    b.d_rows = nullptr;
    // (keyed ops learn their rows only when the index is searched, at the run)
    plan_hot_rows(res, c->tables, b, c->n_cu);
  }
  e = alloc_breaks(c, b);
  if (e == hipSuccess && b.eng_default) {
    const hipError_t es = split_batch(c, b, c->d_hot);
    if (es == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      b.eng_default = false;  // no room for its lists
    } else {
      e = es;
    }
  }
  if (e != hipSuccess) {
    drop();
    return hip_fail(c, e, "batch allocation");
  }
  trim_sub(c);
  const uint64_t id = c->next_batch++;
  c->batches[id] = b;
  *batch_id = id;
  return CC_OK;
}

cc_status cc_submit_batch(cc_ctx *c, const cc_txn *txns, uint64_t n_txns, const cc_op *ops, uint64_t n_ops,
                          int scheme, int on_device, uint64_t *batch_id) {
  return submit_impl(c, txns, n_txns, ops, n_ops, nullptr, scheme, on_device, batch_id);
}

cc_status cc_submit_batch_keyed(cc_ctx *c, const cc_txn *txns, uint64_t n_txns, const cc_op *ops, uint64_t n_ops,
                                const int64_t *op_keys, int scheme, int on_device, uint64_t *batch_id) {
  if (!op_keys && n_ops) return fail(c, CC_E_INVAL, "op_keys is NULL");
  return submit_impl(c, txns, n_txns, ops, n_ops, op_keys, scheme, on_device, batch_id);
}

cc_status cc_create_index(cc_ctx *c, uint32_t tid, const int64_t *keys, uint64_t n) {
  if (!c || (!keys && n)) return CC_E_INVAL;
  if (tid >= c->tables.size()) return fail(c, CC_E_RANGE, "unknown table");
  if (n != c->tables[tid].n_rows) return fail(c, CC_E_INVAL, "one key per row of the table");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  cc_status st = freeze(c);
  if (st) return st;
  for (auto &kv : c->batches)
    if (kv.second.keyed) return fail(c, CC_E_STATE, "release the keyed batches before changing an index");
  // sort (key, row) on the host: index construction is load-time work
  std::vector<std::pair<int64_t, uint32_t>> kr(n);
  for (uint64_t i = 0; i < n; ++i) {
    if (keys[i] == INT64_MAX) return fail(c, CC_E_INVAL, "INT64_MAX is reserved (index padding)");
    kr[i] = {keys[i], (uint32_t)i};
  }
  std::sort(kr.begin(), kr.end());
  for (uint64_t i = 1; i < n; ++i)
    if (kr[i].first == kr[i - 1].first) return fail(c, CC_E_INVAL, "index keys must be distinct");
  auto pad16 = [](uint64_t m) { return (m + 15) / 16 * 16; };
  std::vector<int64_t> level0(pad16(std::max<uint64_t>(n, 1)), INT64_MAX);
  std::vector<uint32_t> rows(std::max<uint64_t>(n, 1), 0u);
  for (uint64_t i = 0; i < n; ++i) {
    level0[i] = kr[i].first;
    rows[i] = kr[i].second;
  }
  // upper levels: the largest key of each 16-key node of the level below
  std::vector<int64_t> tree;
  IndexDesc d{};
  d.n = n;
  std::vector<int64_t> cur = level0;
  uint64_t real = n;  // entries of `cur` that are keys (the rest is padding)
  uint32_t levels = 0;
  while (cur.size() > 16) {
    if (levels >= INDEX_MAX_LEVELS) return fail(c, CC_E_RANGE, "index too large");
    const uint64_t nodes = (real + 15) / 16;
    std::vector<int64_t> up(pad16(nodes), INT64_MAX);
    for (uint64_t j = 0; j < nodes; ++j) up[j] = cur[std::min(j * 16 + 15, real - 1)];
    real = nodes;
    ++levels;
    d.level_off[levels] = tree.size();
    tree.insert(tree.end(), up.begin(), up.end());
    cur.swap(up);
  }
  d.levels = levels;
  const Table &t = c->tables[tid];
  d.row_base = t.row_base;
  d.elem_base = t.elem_base;
  d.n_fields = t.n_fields;
  // Build the new index in full before touching the old one: on any failure
  // the table keeps its previous index (or none), on the host and on the
  // device alike.
  DevIndex nx{};
  auto drop = [](DevIndex &x) {
    if (x.keys) (void)hipFree(x.keys);
    if (x.rows) (void)hipFree(x.rows);
    if (x.tree) (void)hipFree(x.tree);
    x = DevIndex{};
  };
  if (!c->d_idx) HIP_OR(c, dev_malloc(c, &c->d_idx, CC_MAX_TABLES * sizeof(IndexDesc)));
  hipError_t e = dev_malloc(c, &nx.keys, level0.size() * sizeof(int64_t));
  if (e == hipSuccess) e = dev_malloc(c, &nx.rows, rows.size() * sizeof(uint32_t));
  if (e == hipSuccess) e = dev_malloc(c, &nx.tree, std::max<size_t>(tree.size(), 1) * sizeof(int64_t));
  if (e == hipSuccess)
    e = hipMemcpyAsync(nx.keys, level0.data(), level0.size() * sizeof(int64_t), hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(nx.rows, rows.data(), rows.size() * sizeof(uint32_t), hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess && !tree.empty())
    e = hipMemcpyAsync(nx.tree, tree.data(), tree.size() * sizeof(int64_t), hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    drop(nx);
    return hip_fail(c, e, "index upload");
  }
  d.keys = nx.keys;
  d.rows = nx.rows;
  d.tree = nx.tree;
  nx.desc = d;
  std::vector<IndexDesc> all(CC_MAX_TABLES, IndexDesc{});
  for (size_t i = 0; i < c->indexes.size(); ++i) all[i] = c->indexes[i].desc;
  all[tid] = d;
  e = hipMemcpyAsync(c->d_idx, all.data(), all.size() * sizeof(IndexDesc), hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    // the device table may be partly written: put the old descriptors back
    // (best effort) and keep the old index
    for (size_t i = 0; i < c->indexes.size(); ++i) all[i] = c->indexes[i].desc;
    if (tid >= c->indexes.size()) all[tid] = IndexDesc{};
    (void)hipMemcpy(c->d_idx, all.data(), all.size() * sizeof(IndexDesc), hipMemcpyHostToDevice);
    drop(nx);
    return hip_fail(c, e, "index descriptor upload");
  }
  if (c->indexes.size() < c->tables.size()) c->indexes.resize(c->tables.size());
  drop(c->indexes[tid]);
  c->indexes[tid] = nx;
  return CC_OK;
}

cc_status cc_engine_plan(cc_ctx *c, uint64_t batch_id, uint32_t *rows, uint32_t *n_rows, uint64_t *n_txns,
                         int *by_default) {
  if (!c || !rows || !n_rows || !n_txns || !by_default) return CC_E_INVAL;
  auto it = c->batches.find(batch_id);
  if (it == c->batches.end()) return fail(c, CC_E_NOBATCH, "unknown batch");
  Batch &b = it->second;
  static_assert(CC_ENGINE_MAX_ROWS == ENG_MAX, "engine rows");
  for (uint32_t i = 0; i < (uint32_t)ENG_MAX; ++i) rows[i] = i < b.eng.n_rows ? b.eng.row[i] : 0u;
  *n_rows = b.eng.n_rows;
  *n_txns = 0;
  if (b.eng.n_rows && b.plan_txns == ~0ull) {
    if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
    uint32_t n_eng = 0;
    HIP_OR(c, need_sub(c, split_scratch_words(b.n_txns) * sizeof(uint32_t)));
    uint32_t *w = (uint32_t *)c->d_sub;
    HIP_OR(c, launch_split(c->stream, b.d_ops, b.d_txns, b.n_txns, b.eng, nullptr, w, nullptr, nullptr, c->n_cu));
    HIP_OR(c, hipMemcpyAsync(&n_eng, w + 2 + b.n_txns, sizeof n_eng, hipMemcpyDeviceToHost, c->stream));
    HIP_OR(c, hipStreamSynchronize(c->stream));
    trim_sub(c);
    b.plan_txns = n_eng;
  }
  if (b.eng.n_rows) *n_txns = b.plan_txns;
  *by_default = b.eng_default ? 1 : 0;
  return CC_OK;
}

cc_status cc_fetch_rows(cc_ctx *c, uint64_t batch_id, uint32_t *rows) {
  if (!c || !rows) return CC_E_INVAL;
  auto it = c->batches.find(batch_id);
  if (it == c->batches.end()) return fail(c, CC_E_NOBATCH, "unknown batch");
  Batch &b = it->second;
  if (!b.keyed) return fail(c, CC_E_STATE, "the batch has no keyed operations");
  if (!b.ran) return fail(c, CC_E_STATE, "batch has not been run");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  if (b.n_ops) HIP_OR(c, hipMemcpy(rows, b.d_rows, b.n_ops * sizeof(uint32_t), hipMemcpyDeviceToHost));
  return CC_OK;
}

cc_status cc_check_run_params(int scheme, const cc_run_params *pp) {
  return check_run_params(nullptr, scheme, pp ? *pp : cc_run_params{});
}

}  // extern "C"

// One run of a batch whose parameters have been checked (cc_run, and
// cc_run_static with a batch that lives in the static scratch).  host_stats:
// copy the outcomes back for the latency percentiles.
static cc_status run_batch(cc_ctx *c, Batch &b, const cc_run_params &p, bool host_stats) {
  if (p.mode == CC_MODE_SERVE && b.n_txns && !b.d_arrival)
    return fail(c, CC_E_STATE, "CC_MODE_SERVE needs cc_set_arrivals first");
  // contention of the batch: the share of transactions that write its most
  // written row (unknown: treated as contended)
  double hot_share = 1.0;
  bool no_hot_row = false, contended = true;
  // OCC's hot-row engine (plain mode only: it knows no arrivals).  It has the
  // scope of the launch shapes of at most 4 ops per lane (64 lanes unless the
  // caller chose)
  const uint32_t eng_lanes = p.lanes_per_txn ? p.lanes_per_txn : 64;
  const bool eng_fits = (b.max_ops + eng_lanes - 1) / eng_lanes <= 4;
  bool use_eng = b.scheme == CC_OCC && p.mode == CC_MODE_PLAIN && !(p.flags & CC_RUN_LATCH) && eng_fits &&
                       b.n_txns &&
                       ((p.flags & CC_RUN_HOT_ENGINE) ? b.eng.n_rows || b.eng_default
                                                      : !(p.flags & CC_RUN_NO_HOT_ENGINE) && b.eng_default);
  if (use_eng) {
    if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
    hipError_t e = split_batch(c, b, nullptr);
    if (e == hipSuccess) e = need_sub(c, engine_scratch_bytes(b.n_eng_ops, b.has_slot || b.has_cond, b.has_slot));
    if (e != hipSuccess && (e != hipErrorOutOfMemory || (p.flags & CC_RUN_HOT_ENGINE)))
      return hip_fail(c, e, "hot-row engine");
    if (e != hipSuccess) {
      (void)hipGetLastError();  // no room for its lists: the transaction kernel needs none
      use_eng = false;
    }
  }
  uint32_t lanes = 0, wpw = 0;
  int grid = 0;
  auto choose_shape = [&]() {
    hot_share = b.shape_known && b.n_txns ? (double)b.shape_writes / (double)b.n_txns : 1.0;
    // (after the engine by the hot-row map no two transactions write one row)
    no_hot_row = hot_share < 0.001 || (use_eng && b.eng_default);
    contended = !no_hot_row && hot_share >= 0.02;
    lanes = p.lanes_per_txn;
    wpw = p.waves_per_wg;
    grid = (int)p.grid;
    if (lanes == 0 && p.mode == CC_MODE_PLAIN && b.scheme != CC_GACCO && b.scheme != CC_GPUTX) {
      const Shape sh = plain_shape(b.scheme, b.max_ops, b.shape_known, no_hot_row ? 0.0 : hot_share,
                                   use_eng && b.eng_default ? b.rest_clash : b.clash, c->n_cu);
      lanes = sh.lanes;
      if (wpw == 0) {
        wpw = sh.waves;
        if (grid == 0) grid = sh.grid;
      } else {
        // the caller's wavefronts, with as many lanes as they need to exist
        while (lanes < 64 && shape_exists(lanes, b.max_ops, wpw) != hipSuccess) lanes *= 4;
      }
    } else if (lanes == 0) {
      if (no_hot_row && b.max_ops <= 64 && b.scheme != CC_GACCO && b.scheme != CC_GPUTX) {
        // nothing to wait for: 4 lanes per transaction, 4 wavefronts per
        // workgroup (4096 transactions in flight at one workgroup per CU)
        lanes = 4;
        if (wpw == 0) wpw = 4;
      } else {
        lanes = 1;
        while (lanes < 64 && lanes < b.max_ops) lanes *= 4;
      }
    }
    if (wpw == 0) wpw = 1;
  };
  choose_shape();
  if ((p.flags & CC_RUN_HOT_ENGINE) && !eng_fits)
    return fail(c, CC_E_INVAL, "CC_RUN_HOT_ENGINE needs at most 4 ops per lane");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  if (b.scheme == CC_GACCO) return run_gacco(c, b, p, lanes, wpw);
  if (b.scheme == CC_GPUTX) return run_gputx(c, b, p, lanes, wpw);

  RunArgs a{};
  a.ops = b.d_ops;
  a.txns = b.d_txns;
  a.n_txns = b.n_txns;
  a.data = c->d_data;
  a.words = c->d_words;
  if (b.scheme == CC_MVCC && !c->d_aux) {
    HIP_OR(c, dev_malloc(c, &c->d_aux, std::max<uint64_t>(c->total_rows, 1) * sizeof(uint64_t)));
  }
  a.aux = c->d_aux;
  if (b.scheme == CC_MVCC) {
    // the version arena: one slot per op of the batch, or, when serving with
    // a cap, hbm_cap_bytes / 32 slots, reused as a ring; at least 1024 slots,
    // more than one transaction's writes (256), so that no commit's slots wrap
    // onto each other
    const uint64_t slots = (p.mode == CC_MODE_SERVE && p.hbm_cap_bytes)
                               ? std::max<uint64_t>(p.hbm_cap_bytes / 32, 1024)
                               : std::max<uint64_t>(b.n_ops, 1024);
    if (!b.d_nodes || b.node_slots != slots) {
      if (b.d_nodes) (void)hipFree(b.d_nodes);
      b.d_nodes = nullptr;
      b.node_slots = 0;
      if (b.epoch_graph) {
        // a captured epoch holds the old arena's address
        (void)hipGraphExecDestroy(b.epoch_graph);
        b.epoch_graph = nullptr;
      }
      const uint64_t bytes = 32 + slots * 4 * sizeof(uint64_t);
      HIP_OR(c, dev_malloc(c, &b.d_nodes, bytes));
      HIP_OR(c, hipMemsetAsync(b.d_nodes, 0, bytes, c->stream));  // tags 0 (lap 0), ring counter 0
      b.node_slots = slots;
    }
  }
  a.nodes = b.d_nodes ? b.d_nodes + 4 : nullptr;
  a.node_ring = b.d_nodes;
  a.n_nodes = b.node_slots;
  // a slot for every op: op i keeps slot i and no slot is reused in the run
  a.node_reuse = b.node_slots < b.n_ops ? 1u : 0u;
  a.out = b.d_out;
  a.reads = b.d_reads;
  a.ctl = c->d_ctl;
  a.max_attempts = p.max_attempts ? p.max_attempts : (1ull << 24);
  const uint64_t backoff_ns = p.backoff_ns ? p.backoff_ns : 200;
  a.backoff_ticks = (uint32_t)std::max<uint64_t>(1, backoff_ns * c->wallclock_khz / 1000000ull);
  a.ns_per_tick_q16 = (uint32_t)((1000000ull << 16) / c->wallclock_khz);
  a.has_slot = b.has_slot ? 1u : 0u;
  a.eager_install = (p.flags & CC_RUN_EAGER_INSTALL) ? 1u : 0u;
  a.hot0 = b.n_hot ? b.hot_rows[0] : ~0u;
  a.wait_blocker = (p.flags & CC_RUN_WAIT_BLOCKER) ? 1u : 0u;
  a.poll_ticks = 2 * a.backoff_ticks;
  a.jitter_ticks = 2 * a.backoff_ticks;
  a.wait_max_ticks = 256ull * a.backoff_ticks;
  // 128 bases at most, 256 with a hot row: the last transactions of a batch otherwise wait several
  // times as long as it ran (262,144 x 16 ops, Zipf 0.6, a tenth writes, 1024
  // in flight: OCC 2.30 -> 1.53 ms, TicToc 2.39 -> 1.62; Zipf 0.8, 256 in
  // flight: OCC 14.9 -> 12.7).  More where nearly all of a batch meets (16 ops,
  // 9 of 10 writes, Zipf 0.99 on 154,835 rows: 2PL 46.6 ms at 128, 38.1 at 4096; OCC
  // 47.5 at 128, 46.8 at 1024, 48.7 at 4096), where that goes for most operations of
  // a long transaction, whose attempts take as long (65-256 ops, a tenth writes,
  // uniform on 50,000 rows: OCC 3.5 ms at 128, 2.9 at 1024, 3.4 at 4096; 2PL 3.7, 3.1,
  // 3.4; on 5,000 rows 2PL 15.2, 14.8, 14.1; on 200,000 OCC 0.81, 0.92, 1.36; half
  // writes on 100,000 OCC 1.24, 1.27; not TO and MVCC, 1.4 and 1.6 ms on 50,000), and
  // where thousands in flight wait for a hot row (4096, Zipf 0.8: MVCC 45 ms at
  // 128, 34 at 4096).
  auto choose_retries = [&]() {
    a.precheck = (p.flags & CC_RUN_PRECHECK) ? 2u : ((p.flags & CC_RUN_NO_PRECHECK) ? 0u : (contended ? 1u : 0u));
    const double in_flight = (double)(grid ? grid : c->n_cu) * wpw * (64.0 / lanes);
    if (p.mode != CC_MODE_PLAIN || (in_flight > 1024 && (!b.shape_known || contended))) a.backoff_cap = 12;
    else if (!b.shape_known) a.backoff_cap = in_flight <= 256 ? 7u : 10u;
    else if (b.meet > 0.1) a.backoff_cap = b.scheme == CC_2PL_NW || b.scheme == CC_2PL_WD ? 12u : 10u;
    else if (contended) a.backoff_cap = 8;
    else if (b.clash * (double)b.n_ops > 4.0 * (double)b.n_txns && b.scheme != CC_TO && b.scheme != CC_MVCC)
      a.backoff_cap = b.clash > 0.1 && (b.scheme == CC_2PL_NW || b.scheme == CC_2PL_WD) ? 12u : 10u;
    else a.backoff_cap = 7;
  };
  choose_retries();
  a.n_late = 0;
  if (b.scheme == CC_OCC && (p.flags & CC_RUN_HOT_LAST) && b.hot_known) {
    a.n_late = b.n_hot;
    for (uint32_t i = 0; i < b.n_hot; ++i) a.late[i] = b.hot_rows[i];
  }
  a.wd_wait_limit = 64;
  if (p.flags & CC_RUN_LATCH) {
    if (!c->d_latch) {
      // latches are free between critical sections, so they are cleared once
      HIP_OR(c, dev_malloc(c, &c->d_latch, std::max<uint64_t>(c->total_rows, 1) * sizeof(uint32_t)));
      HIP_OR(c, hipMemsetAsync(c->d_latch, 0, std::max<uint64_t>(c->total_rows, 1) * sizeof(uint32_t), c->stream));
    }
    a.latch = c->d_latch;
  }

  const uint32_t defer = p.defer_after ? p.defer_after : (p.mode == CC_MODE_SERVE ? 256 : 16);
  a.pass = 0;
  a.list = nullptr;
  if (p.mode == CC_MODE_SERVE) {
    a.arrival = b.d_arrival;
    a.budget_cap = p.hbm_cap_bytes;
    a.bytes_per_op = CC_SERVE_BYTES_PER_OP;
  }

  HIP_OR(c, hipEventRecord(c->ev[0], c->stream));
  HIP_OR(c, launch_init(c->stream, c->d_words, c->total_rows, c->d_aux, b.scheme == CC_MVCC ? c->total_rows : 0,
                        b.d_out, b.n_txns, c->d_ctl, c->d_lat, p.ts_start));
  float ms_index = 0;
  if (b.keyed) {
    cc_status st = resolve_keys(c, b, p, &ms_index);
    if (st) return st;
    // the rows are known now: counted once a batch, which pays where not all of
    // it is in flight at once (262,144 x 16 ops on 1M rows: 0.1 ms, and the
    // kernel's 1.48 ms become 0.75)
    if (!b.shape_known && p.mode == CC_MODE_PLAIN && p.lanes_per_txn == 0 && b.n_txns > 4096) {
      st = count_keyed(c, b);
      if (st) return st;
      choose_shape();
      choose_retries();
    }
  }
  Ctl h{};
  const RunTail *tail = (const RunTail *)c->h_pin;
  // the latencies of a small batch are looked at behind every pass, which costs
  // less than a synchronisation of its own behind the last
  const bool lat_early = host_stats && b.n_txns && b.n_txns <= (uint64_t)LAT_SMALL;
  const int64_t *lat_arrival = p.mode == CC_MODE_SERVE && b.d_arrival ? b.d_arrival + b.n_txns : nullptr;
  bool have_tail = false, have_latency = false;  // the last tail is the run's, and so are its latencies
  double kernel_ms = 0;
  uint32_t passes = 0, epochs = 0;
  int first_grid = 0;
  bool epoch_limit = false;
  const bool strict = (p.flags & CC_RUN_STRICT_FENCES) != 0;
  const bool latch = (p.flags & CC_RUN_LATCH) != 0;

  // Plain passes over the pending transactions: each pass runs 8x fewer
  // workgroups than the last, down to a single wavefront that never defers,
  // so every transaction eventually runs without concurrency.
  auto plain_passes = [&](int grid, uint32_t waves, bool first_is_all) -> cc_status {
    bool all = first_is_all;
    for (;;) {
      if (!all) {
        HIP_OR(c, launch_compact(c->stream, b.d_out, b.n_txns, a.max_attempts, b.d_list, c->d_ctl));
        HIP_OR(c, queue_tail(c, b, nullptr, false));
        HIP_OR(c, hipStreamSynchronize(c->stream));
        h = tail->ctl;
        a.list = b.d_list;
        a.n_txns = h.pending_n;
        a.pass = 1;  // attempt counts continue from the outcome records
        a.n_from_ctl = 0;
        a.arrival = nullptr;  // deferred transactions have all arrived
        a.budget_cap = 0;
      }
      const bool last = grid == 1 && waves == 1;
      a.defer_after = last ? 0u : defer;
      HIP_OR(c, hipEventRecord(c->ev[1], c->stream));
      int grid_used = 0;
      hipError_t e = launch_txn(c->stream, b.scheme, (int)lanes, (int)b.max_ops, (int)waves, grid, strict, latch, a,
                                c->n_cu, &grid_used);
      if (e != hipSuccess) return launch_error(c, e);
      HIP_OR(c, hipEventRecord(c->ev[2], c->stream));
      HIP_OR(c, queue_tail(c, b, lat_arrival, lat_early));
      HIP_OR(c, hipStreamSynchronize(c->stream));
      float ms = 0;
      HIP_OR(c, hipEventElapsedTime(&ms, c->ev[1], c->ev[2]));
      kernel_ms += ms;
      if (first_grid == 0) first_grid = grid_used;
      ++passes;
      all = false;
      h = tail->ctl;
      have_tail = true;
      have_latency = lat_early;
      // a stuck latch stopped the run (reported below)
      if (h.stats[DS_COMMITTED] + h.stats[DS_GAVE_UP] >= b.n_txns || last || h.stop) return CC_OK;
      grid = std::max(1, grid_used / 8);
      if (grid == 1) waves = 1;
    }
  };

  if (b.n_txns && p.mode == CC_MODE_EPOCH) {
    // Epochs: every pending transaction gets defer_after (default 1) attempts,
    // aborted ones wait for the next epoch.  One epoch = [reset claim counter,
    // list the pending transactions, persistent transaction kernel over that
    // list]; EPOCHS_PER_GRAPH epochs are captured once as a hipGraph and the
    // graph is replayed until nothing is pending.  The kernel reads the
    // pending count from the control block, so the graph's arguments are fixed.
    // A replay that commits almost nothing (symmetric conflicts repeating
    // epoch after epoch) hands the rest to the plain passes, which always
    // finish.
    constexpr uint32_t EPOCHS_PER_GRAPH = 4;
    const uint32_t max_epochs = p.max_epochs ? p.max_epochs : (1u << 20);
    a.defer_after = p.defer_after ? p.defer_after : 1;
    a.pass = 1;
    a.list = b.d_list;
    a.n_from_ctl = 1;
    const uint64_t key[4] = {(uint64_t)lanes | ((uint64_t)wpw << 8) | ((uint64_t)p.grid << 16),
                             (uint64_t)p.flags | ((uint64_t)a.defer_after << 32), a.max_attempts,
                             (uint64_t)a.backoff_ticks | ((uint64_t)p.ts_start << 32)};
    if (!b.epoch_graph || std::memcmp(key, b.epoch_key, sizeof key) != 0) {
      if (b.epoch_graph) (void)hipGraphExecDestroy(b.epoch_graph);
      b.epoch_graph = nullptr;
      hipGraph_t g = nullptr;
      HIP_OR(c, hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
      hipError_t e = hipSuccess;
      int grid_used = 0;
      for (uint32_t i = 0; i < EPOCHS_PER_GRAPH && e == hipSuccess; ++i) {
        e = launch_compact(c->stream, b.d_out, b.n_txns, a.max_attempts, b.d_list, c->d_ctl);
        if (e == hipSuccess)
          e = launch_txn(c->stream, b.scheme, (int)lanes, (int)b.max_ops, (int)wpw, (int)p.grid, strict, latch, a,
                         c->n_cu, &grid_used);
      }
      const hipError_t e2 = hipStreamEndCapture(c->stream, &g);
      if (e != hipSuccess) {
        if (e2 == hipSuccess && g) (void)hipGraphDestroy(g);
        return launch_error(c, e);
      }
      if (e2 != hipSuccess) return hip_fail(c, e2, "hipStreamEndCapture");
      e = hipGraphInstantiate(&b.epoch_graph, g, nullptr, nullptr, 0);
      (void)hipGraphDestroy(g);
      if (e != hipSuccess) {
        b.epoch_graph = nullptr;
        return hip_fail(c, e, "hipGraphInstantiate");
      }
      std::memcpy(b.epoch_key, key, sizeof key);
      b.epoch_grid = grid_used;
    }
    first_grid = b.epoch_grid;
    uint64_t done_before = 0;
    for (;;) {
      HIP_OR(c, hipEventRecord(c->ev[1], c->stream));
      HIP_OR(c, hipGraphLaunch(b.epoch_graph, c->stream));
      HIP_OR(c, hipEventRecord(c->ev[2], c->stream));
      HIP_OR(c, queue_tail(c, b, nullptr, false));
      HIP_OR(c, hipStreamSynchronize(c->stream));
      float ms = 0;
      HIP_OR(c, hipEventElapsedTime(&ms, c->ev[1], c->ev[2]));
      kernel_ms += ms;
      epochs += EPOCHS_PER_GRAPH;
      h = tail->ctl;
      have_tail = true;
      const uint64_t done = h.stats[DS_COMMITTED] + h.stats[DS_GAVE_UP];
      if (done >= b.n_txns || h.stop) break;
      if (epochs >= max_epochs) {
        epoch_limit = true;
        break;
      }
      // fewer than 1/256 of the pending transactions committed in four epochs:
      // the epochs are stalled on conflicts; finish with the plain passes
      const uint64_t pending = b.n_txns - done;
      if ((done - done_before) * 256 < pending || done == done_before) {
        // continue as a plain run would: same grid, then 8x smaller passes
        cc_status st = plain_passes(b.epoch_grid, wpw, false);
        if (st) return st;
        break;
      }
      done_before = done;
    }
  } else if (b.n_txns) {
    if (use_eng) {
      // OCC's hot-row engine: the transactions on the batch's hot rows run
      // first, in their order; the rest then run as usual
      HIP_OR(c, hipEventRecord(c->ev[4], c->stream));
      HIP_OR(c, launch_engine(c->stream, strict, a, b.d_eng_desc, b.n_eng_txns, b.n_eng_ops, c->total_cells,
                              b.has_slot || b.has_cond, b.has_slot, c->d_sub, p.ts_start, wait_limit_ticks(c, p),
                              c->n_cu));
      HIP_OR(c, hipEventRecord(c->ev[5], c->stream));
      HIP_OR(c, hipEventRecord(c->ev[2], c->stream));
      ++passes;
      a.list = b.d_part + b.n_eng_txns;
      a.n_txns = b.n_txns - b.n_eng_txns;
    }
    if (a.n_txns) {
      cc_status st = plain_passes(grid, wpw, true);
      if (st) return st;
    }
  }
  // the run ends with its last kernel (ev[2]); nothing to run ends with its initialisation
  const bool want_latency = host_stats && b.n_txns && !have_latency;
  if (!passes && !epochs) HIP_OR(c, hipEventRecord(c->ev[2], c->stream));
  if (!have_tail || want_latency) {
    HIP_OR(c, queue_tail(c, b, lat_arrival, want_latency));
    HIP_OR(c, hipStreamSynchronize(c->stream));
    h = tail->ctl;
  }
  float ms_run = 0, engine_ms = 0;
  HIP_OR(c, hipEventElapsedTime(&ms_run, c->ev[0], c->ev[2]));
  if (use_eng) HIP_OR(c, hipEventElapsedTime(&engine_ms, c->ev[4], c->ev[5]));
  kernel_ms += engine_ms;
  std::memset(b.stats, 0, sizeof(b.stats));
  b.stats[CC_STAT_COMMITTED] = h.stats[DS_COMMITTED];
  b.stats[CC_STAT_ATTEMPTS] = h.stats[DS_ATTEMPTS];
  b.stats[CC_STAT_ABORT_LOCK] = h.stats[DS_ABORT_LOCK];
  b.stats[CC_STAT_ABORT_VALID] = h.stats[DS_ABORT_VALID];
  b.stats[CC_STAT_KERNEL_NS] = (uint64_t)(kernel_ms * 1e6);
  b.stats[CC_STAT_RUN_NS] = (uint64_t)((double)ms_run * 1e6);
  b.stats[CC_STAT_TICKETS] = h.ticket - p.ts_start;
  b.stats[CC_STAT_MAX_ATTEMPTS] = h.stats[DS_MAX_ATTEMPTS];
  b.stats[CC_STAT_PASSES] = passes;
  b.stats[CC_STAT_DEFERRED] = h.stats[DS_DEFERRED];
  b.stats[CC_STAT_ENGINE_TXNS] = use_eng ? b.n_eng_txns : 0;
  b.stats[CC_STAT_ENGINE_ROWS] = use_eng ? b.eng.n_rows : 0;
  b.stats[CC_STAT_ENGINE_NS] = (uint64_t)(engine_ms * 1e6);
  b.stats[CC_STAT_ENGINE_WAITS] = use_eng ? b.eng_behind : 0;
  b.stats[CC_STAT_GRID] = (uint64_t)first_grid;
  b.stats[CC_STAT_EPOCHS] = epochs;
  const double ns_per_tick = 1e6 / (double)c->wallclock_khz;
  b.stats[CC_STAT_T_USEFUL_NS] = (uint64_t)((double)h.stats[DS_T_USEFUL] * ns_per_tick);
  b.stats[CC_STAT_T_ABORT_NS] = (uint64_t)((double)h.stats[DS_T_ABORT] * ns_per_tick);
  b.stats[CC_STAT_T_WAIT_NS] = (uint64_t)((double)h.stats[DS_T_WAIT] * ns_per_tick);
  b.stats[CC_STAT_GAVE_UP] = h.stats[DS_GAVE_UP];
  b.stats[CC_STAT_ADMIT_WAITS] = h.stats[DS_ADMIT_WAITS];
  b.stats[CC_STAT_WD_WAITS] = h.stats[DS_WD_WAITS];
  b.stats[CC_STAT_HOT_ACQ] = h.stats[DS_HOT_ACQ];
  b.stats[CC_STAT_HOT_FAILED] = h.stats[DS_HOT_FAILED];
  b.stats[CC_STAT_HOT_HOLD_NS] = (uint64_t)((double)h.stats[DS_HOT_HOLD] * ns_per_tick);
  b.stats[CC_STAT_HOT_WRITES] = b.hot_writes;
  if (use_eng && (b.eng_default || b.eng.row[0] == a.hot0)) {
    // every write of the most written row is in the engine, whose rows are its
    // own as long as it runs
    b.stats[CC_STAT_HOT_ACQ] += b.hot_writes;
    b.stats[CC_STAT_HOT_HOLD_NS] += b.stats[CC_STAT_ENGINE_NS];
  }
  b.stats[CC_STAT_BLOCKED_WAITS] = h.stats[DS_BLOCKED_WAITS];
  b.stats[CC_STAT_VERSION_SLOTS] = b.node_slots;
  b.stats[CC_STAT_VERSION_MISSES] = h.stats[DS_VERSION_MISS];
  for (int i = 0; i < 4; ++i)
    b.stats[CC_STAT_OCC_R1_NS + i] = (uint64_t)((double)h.stats[DS_R1 + i] * ns_per_tick);
  b.stats[CC_STAT_INDEX_NS] = (uint64_t)((double)ms_index * 1e6);
  b.ran = true;
  if (b.n_txns && host_stats) {
    const cc_status st = take_latency(c, b, p.mode == CC_MODE_SERVE);
    if (st) return st;
  }
  if (h.stop && use_eng && !h.stats[DS_LATCH_STUCK])
    return fail(c, CC_E_LIVELOCK, "the hot-row engine stopped: a value was not resolved within the wait limit");
  if (h.stats[DS_LATCH_STUCK] || h.stop)
    return fail(c, CC_E_LIVELOCK, "a row latch was not obtained within the spin limit; table contents are undefined");
  if (h.stats[DS_TS_OVERFLOW]) return fail(c, CC_E_TS_OVERFLOW, "timestamp overflow during the run");
  if (epoch_limit) return fail(c, CC_E_LIVELOCK, "max_epochs reached with transactions pending");
  if (h.stats[DS_COMMITTED] != b.n_txns) {
    char msg[160];
    std::snprintf(msg, sizeof msg, "%llu of %llu transactions committed (attempt limit reached)",
                  (unsigned long long)h.stats[DS_COMMITTED], (unsigned long long)b.n_txns);
    return fail(c, CC_E_LIVELOCK, msg);
  }
  return CC_OK;
}

extern "C" {

cc_status cc_run(cc_ctx *c, uint64_t batch_id, const cc_run_params *pp) {
  if (!c) return CC_E_INVAL;
  auto it = c->batches.find(batch_id);
  if (it == c->batches.end()) return fail(c, CC_E_NOBATCH, "unknown batch");
  Batch &b = it->second;
  cc_run_params p{};
  if (pp) p = *pp;
  const cc_status pst = check_run_params(c, b.scheme, p);
  if (pst) return pst;
  return run_batch(c, b, p, true);
}

cc_status cc_run_static(cc_ctx *c, const cc_txn *txns, uint64_t n_txns, const cc_op *ops, uint64_t n_ops, int scheme,
                        const cc_run_params *pp, cc_outcome *per_txn, int64_t *per_op_read, uint64_t *counters,
                        uint32_t n_counters) {
  if (!c) return CC_E_INVAL;
  if ((n_txns && (!txns || !per_txn)) || (n_ops && (!ops || !per_op_read)) || (n_counters && !counters))
    return fail(c, CC_E_INVAL, "null array");
  if (scheme != CC_OCC && scheme != CC_2PL_NW && scheme != CC_2PL_WD && scheme != CC_TO && scheme != CC_TICTOC)
    return fail(c, CC_E_INVAL, "cc_run_static runs CC_OCC, CC_2PL_NW, CC_2PL_WD, CC_TO and CC_TICTOC");
  cc_run_params p{};
  if (pp) p = *pp;
  const cc_status pst = check_run_params(c, scheme, p);
  if (pst) return pst;
  if (p.mode != CC_MODE_PLAIN) return fail(c, CC_E_INVAL, "cc_run_static runs in CC_MODE_PLAIN only");
  if (p.flags & CC_RUN_LATCH) return fail(c, CC_E_INVAL, "cc_run_static does not take CC_RUN_LATCH");
  if (n_txns > CC_STATIC_MAX_TXNS || n_ops > CC_STATIC_MAX_OPS)
    return fail(c, CC_E_RANGE, "batch larger than the static scratch (CC_STATIC_MAX_TXNS, CC_STATIC_MAX_OPS)");
  if (!c->frozen) return fail(c, CC_E_STATE, "load the tables before running a batch");
  if (!c->d_static) return fail(c, CC_E_STATE, "no static scratch on this context's device");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  if (!device_range(c, txns, n_txns * sizeof(cc_txn)) || !device_range(c, ops, n_ops * sizeof(cc_op)) ||
      !device_range(c, per_txn, n_txns * sizeof(cc_outcome)) || !device_range(c, per_op_read, n_ops * sizeof(int64_t)))
    return fail(c, CC_E_INVAL, "arrays must lie in device memory of the context's device");
  unsigned char *sc = c->d_static;
  Batch b;
  b.scheme = scheme;
  b.n_txns = n_txns;
  b.n_ops = n_ops;
  b.d_ops = (DevOp *)(sc + STATIC_OFF_OPS);
  b.d_txns = (DevTxn *)(sc + STATIC_OFF_TXNS);
  b.d_list = (uint32_t *)(sc + STATIC_OFF_LIST);
  b.d_out = (DevOutcome *)per_txn;
  b.d_reads = per_op_read;
  IngestArgs ia = ingest_args(c, txns, n_txns, ops, n_ops);
  ia.dops = b.d_ops;
  ia.dtx = b.d_txns;
  ia.owner = (uint32_t *)(sc + STATIC_OFF_OWNER);
  ia.out = (uint64_t *)(sc + STATIC_OFF_INGEST);
  uint64_t res[INGEST_N] = {};
  hipError_t e = launch_ingest(c->stream, ia, c->n_cu);
  // the rows' writes, for the launch shape (the owner words are free again)
  if (e == hipSuccess && c->d_cnt && n_ops)
    e = launch_count_writes(c->stream, b.d_ops, n_ops, c->d_cnt, ia.owner, ia.out + INGEST_TOP, ia.out + INGEST_ERR,
                            c->n_cu);
  if (e == hipSuccess) e = launch_fill_zero(c->stream, per_op_read, n_ops);
  if (e == hipSuccess) e = hipMemcpyAsync(res, ia.out, sizeof res, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    (void)hipFree(c->d_cnt);  // the counts may be anything now
    c->d_cnt = nullptr;
    return hip_fail(c, e, "batch ingest");
  }
  if (res[INGEST_ERR] != ~0ull) {
    const uint64_t w = res[INGEST_ERR];
    const cc_status code = -(cc_status)(w & 15u);
    return fail(c, code, std::string(ingest_message((uint32_t)((w >> 4) & 0xFFFu))) + " (transaction " +
                             std::to_string(w >> 16) + ")");
  }
  b.max_ops = (uint32_t)res[INGEST_MAX_OPS];
  b.has_slot = (res[INGEST_KINDS] & 1) != 0;
  if (c->d_cnt && n_txns) set_conflicts(b, res[INGEST_TOP], res[INGEST_PAIRS], res[INGEST_WRITES]);
  const cc_status st = run_batch(c, b, p, false);
  for (uint32_t i = 0; i < n_counters; ++i) counters[i] = i < CC_N_STATS ? b.stats[i] : 0;
  return st;
}

cc_status cc_fetch_outcomes(cc_ctx *c, uint64_t batch_id, cc_outcome *per_txn, int64_t *per_op, int on_device) {
  if (!c) return CC_E_INVAL;
  auto it = c->batches.find(batch_id);
  if (it == c->batches.end()) return fail(c, CC_E_NOBATCH, "unknown batch");
  Batch &b = it->second;
  if (!b.ran) return fail(c, CC_E_STATE, "batch has not been run");
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  const hipMemcpyKind k = on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  if (per_txn && b.n_txns) HIP_OR(c, hipMemcpyAsync(per_txn, b.d_out, b.n_txns * sizeof(cc_outcome), k, c->stream));
  if (per_op && b.n_ops) HIP_OR(c, hipMemcpyAsync(per_op, b.d_reads, b.n_ops * sizeof(int64_t), k, c->stream));
  HIP_OR(c, hipStreamSynchronize(c->stream));
  return CC_OK;
}

cc_status cc_set_arrivals(cc_ctx *c, uint64_t batch_id, const int64_t *arrival_ns, uint64_t n) {
  if (!c || (n && !arrival_ns)) return CC_E_INVAL;
  auto it = c->batches.find(batch_id);
  if (it == c->batches.end()) return fail(c, CC_E_NOBATCH, "unknown batch");
  Batch &b = it->second;
  if (n != b.n_txns) return fail(c, CC_E_INVAL, "one arrival time per transaction");
  std::vector<int64_t> ticks(std::max<uint64_t>(2 * n, 1), 0);
  for (uint64_t t = 0; t < n; ++t) {
    if (arrival_ns[t] < 0 || (t && arrival_ns[t] < arrival_ns[t - 1]))
      return fail(c, CC_E_INVAL, "arrival times must be non-negative and non-decreasing");
    ticks[t] = (int64_t)((double)arrival_ns[t] * (double)c->wallclock_khz / 1e6);
    ticks[n + t] = arrival_ns[t];
  }
  if (!activate(c)) return fail(c, CC_E_HIP, "hipSetDevice failed");
  if (!b.d_arrival) HIP_OR(c, dev_malloc(c, &b.d_arrival, ticks.size() * sizeof(int64_t)));
  HIP_OR(c, hipMemcpyAsync(b.d_arrival, ticks.data(), 2 * n * sizeof(int64_t), hipMemcpyHostToDevice, c->stream));
  HIP_OR(c, hipStreamSynchronize(c->stream));
  b.arrival_ns.assign(arrival_ns, arrival_ns + n);
  return CC_OK;
}

cc_status cc_stats(cc_ctx *c, uint64_t batch_id, uint64_t *counters, uint32_t n) {
  if (!c || (!counters && n)) return CC_E_INVAL;
  auto it = c->batches.find(batch_id);
  if (it == c->batches.end()) return fail(c, CC_E_NOBATCH, "unknown batch");
  for (uint32_t i = 0; i < n && i < CC_N_STATS; ++i) counters[i] = it->second.stats[i];
  return CC_OK;
}

cc_status cc_release_batch(cc_ctx *c, uint64_t batch_id) {
  if (!c) return CC_E_INVAL;
  auto it = c->batches.find(batch_id);
  if (it == c->batches.end()) return fail(c, CC_E_NOBATCH, "unknown batch");
  activate(c);
  (void)hipStreamSynchronize(c->stream);
  free_batch(c, it->second);
  c->batches.erase(it);
  trim_sub(c);
  return CC_OK;
}

}  // extern "C"
