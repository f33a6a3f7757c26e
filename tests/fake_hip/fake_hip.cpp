// A HIP runtime of host memory, for tests of the engine's host side without a
// GPU: what it allocates, copies and gives back, and what it does when one of
// those fails.  Loaded before libcc.so with RTLD_GLOBAL, so that the library's
// HIP calls land here (tests/test_host_memory.py).
//
// "Device" memory is anonymous host memory, all zeros, counted against a
// capacity; streams run at once.  Kernels do nothing but write the results that
// the host reads: a batch is well formed, has the conflicts the test asks for,
// and commits.
#include <sys/mman.h>

#include <cstring>
#include <map>
#include <string>

#include "../../paper_2406_10158_amd/csrc/engine.h"

using namespace cce;

namespace {
std::map<char *, size_t> mem;           // allocations by address
size_t used = 0, capacity = ~size_t(0), peak = 0;
std::map<const void *, std::string> kernels;
std::string fail_call;                  // the call to fail, and how many of it succeed first
long fail_after = 0;
uint64_t pairs = 0, kinds = 0, engine_ops = 0;
hipError_t last = hipSuccess;

hipError_t done(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
bool fails(const char *call) { return fail_call == call && fail_after-- == 0; }
template <class T>
T arg(void **a, int i) {
  return *(T *)a[i];
}
}  // namespace

extern "C" {

// ---- what the tests set and look at -----------------------------------------
void fake_reset() {
  capacity = ~size_t(0);
  peak = used;
  fail_call.clear();
  pairs = kinds = engine_ops = 0;
}
void fake_capacity(size_t bytes) { capacity = bytes; }
size_t fake_used() { return used; }
size_t fake_peak() { return peak; }
void fake_fail(const char *call, long after) {
  fail_call = call;
  fail_after = after;
}
// results of the batches submitted from now on: pairs of writes that meet, kinds of operations (IngestOut), and
// the operations of the hot-row engine's share (all of its transactions)
void fake_batch(uint64_t meet_pairs, uint64_t op_kinds, uint64_t eng_ops) {
  pairs = meet_pairs;
  kinds = op_kinds;
  engine_ops = eng_ops;
}

// ---- the runtime ---------------------------------------------------------------
hipError_t hipMalloc(void **p, size_t bytes) {
  *p = nullptr;
  if (fails("hipMalloc") || bytes > capacity || used > capacity - bytes) return done(hipErrorOutOfMemory);
  void *m = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return done(hipErrorOutOfMemory);
  mem[(char *)m] = bytes;
  used += bytes;
  peak = used > peak ? used : peak;
  *p = m;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (!p) return hipSuccess;
  auto it = mem.find((char *)p);
  if (it == mem.end()) return done(hipErrorInvalidValue);
  used -= it->second;
  munmap(p, it->second);
  mem.erase(it);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
  *p = std::calloc(1, bytes);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind k, hipStream_t) {
  // (only returned: a runtime whose last error is the last call's has forgotten it after the next)
  if (k == hipMemcpyHostToDevice && fails("hipMemcpyHtoD")) return hipErrorInvalidValue;
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) {
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) {
  if (fails("hipMemsetAsync")) return done(hipErrorInvalidValue);
  if (v) std::memset(p, v, n);
  else if (n < (1u << 20)) std::memset(p, 0, n);  // (the rest of a large one is zero as it is)
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **a, size_t, hipStream_t) {
  if (!grid.x) return done(hipErrorInvalidConfiguration);
  const std::string &name = kernels[f];
  auto is = [&](const char *s) { return name.find(s) != std::string::npos; };
  if (is("ingest_local_kernel") || is("ingest_pack_kernel")) {
    const IngestArgs &in = *(IngestArgs *)a[0];
    std::memset(in.out, 0, INGEST_N * sizeof(uint64_t));
    in.out[INGEST_ERR] = ~0ull;
    for (uint64_t t = 0; t < in.n_txns; ++t)
      if (in.txns[t].n_ops > in.out[INGEST_MAX_OPS]) in.out[INGEST_MAX_OPS] = in.txns[t].n_ops;
    in.out[INGEST_PAIRS] = pairs;
    in.out[INGEST_TOP] = pairs ? 2 : 0;
    in.out[INGEST_KINDS] = kinds;
  } else if (is("split_lists_kernel")) {
    const uint64_t n = arg<uint64_t>(a, 1);
    const_cast<uint32_t *>(arg<const uint32_t *>(a, 2))[n] = (uint32_t)n;
    const_cast<uint32_t *>(arg<const uint32_t *>(a, 3))[n] = (uint32_t)engine_ops;
  } else if (is("init_kernel")) {
    std::memset(arg<Ctl *>(a, 6), 0, sizeof(Ctl));
    std::memset(arg<LatState *>(a, 7), 0, sizeof(LatState));
  } else if (is("engine_commit_kernel")) {
    arg<Ctl *>(a, 3)->stats[DS_COMMITTED] = arg<uint64_t>(a, 1);
  } else if (is("chain_outcomes_kernel")) {
    arg<Ctl *>(a, 3)->stats[DS_COMMITTED] = arg<uint64_t>(a, 1);
  } else if (is("txn_kernel")) {
    RunArgs &r = *(RunArgs *)a[0];
    r.ctl->stats[DS_COMMITTED] += r.n_txns;
  }
  return hipSuccess;
}

hipError_t hipGetDeviceCount(int *n) {
  *n = 1;
  return hipSuccess;
}
#undef hipGetDeviceProperties
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  std::memset((void *)p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 100000;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamCreate(hipStream_t *s) {
  *s = (hipStream_t)1;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = (hipEvent_t)1;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 1;
  return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static char *scratch = (char *)mmap(nullptr, STATIC_SCRATCH_BYTES, PROT_READ | PROT_WRITE,
                                      MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  *p = scratch;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 1;
  return hipSuccess;
}

// ---- what the compiler's code calls --------------------------------------------
struct Config {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
};
static Config config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  config = {grid, block, shared, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *s = config.stream;
  return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
  // (called while the library is loaded, before anything here is used)
  kernels[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}
