// A GPU for tests of the executor's dispatch on machines without one: the runtime calls and kernel launches that
// csrc/executor.cpp makes, on host memory.  Linked with the library's host sources in place of the HIP runtime and the
// kernels.  What is enqueued on a stream runs later, when the host asks about an event: some stream, drawn at random,
// takes its next step.  So streams overtake each other, completions are seen late, and work that was enqueued without
// the order it needs reads what is not there yet.
//
// A kernel vertex writes one 32-bit word, a mix of the first words of its operands (additions: their sum, so that
// increments commute); a graph's results depend on every vertex and on nothing else.
#include <algorithm>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <vector>

#include "kernels.h"

namespace {

struct Event { uint64_t recorded = 0, reached = 0; };
struct Step {
  std::function<void()> run;
  Event* wait = nullptr;  // not before this event has reached `at`
  uint64_t at = 0;
  bool kernel = false;
};
struct Stream { int index; std::deque<Step> steps; };

// what the executor enqueued: kind 0 kernel, 1 copy kernel, 2 copy kernel inside the GPU, 3 runtime copy
struct Entry { int32_t kind, stream, n, detail, kernels_before, to_gpu; };

std::map<int, Stream> streams;
std::map<const char*, std::pair<size_t, hipMemoryType>> memory;  // start -> size, kind
std::vector<Entry> entries;
std::vector<int32_t> stages;  // of the launches of small products
uint64_t rng = 1, serial = 0, idle_asks = 0;
int64_t calls_until_failure = -1, enqueued_after_failure = -1;  // -1: no failure yet

uint64_t mix(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
Stream& of(hipStream_t s) { return *(Stream*)s; }
bool fails() {
  if (calls_until_failure < 0 || calls_until_failure-- > 0) return false;
  enqueued_after_failure = 0;
  return true;
}
int64_t pending() {
  int64_t n = 0;
  for (auto& s : streams) n += (int64_t)s.second.steps.size();
  return n;
}
bool step(Stream& s) {
  if (s.steps.empty()) return false;
  Step& f = s.steps.front();
  if (f.wait && f.wait->reached < f.at) return false;
  auto run = std::move(f.run);
  s.steps.pop_front();
  if (run) run();
  return true;
}
bool step_any() {  // one step of one stream, starting the search at a random one
  const int n = (int)streams.size();
  const int first = n ? (int)((rng = mix(rng)) % n) : 0;
  for (int k = 0; k < n; ++k)
    if (step(std::next(streams.begin(), (first + k) % n)->second)) return true;
  return false;
}
void push(hipStream_t s, std::function<void()> run, bool kernel = false) {
  Step st;
  st.run = std::move(run);
  st.kernel = kernel;
  of(s).steps.push_back(std::move(st));
}
const std::pair<const char* const, std::pair<size_t, hipMemoryType>>* find(const void* p) {
  auto it = memory.upper_bound((const char*)p);
  if (it == memory.begin()) return nullptr;
  --it;
  return (const char*)p < it->first + it->second.first ? &*it : nullptr;
}
bool on_gpu(const void* p) {
  auto* m = find(p);
  return m && m->second.second == hipMemoryTypeDevice;
}
void log(int kind, hipStream_t s, int n, int detail, const void* dst) {
  int before = 0;
  for (auto& st : of(s).steps) before += st.kernel;
  enqueued_after_failure += enqueued_after_failure >= 0;
  entries.push_back({kind, of(s).index, n, detail, before, dst ? on_gpu(dst) : 0});
}
uint32_t word(const void* p) { uint32_t w; memcpy(&w, p, 4); return w; }
void vertex(int cls, const tn::DeviceTables& t, uint32_t i) {
  const tn::OpDesc& d = t.descs[i];
  uint32_t w = 0;
  if (cls == tn::LC_ADD) {
    for (int k = 0; k < d.n_in; ++k) w += word(t.ptrs[d.ptr0 + k]);
  } else if (cls != tn::LC_ZERO) {
    uint64_t h = 7;
    for (int k = 0; k < d.n_in; ++k) h = mix(h ^ word(t.ptrs[d.ptr0 + k]));
    w = (uint32_t)h;
  }
  memcpy(d.out, &w, 4);
}
void* allocate(size_t n, hipMemoryType kind) {
  void* p = aligned_alloc(4096, (n + 4095) / 4096 * 4096 + 4096);
  memset(p, 0xA5, n);
  memory[(const char*)p] = {n, kind};
  return p;
}
hipError_t release(void* p) {
  memory.erase((const char*)p);
  free(p);
  return hipSuccess;
}
hipError_t copies(int kind, const tn::CopyBatch& b, int wgs, hipStream_t s) {
  if (b.n <= 0 || b.total_blocks <= 0) return hipSuccess;
  if (fails()) return hipErrorLaunchFailure;
  log(kind, s, b.n, wgs, b.it[0].dst);
  for (int k = 0; k < b.n; ++k) {
    const tn::CopyItem it = b.it[k];
    push(s, [it] { memcpy(it.dst, it.src, it.bytes); });
  }
  return hipSuccess;
}

}  // namespace

extern "C" {

// ---- for the tests --------------------------------------------------------------------------
void* fake_stream(int index) {
  Stream& s = streams[index];
  s.index = index;
  return &s;
}
void* fake_alloc(uint64_t bytes, int gpu) { return allocate(bytes, gpu ? hipMemoryTypeDevice : hipMemoryTypeHost); }
void fake_reset(uint64_t seed) {  // forgets streams and the log, frees nothing
  streams.clear();
  entries.clear();
  stages.clear();
  rng = mix(seed + 1);
  idle_asks = 0;
  calls_until_failure = enqueued_after_failure = -1;
}
int64_t fake_enqueued_after_failure() { return enqueued_after_failure; }
void fake_fail_after(int64_t calls) { calls_until_failure = calls; }
int64_t fake_pending() { return pending(); }
int64_t fake_log(int32_t* out, int64_t cap) {
  for (int64_t i = 0; i < (int64_t)entries.size() && i < cap; ++i) memcpy(out + 6 * i, &entries[i], sizeof(Entry));
  return (int64_t)entries.size();
}

int64_t fake_stages(int32_t* out, int64_t cap) {
  for (int64_t i = 0; i < (int64_t)stages.size() && i < cap; ++i) out[i] = stages[i];
  return (int64_t)stages.size();
}

// ---- the runtime ----------------------------------------------------------------------------
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "planted"; }
hipError_t hipMalloc(void** p, size_t n) { *p = allocate(n, hipMemoryTypeDevice); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = allocate(n, hipMemoryTypeHost); return hipSuccess; }
hipError_t hipFree(void* p) { return release(p); }
hipError_t hipHostFree(void* p) { return release(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  if (fails()) return hipErrorUnknown;
  log(3, st, 1, 0, d);
  push(st, [=] { memcpy(d, s, n); });
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  auto* m = find(p);
  if (!m) return hipErrorInvalidValue;  // pageable
  memset(a, 0, sizeof *a);
  a->type = m->second.second;
  a->devicePointer = (void*)p;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  auto* m = find(p);
  if (!m) return hipErrorInvalidValue;
  *base = (hipDeviceptr_t)m->first;
  *size = m->second.first;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t) new Event; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (fails()) return hipErrorUnknown;
  Event* ev = (Event*)e;
  const uint64_t mark = ev->recorded = ++serial;
  push(s, [ev, mark] { ev->reached = std::max(ev->reached, mark); });
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  Event* ev = (Event*)e;
  if (ev->reached >= ev->recorded) return hipSuccess;
  if (!step_any() && ++idle_asks > 1000) return hipErrorUnknown;  // nothing left that could reach it
  return ev->reached >= ev->recorded ? hipSuccess : hipErrorNotReady;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  Step st;
  st.wait = (Event*)e;
  st.at = st.wait->recorded;
  of(s).steps.push_back(std::move(st));
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  while (!of(s).steps.empty())
    if (!step(of(s)) && !step_any()) return hipErrorUnknown;
  return hipSuccess;
}

}  // extern "C"

// ---- the kernels ----------------------------------------------------------------------------
namespace tn {

hipError_t static_table_region(void** p) {
  static char region[kStaticTableBytes];
  *p = region;
  return hipSuccess;
}
int32_t blocks_for(int, const OpDesc&, const int32_t*) { return 1; }
hipError_t launch_copies(const CopyBatch& b, int wgs, hipStream_t s) { return copies(1, b, wgs, s); }
hipError_t launch_device_copies(const CopyBatch& b, hipStream_t s) { return copies(2, b, 0, s); }
hipError_t launch_batch(int cls, int, int, const DeviceTables& t, const Batch& b, int32_t, hipStream_t s) {
  if (fails()) return hipErrorLaunchFailure;
  log(0, s, b.n, cls, nullptr);
  if (cls == LC_GEMM_F32 || cls == LC_GEMM_BF16_SMALL) stages.push_back(b.stages);
  for (int k = 0; k < b.n; ++k) {
    const uint32_t i = b.at(k);
    push(s, [=] { vertex(cls, t, i); }, true);
  }
  return hipSuccess;
}
hipError_t launch_gemm_rows(int, const DeviceTables& t, uint32_t, const RowVertex* rows, int n, int32_t, hipStream_t s) {
  if (fails()) return hipErrorLaunchFailure;
  log(0, s, n, LC_GEMM_ROWS, nullptr);
  stages.push_back(0);
  for (int k = 0; k < n; ++k) stages.back() = std::max(stages.back(), rows[k].stages);
  for (int k = 0; k < n; ++k) {
    const uint32_t i = rows[k].desc;
    push(s, [=] { vertex(LC_GEMM_ROWS, t, i); }, true);
  }
  return hipSuccess;
}

}  // namespace tn
