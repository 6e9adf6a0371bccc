// Test-only stand-in for the HIP runtime and the kernels' launchers: the library's host code
// (runtime.cpp, networks.cpp) is linked with it into a shared object that runs without a GPU, so that
// the CPU tests can look at what a call allocates, copies, waits for and launches. Device memory is
// host memory that starts at zero, copies run at once, and kernels do nothing but what the host reads
// of them (the tests set those values). An event completes at once, or, held, when it is waited for.
#include <hip/hip_runtime_api.h>

#include <sys/mman.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "../../paper_2608_27612_amd/csrc/band.h"
#include "../../paper_2608_27612_amd/csrc/emr_internal.h"
#include "../../paper_2608_27612_amd/csrc/network.h"

namespace {
struct Fake {
  std::recursive_mutex mu;
  std::map<void*, size_t> device, pinned;
  size_t held = 0, limit = ~size_t(0);
  bool hold_events = false, capturing = false;
  std::atomic<bool> block_waits{false};
  int waits = 0;        // stream and event waits of the host
  int copies = 0;       // host-to-device copies from pinned memory
  int slow_copies = 0;  // the same from other memory
  const void* totals = nullptr;  // of the last discover launch
  uint64_t total = 0;   // what the next record calls and filters report
  uint32_t bind_error = 0;
  uint32_t* bind_word = nullptr;  // held with the events
};
Fake& F() {
  static Fake* f = new Fake;
  return *f;
}
using Lock = std::lock_guard<std::recursive_mutex>;
struct Event {
  bool pending = false;
};
bool inside(const std::map<void*, size_t>& m, const void* p) {
  auto it = m.upper_bound(const_cast<void*>(p));
  if (it == m.begin()) return false;
  --it;
  return (const char*)p < (const char*)it->first + it->second;
}
hipError_t take(std::map<void*, size_t>& m, void** p, size_t n, size_t* held) {
  Lock l(F().mu);
  n = (n + 4095) & ~size_t(4095);
  if (held && *held + n > F().limit) return hipErrorOutOfMemory;
  void* q = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (q == MAP_FAILED) return hipErrorOutOfMemory;
  m[q] = n;
  if (held) *held += n;
  *p = q;
  return hipSuccess;
}
hipError_t give(std::map<void*, size_t>& m, void* p, size_t* held) {
  if (!p) return hipSuccess;
  Lock l(F().mu);
  auto it = m.find(p);
  if (it == m.end()) return hipErrorInvalidValue;
  if (held) *held -= it->second;
  munmap(p, it->second);
  m.erase(it);
  return hipSuccess;
}
}  // namespace

extern "C" {

// ------------------------------------------------------------------ the tests' side
void fake_limit(int64_t bytes) { F().limit = bytes < 0 ? ~size_t(0) : F().held + (size_t)bytes; }
void fake_hold_events(int on) {
  F().hold_events = on != 0;
  if (on || !F().bind_word) return;
  *F().bind_word = F().bind_error;
  F().bind_word = nullptr;
}
void fake_block_waits(int on) { F().block_waits = on != 0; }
void fake_capturing(int on) { F().capturing = on != 0; }
void fake_total(int64_t n) { F().total = (uint64_t)n; }
void fake_bind_error(uint32_t bits) { F().bind_error = bits; }
const void* fake_totals(void) { return F().totals; }
int64_t fake_held(void) { return (int64_t)F().held; }
int64_t fake_size(const void* p) {
  auto it = F().device.find(const_cast<void*>(p));
  return it == F().device.end() ? -1 : (int64_t)it->second;
}
void fake_counts(int32_t* out) {
  out[0] = F().waits;
  out[1] = F().copies;
  out[2] = F().slow_copies;
}

// ------------------------------------------------------------------ HIP
hipError_t hipMalloc(void** p, size_t n) { return take(F().device, p, n, &F().held); }
hipError_t hipFree(void* p) { return give(F().device, p, &F().held); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return take(F().pinned, p, n, nullptr); }
hipError_t hipHostFree(void* p) { return give(F().pinned, p, nullptr); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) {
  std::memset(p, v, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyHostToDevice) {
    Lock l(F().mu);
    ++(inside(F().pinned, s) ? F().copies : F().slow_copies);
  }
  std::memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error of the stand-in runtime"; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 8;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t) new int(0);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  while (F().block_waits) std::this_thread::yield();
  Lock l(F().mu);
  ++F().waits;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = F().capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t) new Event;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete (Event*)e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  ((Event*)e)->pending = F().hold_events;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  return ((Event*)e)->pending && F().hold_events ? hipErrorNotReady : hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  Lock l(F().mu);
  ++F().waits;
  ((Event*)e)->pending = false;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipModuleLoadData(hipModule_t*, const void*) { return hipErrorNotSupported; }
hipError_t hipModuleUnload(hipModule_t) { return hipSuccess; }
hipError_t hipModuleGetFunction(hipFunction_t*, hipModule_t, const char*) { return hipErrorNotSupported; }
hipError_t hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(int*, hipFunction_t, int, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipModuleLaunchKernel(hipFunction_t, unsigned, unsigned, unsigned, unsigned, unsigned,
                                 unsigned, unsigned, hipStream_t, void**, void**) {
  return hipErrorNotSupported;
}

// ------------------------------------------------------------------ the kernels' launchers
extern const uint8_t emr_jit_template_begin[1] = {0}, emr_jit_template_end[1] = {0};
namespace {
void hand_over(uint32_t* host) {
  if (!host) return;
  host[emr::kFlagTotal] = (uint32_t)F().total;
  host[emr::kFlagTotal + 1] = (uint32_t)(F().total >> 32);
}
}  // namespace
hipError_t emr_launch_fill(void* p, int64_t n_words, uint32_t value, hipStream_t) {
  for (int64_t i = 0; i < n_words; ++i) ((uint32_t*)p)[i] = value;
  return hipSuccess;
}
hipError_t emr_launch_grid(float*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t emr_launch_bind(const emr::BindArgs* a, hipStream_t) {
  if (!F().bind_error) return hipSuccess;
  if (F().hold_events)
    F().bind_word = a->err;
  else
    *a->err = F().bind_error;
  return hipSuccess;
}
hipError_t emr_launch_discover(const emr::DiscoverArgs* a, int, uint32_t, hipStream_t, hipEvent_t,
                               hipEvent_t) {
  F().totals = a->pair_total;
  for (uint32_t r = 0; r < a->n_pairs && a->pair_total; ++r)
    if (a->pair_total[r] != 0u) return hipErrorInvalidValue;  // (a record call's totals start at 0)
  return hipSuccess;
}
hipError_t emr_launch_compact(const emr::ScanArgs* S, const emr::MoveArgs*, hipStream_t) {
  for (uint32_t r = 0; r < S->n_pairs; ++r) S->pair_total[r] = 1u, S->clear_total[r] = 0u;
  hand_over(S->host);
  return hipSuccess;
}
hipError_t emr_launch_finalize(uint32_t*, uint32_t*, hipStream_t) { return hipSuccess; }
hipError_t emr_launch_scan(const emr::ScanArgs*, hipStream_t) { return hipSuccess; }
hipError_t emr_launch_hidden(const emr::HiddenArgs*, int, hipStream_t) { return hipSuccess; }
hipError_t emr_launch_express(const emr::ExpressArgs* A, hipStream_t) {
  hand_over(A->spans.host);
  return hipSuccess;
}
hipError_t emr_launch_chain(const emr::ChainArgs*, hipStream_t) { return hipSuccess; }
hipError_t emr_launch_band(const emr::BandArgs*, hipStream_t) { return hipSuccess; }
hipError_t emr_launch_band_select(const emr::BandSelectArgs*, hipStream_t) { return hipSuccess; }
hipError_t emr_launch_tile_geo(uint32_t*, uint32_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t emr_noalloc_scratch(void**) { return hipErrorNotSupported; }
int emr_discover_per_cu(int) { return 1; }
hipError_t emr_discover_setup(const emr::DiscoverArgs*, uint32_t, int, int, emr::DiscoverScalars*,
                              uint32_t*) {
  return hipErrorNotSupported;
}
hipError_t emr_launch_net(int, const void*, hipStream_t) { return hipSuccess; }
hipError_t emr_net_sort(void*, size_t* bytes, const uint32_t*, uint32_t*, const uint64_t*, uint64_t*,
                        uint32_t, int, hipStream_t) {
  *bytes = 256;
  return hipSuccess;
}

}  // extern "C"
