// Networks built from a population's discovered substrates, and their activation (the networks the
// experiments evaluate, Section 5: XOR over its four patterns, with the hidden-to-hidden
// connection type of Section 4's configurations).
//
// The host drives the phases through the library's own entry points: Phase 1 on the substrate
// sources (emr_discover), its hidden nodes (emr_hidden_sources, which also records every hidden
// cell in a per-genome bitmap) and expressed connections (emr_express); then each hidden-to-hidden
// phase queries the previous phase's new hidden nodes, up to the requested number of phases or
// until no genome finds a new one. The network kernels (network.hip) then number the nodes, map
// every expressed connection to an edge, prune to the input-to-output paths (passes over every
// edge of the population until one changes nothing) and group each kept node's incoming edges (a
// stable sort of the edges by destination). The host waits where it needs a count: a phase's
// records, its new nodes and connections, the pruning's end, and the networks' offsets.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/emr.h"
#include "network.h"

namespace emr {
emr_status set_error(emr_status st, const std::string& msg);
}
extern "C" hipError_t emr_launch_net(int step, const void* args, hipStream_t s);
extern "C" hipError_t emr_net_sort(void* tmp, size_t* bytes, const uint32_t* kin, uint32_t* kout,
                                   const uint64_t* vin, uint64_t* vout, uint32_t n, int bits,
                                   hipStream_t s);

namespace {

emr_status failf(emr_status st, const char* fmt, ...) {
  char b[512];
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(b, sizeof b, fmt, ap);
  va_end(ap);
  return emr::set_error(st, b);
}

#define NET_HIP(call)                                                                          \
  do {                                                                                         \
    hipError_t e_ = (call);                                                                    \
    if (e_ != hipSuccess) return failf(EMR_E_DEVICE, "%s: %s", #call, hipGetErrorString(e_)); \
  } while (0)
#define NET_TRY(call)              \
  do {                             \
    emr_status s_ = (call);        \
    if (s_ != EMR_OK) return s_;   \
  } while (0)

// Device memory of the network builds, kept for reuse: a build allocates and frees dozens of
// buffers whose sizes change little from one generation to the next, and a hipMalloc / hipFree
// pair costs about 0.1 ms. A freed buffer enters its device's cache with an event recorded on the
// stream that used it (no event when the caller has already waited for that work) and is handed
// out again once that event has completed, to a request of at most its size and more than half
// of it. At most kCacheBytes stay cached per device; a buffer beyond that is freed. Cached memory
// is held until the process ends.
constexpr size_t kCacheBytes = size_t(8) << 30;

struct CacheEntry {
  void* p;
  hipEvent_t ev;  // nullptr: idle
};
struct DevCache {
  std::mutex mu;
  std::map<int, std::multimap<size_t, CacheEntry>> blocks;
  std::map<int, size_t> held;
  std::vector<hipEvent_t> spare;
};
DevCache& dev_cache() {
  static DevCache* c = new DevCache;  // (never destroyed: cached buffers live as long as the process)
  return *c;
}

// A cached buffer of at least `bytes` on device `dev` whose last use has completed, or nullptr.
void* cache_take(int dev, size_t bytes, size_t* cap) {
  DevCache& C = dev_cache();
  std::lock_guard<std::mutex> lk(C.mu);
  auto& m = C.blocks[dev];
  for (auto it = m.lower_bound(bytes); it != m.end() && it->first / 2 < bytes; ++it) {
    if (it->second.ev) {
      const hipError_t q = hipEventQuery(it->second.ev);
      if (q != hipSuccess) {
        (void)hipGetLastError();  // (not ready is no error of the caller's)
        continue;
      }
      C.spare.push_back(it->second.ev);
    }
    void* p = it->second.p;
    *cap = it->first;
    C.held[dev] -= it->first;
    m.erase(it);
    return p;
  }
  return nullptr;
}

// Frees every cached buffer of `dev` (waiting for the last use of each).
void cache_flush(int dev) {
  DevCache& C = dev_cache();
  std::lock_guard<std::mutex> lk(C.mu);
  auto& m = C.blocks[dev];
  for (auto& kv : m) {
    if (kv.second.ev) {
      (void)hipEventSynchronize(kv.second.ev);
      C.spare.push_back(kv.second.ev);
    }
    (void)hipFree(kv.second.p);
  }
  m.clear();
  C.held[dev] = 0;
}

// Returns a buffer to the cache; `s` is the stream of its last use, or nullptr with `idle` when
// that use is known to have completed.
void cache_give(int dev, void* p, size_t cap, hipStream_t s, bool idle) {
  DevCache& C = dev_cache();
  std::unique_lock<std::mutex> lk(C.mu);
  if (C.held[dev] + cap > kCacheBytes) {
    lk.unlock();
    (void)hipFree(p);  // (waits for the device's outstanding work)
    return;
  }
  hipEvent_t ev = nullptr;
  if (!idle) {
    if (!C.spare.empty()) {
      ev = C.spare.back();
      C.spare.pop_back();
    } else if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      lk.unlock();
      (void)hipFree(p);
      return;
    }
    if (hipEventRecord(ev, s) != hipSuccess) {
      (void)hipGetLastError();
      C.spare.push_back(ev);
      lk.unlock();
      (void)hipFree(p);
      return;
    }
  }
  C.blocks[dev].emplace(cap, CacheEntry{p, ev});
  C.held[dev] += cap;
}

// A device allocation of a build or of the networks handle, from the cache.
struct Dev {
  void* p = nullptr;
  size_t bytes = 0;   // asked for
  size_t cap = 0;     // the buffer's size
  int dev = 0;
  hipStream_t s = nullptr;  // the stream its users run on
  Dev() = default;
  Dev(const Dev&) = delete;
  Dev& operator=(const Dev&) = delete;
  ~Dev() { reset(); }
  // Back to the cache, usable once the work queued on `s` so far has completed.
  void reset() { release(false); }
  // Back to the cache when the caller has waited for every use of the buffer.
  void reset_idle() { release(true); }
  void take(Dev& o) {
    reset();
    p = o.p;
    bytes = o.bytes;
    cap = o.cap;
    dev = o.dev;
    s = o.s;
    o.p = nullptr;
    o.bytes = o.cap = 0;
  }
  template <class T>
  T* as() const {
    return static_cast<T*>(p);
  }

 private:
  void release(bool idle) {
    if (p) cache_give(dev, p, cap, s, idle);
    p = nullptr;
    bytes = cap = 0;
  }
};

emr_status alloc(Dev& d, size_t bytes, const char* what, hipStream_t s) {
  d.reset();
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return failf(EMR_E_DEVICE, "networks: no current device");
  }
  const size_t want = bytes ? (bytes + 255) & ~size_t(255) : 256;
  size_t cap = 0;
  void* p = cache_take(dev, want, &cap);
  if (!p) {
    cap = want;
    if (hipMalloc(&p, want) != hipSuccess) {
      (void)hipGetLastError();
      cache_flush(dev);
      if (hipMalloc(&p, want) != hipSuccess) {
        (void)hipGetLastError();
        return failf(EMR_E_NOMEM, "networks: cannot allocate %zu bytes for %s", bytes, what);
      }
    }
  }
  d.p = p;
  d.bytes = bytes;
  d.cap = cap;
  d.dev = dev;
  d.s = s;
  return EMR_OK;
}

emr_status to_host(void* dst, const void* src, size_t bytes, hipStream_t s) {
  if (bytes == 0) return EMR_OK;
  NET_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s));
  NET_HIP(hipStreamSynchronize(s));
  return EMR_OK;
}

emr_status to_device(void* dst, const void* src, size_t bytes, hipStream_t s) {
  if (bytes == 0) return EMR_OK;
  NET_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s));
  return EMR_OK;
}

constexpr int32_t kMaxSubstrate = 1024;
constexpr int32_t kMaxIterations = 64;
constexpr int32_t kMaxSteps = 1 << 20;
constexpr int32_t kMaxPatterns = 1 << 16;

// One phase: its sources, discovery, and expressed connections.
struct Phase {
  std::vector<emr_source> sources;
  std::vector<int32_t> offs;  // per-genome sources (empty: the shared substrate)
  int64_t n_pairs = 0;
  Dev parent, w4, rcount, roffset;
  int64_t rcap = 0, rtotal = 0;
  Dev cell, w, ccount, coffset;
  int64_t ccap = 0, ctotal = 0;
  // the hidden-node call (until it is checked) and the new nodes it found
  Dev hws, hsrc, hcell, hoff, cws;
  int64_t hcap = 0, n_new = 0;
  Dev src_cell;   // [sources] heap cells of the queried hidden nodes
  Dev src_offs;   // [n_genomes + 1] int64 copy of offs
  Dev ws;         // the discovery's workspace, released once it is checked

  void release_idle() {
    for (Dev* d : {&parent, &w4, &rcount, &roffset, &cell, &w, &ccount, &coffset, &src_cell,
                   &src_offs, &ws, &hws, &hsrc, &hcell, &hoff, &cws})
      d->reset_idle();
  }

  bool shared() const { return offs.empty(); }
  const int32_t* offs_ptr() const { return offs.empty() ? nullptr : offs.data(); }
  int32_t n_shared() const { return offs.empty() ? (int32_t)sources.size() : 0; }
  emr_result result() const {
    emr_result r;
    r.parent = parent.as<uint32_t>();
    r.w4 = w4.as<float>();
    r.capacity = rcap;
    r.pair_count = rcount.as<int64_t>();
    r.pair_offset = roffset.as<int64_t>();
    r.workspace = ws.p;
    r.workspace_bytes = (int64_t)ws.bytes;
    return r;
  }
};

}  // namespace

struct emr_networks {
  int device = 0;
  int32_t n_genomes = 0, n_sub = 0, n_in = 0, n_out = 0, depth = 0;
  int64_t words = 0;
  std::vector<emr_source> substrate;
  std::vector<int32_t> slots;  // in_slot[n_sub], then out_slot[n_sub]
  std::vector<std::unique_ptr<Phase>> phases;
  Dev known;
  Dev node_offset, node_cell, node_in, in_offset, in_src, in_w, d_slots;
  Dev d_out_node;  // [n_out] substrate index of output o
  int64_t nodes = 0, edges = 0;
  Dev state, patterns;
  // genomes in the order of the activation launches (order_genomes): their loads and node counts, the
  // sums over those before each, and the most nodes of those before each in its class
  Dev order;
  std::vector<double> order_load, batches_before;
  std::vector<int64_t> nodes_before, edges_before;
  std::vector<uint32_t> order_host, order_nodes, most_before, class_first;
  // pinned staging of an activation's patterns and targets, and the event of its last copy
  void* pin = nullptr;
  size_t pin_bytes = 0;
  hipEvent_t pin_done = nullptr;
  bool pin_pending = false;
  // the end of the last activation (its outputs written)
  hipEvent_t done = nullptr;
  bool done_pending = false;
  // The build synchronized with its stream before the handle was returned (or, failing, before
  // the handle was destroyed), and the last activation is waited for here: every buffer is idle.
  ~emr_networks() {
    if (done) {
      if (done_pending) (void)hipEventSynchronize(done);
      (void)hipEventDestroy(done);
    }
    if (pin_done) {
      if (pin_pending) (void)hipEventSynchronize(pin_done);
      (void)hipEventDestroy(pin_done);
    }
    if (pin) (void)hipHostFree(pin);
    for (auto& ph : phases) ph->release_idle();
    for (Dev* d : {&known, &node_offset, &node_cell, &node_in, &in_offset, &in_src, &in_w,
                   &d_slots, &d_out_node, &state, &patterns, &order})
      d->reset_idle();
  }
};

namespace {

struct Build {
  const emr_population* pop;
  emr_networks* net;
  float theta;
  int32_t type_mask;
  float w_min;
  hipStream_t s;
};

// Moves the first bytes of buffers into buffers of that size, in one launch, and gives the larger
// ones back; without the memory for it a buffer stays as it is.
struct Fit {
  Dev* d;
  size_t bytes;
  const char* what;
};
emr_status fit(const Fit* items, int n, hipStream_t s) {
  Dev small[emr::kNetFits];
  emr::NetFitArgs a{};
  for (int i = 0; i < n && i < emr::kNetFits; ++i) {
    if (alloc(small[i], items[i].bytes, items[i].what, s) != EMR_OK) continue;
    const uint32_t k = a.count++;
    a.src[k] = items[i].d->p;
    a.dst[k] = small[i].p;
    a.units[k] = ((int64_t)items[i].bytes + 15) / 16;  // (sizes are whole 256-byte blocks)
  }
  NET_HIP(emr_launch_net(15, &a, s));
  for (int i = 0; i < n && i < emr::kNetFits; ++i)
    if (small[i].p) items[i].d->take(small[i]);
  return EMR_OK;
}

// A retry runs the phase's discovery a second time (and a heavy population's hidden phase is most of
// a generation; one random population of 1000 in ten keeps more than 16M records), so the first guess
// is large: 64M records (1.3 GB, as much again for the pool). Records that fill less than half then
// move to buffers of their number, which the phase keeps as long as the networks live (20 us for 3M,
// 150 us for 18M records, of builds of 3.9 and 8 ms). Where the memory for the large
// guess is short the guess is 16M, which the phase may keep.
constexpr size_t kFitBytes = size_t(4) << 20;  // (below this a copy's launch costs more than it frees)
constexpr int64_t kFirstRecords = int64_t(1) << 26, kKeptRecords = int64_t(1) << 24;

// The phase's discovery, retried once with the exact capacity when the first guess was short.
emr_status discover_phase(Build& B, Phase& P) {
  emr_networks& N = *B.net;
  const emr_source* src = P.sources.data();
  const int32_t n = (int32_t)P.sources.size();
  P.n_pairs = P.shared() ? (int64_t)N.n_genomes * n : P.offs[N.n_genomes];
  NET_TRY(alloc(P.rcount, (size_t)P.n_pairs * 8, "pair counts", B.s));
  NET_TRY(alloc(P.roffset, (size_t)(P.n_pairs + 1) * 8, "pair offsets", B.s));
  int64_t n_pos = 0, Q = 0;
  NET_TRY(emr_grid_count(N.depth, &n_pos, &Q));
  auto room = [&](int64_t cap) -> emr_status {
    int64_t wsb = 0;
    NET_TRY(emr_workspace_bytes(B.pop, src, n, P.offs_ptr(), P.n_shared(), N.depth, cap, &wsb));
    NET_TRY(alloc(P.ws, (size_t)wsb, "discover workspace", B.s));
    NET_TRY(alloc(P.parent, (size_t)cap * 4, "records", B.s));
    return alloc(P.w4, (size_t)cap * 16, "records", B.s);
  };
  int64_t cap = std::max<int64_t>(1, std::min(P.n_pairs * Q, kFirstRecords));
  for (int attempt = 0;; ++attempt) {
    emr_status st = room(cap);
    if (st == EMR_E_NOMEM && attempt == 0 && cap > kKeptRecords) {
      for (Dev* d : {&P.ws, &P.parent, &P.w4}) d->reset_idle();
      cap = kKeptRecords;
      st = room(cap);
    }
    NET_TRY(st);
    P.rcap = cap;
    const emr_result r = P.result();
    NET_TRY(emr_discover(B.pop, src, n, P.offs_ptr(), P.n_shared(), N.depth, B.theta, &r, B.s));
    int64_t total = 0;
    st = emr_result_check(&r, &total, nullptr, B.s);
    if (st == EMR_OK) {
      P.rtotal = total;
      break;
    }
    if (st != EMR_E_CAPACITY || attempt > 0) return st;
    cap = total;
  }
  P.ws.reset_idle();  // (the check waited for the call)
  if (P.rcap > kKeptRecords && 2 * P.rtotal < P.rcap) {
    P.rcap = std::max<int64_t>(1, P.rtotal);
    const Fit records[] = {{&P.parent, (size_t)P.rcap * 4, "records"},
                           {&P.w4, (size_t)P.rcap * 16, "records"}};
    NET_TRY(fit(records, 2, B.s));
  }
  return EMR_OK;
}

// Enqueues the phase's new hidden nodes (or-ed into the bitmap).
emr_status hidden_phase(Build& B, Phase& P) {
  emr_networks& N = *B.net;
  P.hcap = P.rtotal * 4 > 0 ? P.rtotal * 4 : 1;  // every record adds 4 cells at most
  int64_t hb = 0;
  NET_TRY(emr_hidden_workspace_bytes(N.n_genomes, N.depth, &hb));
  NET_TRY(alloc(P.hws, (size_t)hb, "hidden-node workspace", B.s));
  NET_TRY(alloc(P.hsrc, (size_t)P.hcap * sizeof(emr_source), "hidden sources", B.s));
  NET_TRY(alloc(P.hcell, (size_t)P.hcap * 4, "hidden cells", B.s));
  NET_TRY(alloc(P.hoff, (size_t)(N.n_genomes + 1) * 8, "hidden offsets", B.s));
  emr_hidden h;
  h.sources = P.hsrc.as<emr_source>();
  h.cell = P.hcell.as<uint32_t>();
  h.capacity = P.hcap;
  h.offsets = P.hoff.as<int64_t>();
  h.known = N.known.as<uint32_t>();
  h.workspace = P.hws.p;
  h.workspace_bytes = hb;
  const emr_result r = P.result();
  return emr_hidden_sources(B.pop, P.sources.data(), (int32_t)P.sources.size(), P.offs_ptr(),
                            P.n_shared(), N.depth, &r, &h, B.s);
}

// Enqueues the phase's connections.
emr_status express_phase(Build& B, Phase& P) {
  emr_networks& N = *B.net;
  P.ccap = P.rtotal * 4 > 0 ? P.rtotal * 4 : 1;  // four children per record at most
  int64_t eb = 0;
  NET_TRY(emr_express_workspace_bytes(P.n_pairs, &eb));
  NET_TRY(alloc(P.cws, (size_t)eb, "connection workspace", B.s));
  NET_TRY(alloc(P.cell, (size_t)P.ccap * 4, "connections", B.s));
  NET_TRY(alloc(P.w, (size_t)P.ccap * 4, "connections", B.s));
  NET_TRY(alloc(P.ccount, (size_t)P.n_pairs * 8, "connection counts", B.s));
  NET_TRY(alloc(P.coffset, (size_t)(P.n_pairs + 1) * 8, "connection offsets", B.s));
  emr_connections c;
  c.cell = P.cell.as<uint32_t>();
  c.w = P.w.as<float>();
  c.capacity = P.ccap;
  c.pair_count = P.ccount.as<int64_t>();
  c.pair_offset = P.coffset.as<int64_t>();
  c.workspace = P.cws.p;
  c.workspace_bytes = eb;
  const emr_result r = P.result();
  return emr_express(B.pop, P.sources.data(), (int32_t)P.sources.size(), P.offs_ptr(),
                     P.n_shared(), N.depth, &r, B.type_mask, B.w_min, &c, B.s);
}

// Checks both calls; `next`, when given, receives the new hidden nodes to query: host sources and
// offsets, device cells and offsets.
emr_status finish_phase(Build& B, Phase& P, Phase* next) {
  emr_networks& N = *B.net;
  NET_TRY(emr_call_check(P.hws.p, P.hcap, &P.n_new, nullptr, B.s));
  if (next && P.n_new > 0) {
    if (P.n_new > INT32_MAX)
      return failf(EMR_E_LIMIT, "networks: %lld hidden sources in one phase", (long long)P.n_new);
    next->sources.resize((size_t)P.n_new);
    std::vector<int64_t> off((size_t)N.n_genomes + 1);
    NET_HIP(hipMemcpyAsync(next->sources.data(), P.hsrc.p, (size_t)P.n_new * sizeof(emr_source),
                           hipMemcpyDeviceToHost, B.s));
    NET_TRY(to_host(off.data(), P.hoff.p, off.size() * 8, B.s));
    next->offs.resize(off.size());
    for (size_t g = 0; g < off.size(); ++g) next->offs[g] = (int32_t)off[g];
    next->src_cell.take(P.hcell);
    next->src_offs.take(P.hoff);
  }
  NET_TRY(emr_call_check(P.cws.p, P.ccap, &P.ctotal, nullptr, B.s));
  for (Dev* d : {&P.hws, &P.hsrc, &P.hcell, &P.hoff, &P.cws}) d->reset();
  return EMR_OK;
}

emr_status order_genomes(emr_networks& N, const int64_t* node_off, const int64_t* edge_off,
                         hipStream_t s);

// Numbers the nodes, maps the connections to edges, prunes, and groups the kept edges by
// destination. The sizes that the host needs are known or bounded beforehand (the phases' hidden
// nodes and connections), so it waits only for the reach passes and once at the end.
emr_status assemble(Build& B) {
  emr_networks& N = *B.net;
  const uint32_t G = (uint32_t)N.n_genomes;
  const hipStream_t s = B.s;
  const size_t K = N.phases.size();
  static_assert(kMaxIterations + 1 <= emr::kNetMaxPhases, "phases of a build");
  int64_t n_raw = (int64_t)G * N.n_sub, e_raw = 0;
  for (const auto& p : N.phases) {
    n_raw += p->n_new;
    e_raw += p->ctotal;
  }
  // raw node and edge numbers are u32 (kNoNode, the largest, marks a dropped edge)
  if (n_raw >= (int64_t)emr::kNoNode)
    return failf(EMR_E_LIMIT, "networks: %lld raw nodes (at most 2^32 - 2)", (long long)n_raw);
  if (e_raw >= (int64_t)emr::kNoNode)
    return failf(EMR_E_LIMIT, "networks: %lld raw edges (at most 2^32 - 2)", (long long)e_raw);
  // the host's small tables in one upload: the phases' offset tables, then the substrate directions
  std::vector<uint64_t> tab(2 * K + ((size_t)N.n_sub + 7) / 8);
  for (size_t k = 0; k < K; ++k) {
    Phase& P = *N.phases[k];
    tab[k] = (uint64_t)(uintptr_t)P.coffset.p;
    tab[K + k] = P.shared() ? 0 : (uint64_t)(uintptr_t)P.src_offs.p;
  }
  uint8_t* dir = reinterpret_cast<uint8_t*>(tab.data() + 2 * K);
  for (int32_t j = 0; j < N.n_sub; ++j) dir[j] = N.substrate[j].dir == EMR_DIR_OUT ? 0 : 1;
  Dev rank, hidden, err, d_tab, raw_node, raw_edge, seg, eu, ev, ew, flags, kept_n, gid, sum;
  NET_TRY(alloc(rank, (size_t)G * (size_t)N.words * 4, "bitmap ranks", s));
  NET_TRY(alloc(hidden, (size_t)G * 4, "hidden counts", s));
  // the error word, the pass words and, after the last of them, the kept node count: the host reads
  // the last pass word and the count in one copy
  static_assert((2 + emr::kNetPasses) % 2 == 0, "the count is 8-byte aligned");
  const size_t err_bytes = 4 * (2 + emr::kNetPasses) + 8;
  NET_TRY(alloc(err, err_bytes, "error and pass words", s));
  NET_TRY(alloc(d_tab, tab.size() * 8, "phase tables", s));
  NET_TRY(alloc(raw_node, (size_t)(G + 1) * 8, "node offsets", s));
  NET_TRY(alloc(raw_edge, (size_t)(G + 1) * 8, "edge offsets", s));
  NET_TRY(alloc(seg, K * (size_t)G * 8, "phase segments", s));
  NET_TRY(alloc(eu, (size_t)e_raw * 4, "edges", s));
  NET_TRY(alloc(ev, (size_t)e_raw * 4, "edges", s));
  NET_TRY(alloc(ew, (size_t)e_raw * 4, "edges", s));
  NET_TRY(alloc(flags, (size_t)n_raw * 2, "node flags", s));
  NET_TRY(alloc(kept_n, (size_t)G * 4, "kept counts", s));
  NET_TRY(alloc(gid, (size_t)n_raw * 4, "node numbers", s));
  NET_TRY(alloc(sum, (size_t)(2 * (G + 1) + 1) * 8, "network offsets", s));
  NET_TRY(alloc(N.node_offset, (size_t)(G + 1) * 8, "network node offsets", s));
  NET_TRY(alloc(N.node_cell, (size_t)n_raw * 4, "network nodes", s));
  NET_TRY(alloc(N.node_in, (size_t)n_raw * 4, "network input numbers", s));
  NET_TRY(alloc(N.in_offset, (size_t)(n_raw + 1) * 8, "network edge offsets", s));
  NET_TRY(alloc(N.in_src, (size_t)e_raw * 4, "network edges", s));
  NET_TRY(alloc(N.in_w, (size_t)e_raw * 4, "network edges", s));
  NET_HIP(hipMemsetAsync(err.p, 0, err_bytes, s));
  NET_TRY(to_device(d_tab.p, tab.data(), tab.size() * 8, s));
  uint32_t* d_err = err.as<uint32_t>();
  const uint8_t* d_dir = reinterpret_cast<const uint8_t*>(d_tab.as<uint64_t>() + 2 * K);
  emr::NetRankArgs ra{N.known.as<uint32_t>(), rank.as<uint32_t>(), hidden.as<uint32_t>(), N.words,
                      G};
  NET_HIP(emr_launch_net(0, &ra, s));
  emr::NetLayoutArgs la{};
  la.hidden = hidden.as<uint32_t>();
  la.conn_offset = d_tab.as<const int64_t*>();
  la.src_offsets = d_tab.as<const int64_t*>() + K;
  la.seg = seg.as<int64_t>();
  la.raw_edge = raw_edge.as<int64_t>();
  la.raw_node = raw_node.as<int64_t>();
  la.n_raw = n_raw;
  la.e_raw = e_raw;
  la.n_phases = (uint32_t)K;
  la.n_sub = (uint32_t)N.n_sub;
  la.n_genomes = G;
  la.err = d_err;
  NET_HIP(emr_launch_net(1, &la, s));
  for (size_t k = 0; k < K; ++k) {
    Phase& P = *N.phases[k];
    Dev pairs;
    NET_TRY(alloc(pairs, (size_t)P.n_pairs * sizeof(emr::NetPair), "pair table", s));
    emr::NetEdgeArgs ea{};
    ea.conn_offset = P.coffset.as<int64_t>();
    ea.conn_cell = P.cell.as<uint32_t>();
    ea.conn_w = P.w.as<float>();
    ea.n_pairs = P.n_pairs;
    ea.total = P.ctotal;
    ea.src_offsets = P.shared() ? nullptr : P.src_offs.as<int64_t>();
    ea.src_cell = P.shared() ? nullptr : P.src_cell.as<uint32_t>();
    ea.sub_dir = d_dir;
    ea.n_sub = (uint32_t)N.n_sub;
    ea.n_genomes = G;
    ea.known = N.known.as<uint32_t>();
    ea.rank = rank.as<uint32_t>();
    ea.words = N.words;
    ea.seg = seg.as<int64_t>() + k * G;
    ea.raw_edge = raw_edge.as<int64_t>();
    ea.raw_node = raw_node.as<int64_t>();
    ea.pairs = pairs.as<emr::NetPair>();
    ea.eu = eu.as<uint32_t>();
    ea.ev = ev.as<uint32_t>();
    ea.ew = ew.as<float>();
    ea.e_raw = e_raw;
    ea.err = d_err;
    NET_HIP(emr_launch_net(2, &ea, s));
    NET_HIP(emr_launch_net(3, &ea, s));
  }
  // pruning: flags, then passes over every edge until one changes nothing
  emr::NetFlagArgs fa{d_dir, raw_node.as<int64_t>(), flags.as<uint16_t>(), kept_n.as<uint32_t>(),
                      N.node_offset.as<int64_t>(), (uint32_t)N.n_sub, G,
                      reinterpret_cast<int64_t*>(d_err + 2 + emr::kNetPasses)};
  NET_HIP(emr_launch_net(4, &fa, s));
  emr::NetReachArgs rr{eu.as<uint32_t>(), ev.as<uint32_t>(), flags.as<uint16_t>(), d_err + 1, 0u,
                       e_raw, n_raw};
  // a pass that changes something sets at least one more flag: 2 n_raw passes bound the loop
  const int64_t max_pass = 2 * n_raw + 2;
  emr::NetNodeArgs na{N.known.as<uint32_t>(), rank.as<uint32_t>(), N.words,
                      raw_node.as<int64_t>(), flags.as<uint16_t>(), N.d_slots.as<int32_t>(),
                      N.node_offset.as<int64_t>(), gid.as<uint32_t>(), N.node_cell.as<uint32_t>(),
                      N.node_in.as<int32_t>(), d_err, (uint32_t)N.n_sub, G};
  // Each batch of passes ends with the numbering its flags give, which stands if the batch settled:
  // the wait that looks at the passes then brings the kept node count too.
  int64_t kept_nodes = (int64_t)G * N.n_sub;  // (without edges nothing but the substrate is kept)
  if (e_raw == 0) {
    NET_HIP(emr_launch_net(6, &fa, s));
    NET_HIP(emr_launch_net(7, &na, s));
  }
  for (int64_t pass = 0; e_raw > 0; pass += emr::kNetPasses) {
    if (pass > max_pass)
      return failf(EMR_E_DEVICE, "networks: pruning did not settle in %lld passes",
                   (long long)max_pass);
    if (pass > 0) NET_HIP(hipMemsetAsync(d_err + 1, 0, 4 * emr::kNetPasses, s));
    for (rr.pass = 0; rr.pass < (uint32_t)emr::kNetPasses; ++rr.pass)
      NET_HIP(emr_launch_net(5, &rr, s));
    NET_HIP(emr_launch_net(6, &fa, s));
    NET_HIP(emr_launch_net(7, &na, s));
    struct { uint32_t changed, unused; int64_t kept; } seen;
    static_assert(sizeof seen == 16, "the last pass word, a word between, the count");
    NET_TRY(to_host(&seen, d_err + emr::kNetPasses, sizeof seen, s));
    if (seen.changed != 0) continue;
    if (seen.kept < 0 || seen.kept > n_raw)
      return failf(EMR_E_DEVICE, "networks: %lld kept nodes of %lld", (long long)seen.kept,
                   (long long)n_raw);
    kept_nodes = seen.kept;
    break;
  }
  // kept edges grouped by destination, each group in raw order: a stable sort by destination. The
  // dropped edges' key is the kept node count: a key past the raw node count would cost a third
  // radix pass where 17 bits number the raw nodes and 16 the kept ones.
  const uint32_t sentinel = (uint32_t)kept_nodes;
  Dev keys, vals, skeys, svals, tmp;
  NET_TRY(alloc(keys, (size_t)e_raw * 4, "edge keys", s));
  NET_TRY(alloc(vals, (size_t)e_raw * 8, "edge values", s));
  NET_TRY(alloc(skeys, (size_t)e_raw * 4, "edge keys", s));
  NET_TRY(alloc(svals, (size_t)e_raw * 8, "edge values", s));
  if (e_raw > 0) {
    emr::NetKeyArgs ka{eu.as<uint32_t>(), ev.as<uint32_t>(), ew.as<float>(), flags.as<uint16_t>(),
                       gid.as<uint32_t>(), keys.as<uint32_t>(), vals.as<uint64_t>(), e_raw, n_raw,
                       sentinel, d_err};
    NET_HIP(emr_launch_net(8, &ka, s));
    int bits = 1;
    while (bits < 32 && ((uint64_t)1 << bits) <= (uint64_t)sentinel) ++bits;  // keys <= sentinel
    size_t tb = 0;
    NET_HIP(emr_net_sort(nullptr, &tb, keys.as<uint32_t>(), skeys.as<uint32_t>(),
                         vals.as<uint64_t>(), svals.as<uint64_t>(), (uint32_t)e_raw, bits, s));
    NET_TRY(alloc(tmp, tb, "sort storage", s));
    NET_HIP(emr_net_sort(tmp.p, &tb, keys.as<uint32_t>(), skeys.as<uint32_t>(),
                         vals.as<uint64_t>(), svals.as<uint64_t>(), (uint32_t)e_raw, bits, s));
  }
  emr::NetSplitArgs sa{skeys.as<uint32_t>(), svals.as<uint64_t>(), N.node_offset.as<int64_t>(),
                       N.in_offset.as<int64_t>(), sum.as<int64_t>(), N.in_src.as<uint32_t>(),
                       N.in_w.as<float>(), e_raw, n_raw, sentinel, G, d_err};
  NET_HIP(emr_launch_net(14, &sa, s));
  std::vector<int64_t> off(2 * ((size_t)G + 1) + 1);
  NET_TRY(to_host(off.data(), sum.p, off.size() * 8, s));
  if (off.back() != 0)
    return failf(EMR_E_DEVICE, "networks: a network kernel flagged an internal error (0x%llx)",
                 (unsigned long long)off.back());
  N.nodes = off[G];
  N.edges = off[2 * (size_t)G + 1];
  if (N.nodes < 0 || N.nodes > n_raw || N.edges < 0 || N.edges > e_raw)
    return failf(EMR_E_DEVICE, "networks: %lld nodes of %lld, %lld kept edges of %lld",
                 (long long)N.nodes, (long long)n_raw, (long long)N.edges, (long long)e_raw);
  // The arrays of the networks were sized by the raw nodes and edges, so that nothing waited for the
  // kept ones; where pruning left less than half, that moves, and the raw size goes back to the cache.
  const Fit kept[] = {
      {&N.node_cell, (size_t)N.nodes * 4, "network nodes"},
      {&N.node_in, (size_t)N.nodes * 4, "network input numbers"},
      {&N.in_offset, (size_t)(N.nodes + 1) * 8, "network edge offsets"},
      {&N.in_src, (size_t)N.edges * 4, "network edges"},
      {&N.in_w, (size_t)N.edges * 4, "network edges"}};
  Fit move[emr::kNetFits];
  int moves = 0;
  for (const Fit& k : kept)
    if (k.d->bytes > 2 * k.bytes + kFitBytes) move[moves++] = k;
  if (moves > 0) NET_TRY(fit(move, moves, s));
  return order_genomes(N, off.data(), off.data() + G + 1, s);
}

// The genomes in the order of the activation launches: by class of node count (the classes of
// run_forward), the largest load first inside a class.
struct RunClass {
  uint32_t lds;  // LDS of the class's genomes, at most
  uint32_t q;    // float4 pattern groups of a workgroup, at most
};
// The more patterns share one read of the edges the better, as long as two workgroups of 16 waves
// share a CU's LDS: 80 KB at 4, 2 and then 1 float4 of patterns per node, else the whole
// 160 KB. The last class holds what does not fit and always runs stepwise.
constexpr RunClass kRunClass[] = {{80u << 10, 4}, {80u << 10, 2},
                                  {80u << 10, 1}, {160u << 10, 1}, {0xFFFFFFFFu, 1}};
constexpr int kRunClasses = sizeof kRunClass / sizeof kRunClass[0];
// The batches of 64 edges of a genome's nodes beyond one each, as the two totals let them be estimated.
double run_batches(int64_t nodes, int64_t edges) {
  return std::max(0.0, (double)edges / 64.0 - 0.5 * (double)nodes);
}
static_assert(kRunClasses <= emr::kNetRanges && kRunClass[kRunClasses - 2].lds == emr::kNetRunLds,
              "a range per class");

emr_status order_genomes(emr_networks& N, const int64_t* node_off, const int64_t* edge_off,
                         hipStream_t s) {
  const uint32_t G = (uint32_t)N.n_genomes;
  std::vector<uint32_t>& order = N.order_host;
  order.resize(G);
  std::vector<uint8_t> cls(G);
  for (uint32_t g = 0; g < G; ++g) {
    order[g] = g;
    const int64_t n = node_off[g + 1] - node_off[g];
    int c = 0;
    while (c + 1 < kRunClasses &&
           (n > (int64_t)emr::kNetRunLds / 32 || edge_off[g + 1] - edge_off[g] > INT32_MAX ||
            emr::net_run_lds((uint32_t)n, kRunClass[c].q) > kRunClass[c].lds))
      ++c;
    cls[g] = (uint8_t)c;
  }
  auto edges = [&](uint32_t g) { return edge_off[g + 1] - edge_off[g]; };
  auto nodes = [&](uint32_t g) { return node_off[g + 1] - node_off[g]; };
  auto load = [&](uint32_t g) {  // (a batch costs about three quarters of a node)
    return (double)nodes(g) + 0.75 * run_batches(nodes(g), edges(g));
  };
  std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) {
    return cls[a] != cls[b] ? cls[a] < cls[b] : load(a) > load(b);
  });
  N.order_load.resize(G);
  N.order_nodes.resize(G);
  N.nodes_before.assign(G + 1, 0);
  N.edges_before.assign(G + 1, 0);
  N.batches_before.assign(G + 1, 0.0);
  N.most_before.assign(G + 1, 0);
  N.class_first.assign(kRunClasses + 1, 0);
  for (uint32_t k = 0; k < G; ++k) {
    N.order_load[k] = load(order[k]);
    N.order_nodes[k] = (uint32_t)nodes(order[k]);
    N.nodes_before[k + 1] = N.nodes_before[k] + nodes(order[k]);
    N.edges_before[k + 1] = N.edges_before[k] + edges(order[k]);
    N.batches_before[k + 1] = N.batches_before[k] + run_batches(nodes(order[k]), edges(order[k]));
    const bool first = k == 0 || cls[order[k]] != cls[order[k - 1]];
    N.most_before[k + 1] = std::max(N.order_nodes[k], first ? 0u : N.most_before[k]);
    ++N.class_first[cls[order[k]] + 1];
  }
  for (int c = 0; c < kRunClasses; ++c) N.class_first[c + 1] += N.class_first[c];
  NET_TRY(alloc(N.order, (size_t)G * 4, "activation order", s));
  return to_device(N.order.p, order.data(), (size_t)G * 4, s);
}

// The patterns (and targets) on the device: small ones as kernel arguments, others staged in
// pinned memory and copied on the stream (the staging is rewritten only after the previous
// call's copy has completed).
emr_status stage_patterns(emr_networks& M, const float* patterns, size_t n_pat,
                          const float* targets, size_t n_tgt, hipStream_t s) {
  const size_t need = (n_pat + n_tgt) * 4;
  if (M.patterns.bytes < need || !M.patterns.p)
    NET_TRY(alloc(M.patterns, need, "input patterns", s));
  if (n_pat + n_tgt <= emr::kNetStageFloats) {
    emr::NetStageArgs a{};
    a.dst = M.patterns.as<float>();
    a.n = (uint32_t)(n_pat + n_tgt);
    std::memcpy(a.v, patterns, n_pat * 4);
    if (n_tgt) std::memcpy(a.v + n_pat, targets, n_tgt * 4);
    NET_HIP(emr_launch_net(12, &a, s));
    return EMR_OK;
  }
  if (!M.pin_done) NET_HIP(hipEventCreateWithFlags(&M.pin_done, hipEventDisableTiming));
  if (M.pin_pending) NET_HIP(hipEventSynchronize(M.pin_done));
  M.pin_pending = false;
  if (M.pin_bytes < need || !M.pin) {
    if (M.pin) (void)hipHostFree(M.pin);
    M.pin = nullptr;
    M.pin_bytes = 0;
    if (hipHostMalloc(&M.pin, need, hipHostMallocDefault) != hipSuccess) {
      M.pin = nullptr;
      (void)hipGetLastError();
      return failf(EMR_E_NOMEM, "networks: cannot allocate %zu bytes of pinned staging", need);
    }
    M.pin_bytes = need;
  }
  std::memcpy(M.pin, patterns, n_pat * 4);
  if (n_tgt) std::memcpy(static_cast<float*>(M.pin) + n_pat, targets, n_tgt * 4);
  NET_HIP(hipMemcpyAsync(M.patterns.p, M.pin, need, hipMemcpyHostToDevice, s));
  NET_HIP(hipEventRecord(M.pin_done, s));
  M.pin_pending = true;
  return EMR_OK;
}

// Times of an activation's parts, in us, measured on networks of 8 to 2484 nodes alone and on 30 to
// 1000 networks together. A fused run takes kLaunch and the longer of its longest workgroup (per step
// kStep, kNode[q] a node, q = 1, 2 and 4 pattern groups, and kBatch a further batch of 64 edges) and of
// all of them over the kSlots that the chip holds. The stepwise kernels take kSteps and per step
// kStepLaunch, or the time of their nodes and edges for all pattern blocks; a launch over some of the
// genomes has a row of workgroups as long as the largest for each (kStepSlot a node's place). The two
// follow each other on the stream.
struct RunTimes {
  static constexpr double kLaunch = 3.0, kStep = 0.8, kNode[3] = {0.028, 0.036, 0.045};
  static constexpr double kBatch = 0.026, kSlots = 512.0;
  static constexpr double kSteps = 12.0, kStepLaunch = 4.2, kStepNode = 2e-4, kStepEdge = 9.5e-7,
                          kStepSlot = 4e-5;
  static constexpr double kLongest = 2.5e5;  // a longer workgroup is not fused
};
constexpr int32_t kFusedSteps = 1024;  // nor are more steps (one launch stays below a second)

// Where each class's fused genomes begin (those before, its largest loads, run stepwise): the least
// estimated time over cuts at a load, from none stepwise but those that have to be to all.
struct RunCut {
  uint32_t first[kRunClasses];
  double us;
};
RunCut cut_at(const emr_networks& N, double load, int64_t pblocks, const uint32_t* q_of, double steps) {
  using T = RunTimes;
  RunCut r{};
  double longest = 0.0, work = 0.0, step_nodes = 0.0, step_edges = 0.0, stepwise = 0.0, most = 0.0;
  for (int c = 0; c < kRunClasses; ++c) {
    const uint32_t k0 = N.class_first[c], k1 = N.class_first[c + 1];
    const int qi = q_of[c] == 1 ? 0 : (q_of[c] == 2 ? 1 : 2);
    const double limit = std::min(load, (T::kLongest / std::max(steps, 1.0) - T::kStep) / T::kNode[qi]);
    uint32_t k = k1;
    if (c + 1 < kRunClasses && steps <= kFusedSteps)
      k = (uint32_t)(std::partition_point(N.order_load.begin() + k0, N.order_load.begin() + k1,
                                          [&](double l) { return l > limit; }) -
                     N.order_load.begin());
    r.first[c] = k;
    if (k > k0) {
      step_nodes += (double)(N.nodes_before[k] - N.nodes_before[k0]);
      step_edges += (double)(N.edges_before[k] - N.edges_before[k0]);
      stepwise += (double)(k - k0);
      most = std::max(most, (double)N.most_before[k]);
    }
    if (k == k1) continue;
    longest = std::max(longest, T::kStep + T::kNode[qi] * (double)N.order_nodes[k] +
                                    T::kBatch * (N.batches_before[k + 1] - N.batches_before[k]));
    work += (double)((pblocks + q_of[c] - 1) / q_of[c]) *
            (T::kStep * (double)(k1 - k) +
             T::kNode[qi] * (double)(N.nodes_before[k1] - N.nodes_before[k]) +
             T::kBatch * (N.batches_before[k1] - N.batches_before[k]));
  }
  if (longest > 0.0) r.us += T::kLaunch + steps * std::max(longest, work / T::kSlots);
  if (stepwise > 0.0) {
    const double slots = stepwise < (double)N.n_genomes ? stepwise * most : step_nodes;
    r.us += T::kSteps +
            steps * std::max(T::kStepLaunch,
                             (double)pblocks * (T::kStepNode * step_nodes + T::kStepEdge * step_edges +
                                                T::kStepSlot * (slots - step_nodes)));
  }
  return r;
}
RunCut best_cut(const emr_networks& N, int64_t pblocks, const uint32_t* q_of, int32_t steps) {
  double largest = 0.0;
  for (int c = 0; c + 1 < kRunClasses; ++c)
    if (N.class_first[c] < N.class_first[c + 1])
      largest = std::max(largest, N.order_load[N.class_first[c]]);
  RunCut best = cut_at(N, largest, pblocks, q_of, steps);
  // (nothing is shorter than the launches of the stepwise kernels)
  if (best.us <= RunTimes::kSteps + steps * RunTimes::kStepLaunch) return best;
  for (int j = 0; j < 9; ++j) {
    largest = j < 8 ? 0.5 * largest : 0.0;
    const RunCut r = cut_at(N, largest, pblocks, q_of, steps);
    if (r.us < best.us) best = r;
  }
  return best;
}

emr_status run_forward(const emr_networks* N, const float* patterns, int32_t n_patterns,
                       int32_t steps, float* outputs, float* fitness, const float* targets,
                       hipStream_t s) {
  emr_networks& M = const_cast<emr_networks&>(*N);
  int dev = 0;
  NET_HIP(hipGetDevice(&dev));
  if (dev != N->device)
    return failf(EMR_E_INVAL, "networks: built on device %d, current device is %d", N->device, dev);
  const int64_t pblocks = (n_patterns + 3) / 4;
  if (pblocks * (N->nodes ? N->nodes : 1) > ((int64_t)1 << 40))
    return failf(EMR_E_LIMIT, "networks: too many nodes x patterns");
  const size_t n_pat = (size_t)n_patterns * (size_t)N->n_in;
  // A class's pattern groups per workgroup, no more than there are.
  uint32_t q_of[kRunClasses];
  for (int c = 0; c < kRunClasses; ++c) {
    uint32_t q = 1;
    while (q < kRunClass[c].q && (int64_t)q < pblocks) q *= 2;
    q_of[c] = q;
  }
  const RunCut cut = best_cut(*N, pblocks, q_of, steps);
  const uint32_t* fused_first = cut.first;
  emr::NetList list{};
  list.order = N->order.as<uint32_t>();
  list.n_genomes = (uint32_t)N->n_genomes;
  for (int c = 0; c < kRunClasses; ++c) {
    const uint32_t k0 = N->class_first[c], k1 = fused_first[c];
    for (uint32_t k = k0; k < k1; ++k) list.max_nodes = std::max(list.max_nodes, N->order_nodes[k]);
    list.first[c] = k0;
    list.count[c] = k1 - k0;
    list.total += k1 - k0;
  }
  // every genome stepwise: the kernels take the nodes as they lie, without the list
  if (list.total == list.n_genomes && list.total <= 65535u) {
    list.order = nullptr;
    for (int c = 0; c < kRunClasses; ++c) list.first[c] = list.count[c] = 0;
    list.count[0] = list.total;
  }
  // (few patterns of stepwise kernels alone are the initial state's arguments: a launch fewer)
  const bool by_value = list.order == nullptr && n_pat <= emr::kNetStageFloats;
  if (!by_value)
    NET_TRY(stage_patterns(M, patterns, n_pat, targets, targets ? (size_t)n_patterns : 0, s));
  emr::NetRunArgs ra{};
  ra.order = N->order.as<uint32_t>();
  ra.node_offset = N->node_offset.as<int64_t>();
  ra.node_in = N->node_in.as<int32_t>();
  ra.in_offset = N->in_offset.as<int64_t>();
  ra.in_src = N->in_src.as<uint32_t>();
  ra.in_w = N->in_w.as<float>();
  ra.patterns = M.patterns.as<float>();
  ra.targets = targets ? M.patterns.as<float>() + n_pat : nullptr;
  ra.out_node = N->d_out_node.as<int32_t>();
  ra.outputs = outputs;
  ra.fitness = fitness;
  ra.nodes = N->nodes;
  ra.edges = N->edges;
  ra.n_genomes = (uint32_t)N->n_genomes;
  ra.n_inputs = (uint32_t)N->n_in;
  ra.n_outputs = (uint32_t)N->n_out;
  ra.n_patterns = (uint32_t)n_patterns;
  ra.steps = (uint32_t)steps;
  // the classes of 80 KB in one launch, the largest genomes' (the longest workgroups) first; then
  // the class that takes a whole CU's LDS
  for (int part = 0; part < 2; ++part) {
    const int lo = part == 0 ? 0 : kRunClasses - 2, hi = part == 0 ? kRunClasses - 2 : kRunClasses - 1;
    uint64_t blocks = 0;
    ra.lds_bytes = 0;
    for (int r = 0; r < emr::kNetRanges; ++r) ra.count[r] = 0;
    for (int c = hi - 1, r = 0; c >= lo; --c, ++r) {
      ra.first[r] = fused_first[c];
      ra.count[r] = N->class_first[c + 1] - fused_first[c];
      ra.q[r] = q_of[c];
      ra.blocks[r] = (uint32_t)((pblocks + q_of[c] - 1) / q_of[c]);
      blocks += (uint64_t)ra.count[r] * ra.blocks[r];
      for (uint32_t i = fused_first[c]; i < N->class_first[c + 1]; ++i)
        ra.lds_bytes = std::max(ra.lds_bytes, emr::net_run_lds(N->order_nodes[i], q_of[c]));
    }
    if (blocks > 0x7FFFFFFFull)
      return failf(EMR_E_LIMIT, "networks: too many genomes x patterns");
    if (blocks > 0) NET_HIP(emr_launch_net(13, &ra, s));
  }
  if (list.total > 0) {
    // two state buffers of [pblocks][nodes] float4
    const size_t half = (size_t)pblocks * (size_t)(N->nodes ? N->nodes : 1) * 16;
    if (M.state.bytes < 2 * half) NET_TRY(alloc(M.state, 2 * half, "node states", s));
    float* buf[2] = {M.state.as<float>(), reinterpret_cast<float*>(M.state.as<char>() + half)};
    // (a launch covers at most 65535 genomes)
    const emr::NetList whole = list;
    uint32_t done = 0;
    while (done < whole.total) {
      uint32_t skip = done, left = std::min(whole.total - done, 65535u);
      list.total = left;
      done += left;
      for (int c = 0; c < kRunClasses; ++c) {
        const uint32_t cut = std::min(skip, whole.count[c]);
        const uint32_t n = std::min(whole.count[c] - cut, left);
        list.first[c] = whole.first[c] + cut;
        list.count[c] = n;
        skip -= cut;
        left -= n;
      }
      emr::NetStateArgs sa{list, N->node_offset.as<int64_t>(), N->node_in.as<int32_t>(),
                           by_value ? nullptr : M.patterns.as<float>(), buf[0], N->nodes,
                           (uint32_t)N->n_in, (uint32_t)n_patterns, (uint32_t)pblocks, {}};
      if (by_value) std::memcpy(sa.v, patterns, n_pat * 4);
      NET_HIP(emr_launch_net(9, &sa, s));
      int cur = 0;
      for (int32_t t = 0; t < steps; ++t, cur ^= 1) {
        emr::NetStepArgs st{list, N->node_offset.as<int64_t>(), N->node_in.as<int32_t>(),
                            N->in_offset.as<int64_t>(), N->in_src.as<uint32_t>(),
                            N->in_w.as<float>(), buf[cur], buf[cur ^ 1], N->nodes,
                            (uint32_t)pblocks};
        NET_HIP(emr_launch_net(10, &st, s));
      }
      emr::NetOutArgs oa{};
      oa.list = list;
      oa.node_offset = N->node_offset.as<int64_t>();
      oa.out_node = N->d_out_node.as<int32_t>();
      oa.state = buf[cur];
      if (targets) std::memcpy(oa.target, targets, sizeof oa.target);
      oa.outputs = outputs;
      oa.fitness = fitness;
      oa.nodes = N->nodes;
      oa.n_outputs = (uint32_t)N->n_out;
      oa.n_patterns = (uint32_t)n_patterns;
      NET_HIP(emr_launch_net(11, &oa, s));
    }
  }
  if (!M.done) NET_HIP(hipEventCreateWithFlags(&M.done, hipEventDisableTiming));
  NET_HIP(hipEventRecord(M.done, s));
  M.done_pending = true;
  return EMR_OK;
}

// Every phase and the assembly; synchronizes with the stream at the end.
emr_status build_all(Build& B, int32_t n_substrate, int32_t iterations) {
  emr_networks& N = *B.net;
  NET_TRY(alloc(N.known, (size_t)N.n_genomes * (size_t)N.words * 4, "hidden-cell bitmaps", B.s));
  NET_HIP(hipMemsetAsync(N.known.p, 0, N.known.bytes, B.s));
  NET_TRY(alloc(N.d_slots, N.slots.size() * 4, "substrate slots", B.s));
  NET_TRY(to_device(N.d_slots.p, N.slots.data(), N.slots.size() * 4, B.s));
  std::vector<int32_t> out_node((size_t)N.n_out);
  for (int32_t j = 0; j < n_substrate; ++j)
    if (N.slots[(size_t)n_substrate + j] >= 0) out_node[(size_t)N.slots[(size_t)n_substrate + j]] = j;
  NET_TRY(alloc(N.d_out_node, out_node.size() * 4, "output nodes", B.s));
  NET_TRY(to_device(N.d_out_node.p, out_node.data(), out_node.size() * 4, B.s));

  N.phases.push_back(std::make_unique<Phase>());
  N.phases[0]->sources = N.substrate;
  for (int32_t it = 0;; ++it) {
    Phase& P = *N.phases.back();
    NET_TRY(discover_phase(B, P));
    const bool more = it < iterations;
    auto next = more ? std::make_unique<Phase>() : nullptr;
    NET_TRY(hidden_phase(B, P));
    NET_TRY(express_phase(B, P));
    NET_TRY(finish_phase(B, P, next.get()));
    if (!more || P.n_new == 0) break;
    N.phases.push_back(std::move(next));
  }
  NET_TRY(assemble(B));
  NET_HIP(hipStreamSynchronize(B.s));
  return EMR_OK;
}

}  // namespace

extern "C" {

emr_status emr_build_networks(const emr_population* pop, const emr_source* substrate,
                              int32_t n_substrate, int32_t depth, float theta, int32_t type_mask,
                              float w_min, int32_t iterations, emr_networks** out, void* stream) {
  if (!out) return failf(EMR_E_INVAL, "networks: out is NULL");
  *out = nullptr;
  if (!pop || !substrate) return failf(EMR_E_INVAL, "networks: NULL population or substrate");
  if (n_substrate < 1 || n_substrate > kMaxSubstrate)
    return failf(EMR_E_INVAL, "networks: n_substrate %d outside [1, %d]", n_substrate,
                 kMaxSubstrate);
  if (depth < 1 || depth > EMR_MAX_DEPTH)
    return failf(EMR_E_INVAL, "networks: depth %d outside [1, %d]", depth, EMR_MAX_DEPTH);
  if (type_mask < 1 || type_mask > EMR_CONN_ALL)
    return failf(EMR_E_INVAL, "networks: type_mask %d outside [1, 15]", type_mask);
  if (iterations < 0 || iterations > kMaxIterations)
    return failf(EMR_E_INVAL, "networks: iterations %d outside [0, %d]", iterations,
                 kMaxIterations);
  if (std::isnan(theta) || std::isnan(w_min))
    return failf(EMR_E_INVAL, "networks: theta and w_min must not be NaN");
  auto net = std::make_unique<emr_networks>();
  emr_networks& N = *net;
  N.n_sub = n_substrate;
  N.depth = depth;
  N.substrate.assign(substrate, substrate + n_substrate);
  N.slots.assign((size_t)2 * n_substrate, -1);
  for (int32_t j = 0; j < n_substrate; ++j) {
    const emr_source& q = substrate[j];
    if (q.dir != EMR_DIR_OUT && q.dir != EMR_DIR_IN)
      return failf(EMR_E_INVAL, "networks: substrate source %d has direction %d", j, q.dir);
    if (!std::isfinite(q.x) || !std::isfinite(q.y))
      return failf(EMR_E_INVAL, "networks: substrate source %d is not finite", j);
    if (q.dir == EMR_DIR_OUT) N.slots[j] = N.n_in++;
    else N.slots[(size_t)n_substrate + j] = N.n_out++;
  }
  if (N.n_in == 0 || N.n_out == 0)
    return failf(EMR_E_INVAL, "networks: the substrate needs an input and an output");
  NET_TRY(emr_population_info(pop, &N.n_genomes, nullptr, nullptr, nullptr));
  if (N.n_genomes < 1) return failf(EMR_E_INVAL, "networks: empty population");
  NET_HIP(hipGetDevice(&N.device));
  NET_TRY(emr_cell_words(depth, &N.words));
  Build B{pop, &N, theta, type_mask, w_min, (hipStream_t)stream};
  const emr_status st = build_all(B, n_substrate, iterations);
  // after a failure, nothing queued may still use the buffers the handle gives back
  if (st != EMR_OK) {
    (void)hipStreamSynchronize(B.s);
    return st;
  }
  *out = net.release();
  return EMR_OK;
}

emr_status emr_networks_info(const emr_networks* net, emr_network_info* info) {
  if (!net || !info) return failf(EMR_E_INVAL, "networks: NULL argument");
  info->n_genomes = net->n_genomes;
  info->n_substrate = net->n_sub;
  info->n_inputs = net->n_in;
  info->n_outputs = net->n_out;
  info->depth = net->depth;
  info->phases = (int32_t)net->phases.size();
  info->nodes = net->nodes;
  info->edges = net->edges;
  info->node_offset = net->node_offset.as<int64_t>();
  info->node_cell = net->node_cell.as<uint32_t>();
  info->in_offset = net->in_offset.as<int64_t>();
  info->in_src = net->in_src.as<uint32_t>();
  info->in_w = net->in_w.as<float>();
  info->known = net->known.as<uint32_t>();
  info->known_words = net->words;
  return EMR_OK;
}

emr_status emr_networks_phase(const emr_networks* net, int32_t phase, emr_network_phase* out) {
  if (!net || !out) return failf(EMR_E_INVAL, "networks: NULL argument");
  if (phase < 0 || phase >= (int32_t)net->phases.size())
    return failf(EMR_E_INVAL, "networks: phase %d outside [0, %zu)", phase, net->phases.size());
  const Phase& P = *net->phases[phase];
  out->sources = P.sources.data();
  out->n_sources = (int32_t)P.sources.size();
  out->src_offsets = P.offs_ptr();
  out->src_cell = P.shared() ? nullptr : P.src_cell.as<uint32_t>();
  out->n_pairs = P.n_pairs;
  out->parent = P.parent.as<uint32_t>();
  out->w4 = P.w4.as<float>();
  out->pair_offset = P.roffset.as<int64_t>();
  out->records = P.rtotal;
  out->conn_cell = P.cell.as<uint32_t>();
  out->conn_w = P.w.as<float>();
  out->conn_offset = P.coffset.as<int64_t>();
  out->connections = P.ctotal;
  return EMR_OK;
}

emr_status emr_activate(const emr_networks* net, const float* inputs, int32_t n_patterns,
                        int32_t steps, float* outputs, void* stream) {
  if (!net || !outputs) return failf(EMR_E_INVAL, "networks: NULL argument");
  if (n_patterns < 1 || n_patterns > kMaxPatterns)
    return failf(EMR_E_INVAL, "networks: n_patterns %d outside [1, %d]", n_patterns, kMaxPatterns);
  if (steps < 0 || steps > kMaxSteps)
    return failf(EMR_E_INVAL, "networks: steps %d outside [0, %d]", steps, kMaxSteps);
  if (!inputs) return failf(EMR_E_INVAL, "networks: inputs is NULL");
  return run_forward(net, inputs, n_patterns, steps, outputs, nullptr, nullptr,
                     (hipStream_t)stream);
}

emr_status emr_xor_fitness(const emr_networks* net, int32_t bias_input, int32_t steps,
                           float* fitness, void* stream) {
  if (!net || !fitness) return failf(EMR_E_INVAL, "networks: NULL argument");
  if (steps < 0 || steps > kMaxSteps)
    return failf(EMR_E_INVAL, "networks: steps %d outside [0, %d]", steps, kMaxSteps);
  if (net->n_out != 1) return failf(EMR_E_INVAL, "networks: XOR needs one output");
  if (bias_input < -1 || bias_input >= net->n_in || net->n_in != 2 + (bias_input >= 0 ? 1 : 0))
    return failf(EMR_E_INVAL, "networks: XOR needs inputs a, b and at most one bias input "
                 "(%d inputs, bias input %d)", net->n_in, bias_input);
  // (a, b) = (0,0), (0,1), (1,0), (1,1) on the non-bias inputs in order; the bias input holds 1
  static const float ab[4][2] = {{0.f, 0.f}, {0.f, 1.f}, {1.f, 0.f}, {1.f, 1.f}};
  static const float target[4] = {0.f, 1.f, 1.f, 0.f};
  std::vector<float> pat((size_t)4 * net->n_in);
  for (int p = 0; p < 4; ++p) {
    int c = 0;
    for (int j = 0; j < net->n_in; ++j) pat[(size_t)p * net->n_in + j] = j == bias_input ? 1.f : ab[p][c++];
  }
  return run_forward(net, pat.data(), 4, steps, nullptr, fitness, target, (hipStream_t)stream);
}

emr_status emr_copy_to_host(void* host, const void* device, int64_t bytes, void* stream) {
  if (bytes < 0 || (bytes > 0 && (!host || !device)))
    return failf(EMR_E_INVAL, "copy: bad arguments");
  return to_host(host, device, (size_t)bytes, (hipStream_t)stream);
}

void emr_free_networks(emr_networks* net) { delete net; }

}  // extern "C"
