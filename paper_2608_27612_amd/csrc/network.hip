// gfx950 kernels that turn the discovered substrate into networks and run them (the networks the
// experiments evaluate, Section 5): the hidden-cell bitmap's rank (node numbers), the expressed
// connections as edges between node numbers, pruning to the nodes on an input-to-output path, the
// kept nodes' numbering and their incoming edges grouped by destination, and synchronous
// activation over a batch of input patterns with an optional XOR fitness.
//
// Work over edges runs one thread per edge across the whole population: genomes are very unequal (a
// genome with a high-frequency CPPN can hold a large share of the population's edges), so no
// step may give one genome to one workgroup when its cost grows with the genome's edges beyond
// its share of the chip. Steps whose cost follows a genome's node count (its bitmap, its node
// numbering) run one workgroup per genome, and activation one per (genome, pattern block) where
// that takes less than a launch per step (the estimate is in networks.cpp). Numbering and
// layouts: network.h.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "emr_internal.h"
#include "network.h"

namespace emr {
namespace {

// Exclusive prefix sum over the workgroup's kNetThreads threads (every thread must call it);
// *total receives the sum. `part` holds one word per wave.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* part, uint32_t* total) {
  const uint32_t lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, (unsigned)o, kWave);
    if (lane >= (uint32_t)o) x += y;
  }
  if (lane == kWave - 1) part[wv] = x;
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kNetThreads / kWave; ++i) {
    const uint32_t p = part[i];
    before += (i < (int)wv) ? p : 0u;
    tot += p;
  }
  __syncthreads();  // `part` is free again
  *total = tot;
  return before + x - v;
}

// The r with off[r] <= i < off[r + 1], for off[0] <= i < off[n] (empty segments skipped).
__device__ __forceinline__ int64_t find_segment(const int64_t* off, int64_t n, int64_t i) {
  int64_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (off[mid] <= i) lo = mid;
    else hi = mid;
  }
  return lo;
}
// The same from a segment lo with off[lo] <= i on: a gallop, then a search (i is close to lo).
__device__ __forceinline__ int64_t find_segment_from(const int64_t* off, int64_t n, int64_t lo,
                                                     int64_t i) {
  int64_t step = 1, hi = lo + 1;
  while (hi < n && off[hi] <= i) {
    lo = hi;
    step *= 2;
    hi = n - lo > step ? lo + step : n;
  }
  while (hi - lo > 1) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (off[mid] <= i) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Raw node number of heap cell `cell` in genome g (n_sub + its rank among the genome's hidden
// cells), or kNoNode when the cell is not a hidden node.
__device__ __forceinline__ uint32_t node_of(const uint32_t* known, const uint32_t* rank,
                                            int64_t words, uint32_t g, uint32_t n_sub,
                                            uint32_t cell) {
  if (cell == 0u) return kNoNode;
  const uint32_t p = cell - 1u;  // grid position
  const int64_t w = (int64_t)(p >> 5);
  if (w >= words) return kNoNode;
  const uint32_t word = known[(int64_t)g * words + w];
  const uint32_t before = rank[(int64_t)g * words + w];  // (both reads go out together)
  const uint32_t b = p & 31u;
  return ((word >> b) & 1u) == 0u
             ? kNoNode
             : n_sub + before + (uint32_t)__builtin_popcount(word & ((1u << b) - 1u));
}

__device__ __forceinline__ float sigmoid_f(float z) { return 1.0f / (1.0f + expf(-z)); }

__device__ __forceinline__ float comp(const float4& v, uint32_t c) {
  return c == 0u ? v.x : (c == 1u ? v.y : (c == 2u ? v.z : v.w));
}

__device__ __forceinline__ int64_t grid_thread() {
  return (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
}
__device__ __forceinline__ int64_t grid_threads() { return (int64_t)gridDim.x * blockDim.x; }

}  // namespace

// ------------------------------------------------------------------------ node numbers
__global__ void __launch_bounds__(kNetThreads) k_net_rank(NetRankArgs A) {
  __shared__ uint32_t part[kNetThreads / kWave];
  for (uint32_t g = blockIdx.x; g < A.n_genomes; g += gridDim.x) {
    const uint32_t* k = A.known + (int64_t)g * A.words;
    uint32_t* r = A.rank + (int64_t)g * A.words;
    uint32_t run = 0;
    for (int64_t base = 0; base < A.words; base += 4 * kNetThreads) {
      const int64_t w0 = base + 4 * (int64_t)threadIdx.x;
      uint32_t c[4], s = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c[q] = w0 + q < A.words ? (uint32_t)__builtin_popcount(k[w0 + q]) : 0u;
        s += c[q];
      }
      uint32_t total;
      uint32_t acc = run + block_excl_scan(s, part, &total);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (w0 + q < A.words) r[w0 + q] = acc;
        acc += c[q];
      }
      run += total;
    }
    if (threadIdx.x == 0) A.hidden[g] = run;
  }
}

// ------------------------------------------------------------------------ raw edges
// One workgroup: the exclusive sums of the genomes' raw nodes and edges, and each phase's segment
// of a genome's edges. (These sums took the host a copy of every phase's offsets and a wait.)
__global__ void __launch_bounds__(kNetThreads) k_net_layout(NetLayoutArgs A) {
  __shared__ uint32_t part[kNetThreads / kWave];
  __shared__ uint64_t wide[kNetThreads];
  int64_t run_n = 0, run_e = 0;
  for (uint32_t base = 0; base < A.n_genomes; base += kNetThreads) {
    const uint32_t g = base + threadIdx.x;
    int64_t edges = 0;
    uint32_t n = 0;
    if (g < A.n_genomes) {
      n = A.n_sub + A.hidden[g];
      for (uint32_t k = 0; k < A.n_phases; ++k) {
        const int64_t* so = A.src_offsets[k];
        const int64_t p0 = so ? so[g] : (int64_t)g * A.n_sub;
        const int64_t p1 = so ? so[g + 1] : (int64_t)(g + 1) * A.n_sub;
        const int64_t len = A.conn_offset[k][p1] - A.conn_offset[k][p0];
        A.seg[(int64_t)k * A.n_genomes + g] = edges;  // (within the genome; its base added below)
        edges += len;
      }
    }
    uint32_t tn;
    const int64_t en = block_excl_scan(n, part, &tn);
    wide[threadIdx.x] = (uint64_t)edges;  // (a genome's edges can exceed 32 bits: a wide scan)
    __syncthreads();
    for (uint32_t o = 1; o < (uint32_t)kNetThreads; o <<= 1) {
      const uint64_t y = threadIdx.x >= o ? wide[threadIdx.x - o] : 0ull;
      __syncthreads();
      wide[threadIdx.x] += y;
      __syncthreads();
    }
    const int64_t te = (int64_t)wide[kNetThreads - 1];
    const int64_t ee = (int64_t)wide[threadIdx.x] - edges;
    if (g < A.n_genomes) {
      A.raw_node[g] = run_n + en;
      A.raw_edge[g] = run_e + ee;
      for (uint32_t k = 0; k < A.n_phases; ++k) A.seg[(int64_t)k * A.n_genomes + g] += run_e + ee;
    }
    run_n += tn;
    run_e += te;
    __syncthreads();  // `wide` is free again
  }
  if (threadIdx.x == 0) {
    A.raw_node[A.n_genomes] = run_n;
    A.raw_edge[A.n_genomes] = run_e;
    if (run_n != A.n_raw || run_e != A.e_raw) atomicOr(A.err, kNetErrIndex);
  }
}

// One thread per pair of a phase: what its connections' edges have in common.
__global__ void __launch_bounds__(kNetThreads) k_net_pairs(NetEdgeArgs A) {
  for (int64_t r = grid_thread(); r < A.n_pairs; r += grid_threads()) {
    uint32_t g, node, dir;
    int64_t first;
    if (A.src_offsets == nullptr) {
      g = (uint32_t)(r / A.n_sub);
      node = (uint32_t)(r % A.n_sub);
      dir = A.sub_dir[node];
      first = (int64_t)g * A.n_sub;
    } else {
      g = (uint32_t)find_segment(A.src_offsets, A.n_genomes, r);
      first = A.src_offsets[g];
      node = g < A.n_genomes ? node_of(A.known, A.rank, A.words, g, A.n_sub, A.src_cell[r]) : kNoNode;
      dir = 0u;
    }
    NetPair p{0, 0, 0, 0u, kNoNode, 0u, 0u};
    if (g >= A.n_genomes || node == kNoNode ||
        (int64_t)node >= A.raw_node[g + 1] - A.raw_node[g]) {
      atomicOr(A.err, kNetErrIndex);
    } else {
      p.delta = A.seg[g] - A.conn_offset[first];
      p.g_dir = g << 1 | dir;
      p.lo = A.raw_edge[g];
      p.hi = A.raw_edge[g + 1];
      p.base = (uint32_t)A.raw_node[g];  // (the host bounds the raw nodes below kNoNode)
      p.n = (uint32_t)(A.raw_node[g + 1] - A.raw_node[g]);
      p.node = node + p.base;
    }
    A.pairs[r] = p;
  }
}

// The raw edges of N connections i[k] of pair P (i[k] < 0: none), their reads in flight together.
template <int N>
__device__ __forceinline__ void net_edges(const NetEdgeArgs& A, const NetPair& P,
                                          const int64_t (&i)[N]) {
  const uint32_t g = P.g_dir >> 1;
  uint32_t cell[N], cn[N];
  float w[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    cell[k] = i[k] >= 0 ? A.conn_cell[i[k]] : 0u;
    w[k] = i[k] >= 0 ? A.conn_w[i[k]] : 0.0f;
  }
#pragma unroll
  for (int k = 0; k < N; ++k)
    cn[k] = node_of(A.known, A.rank, A.words, g, A.n_sub, cell[k]);  // (cell 0: none)
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (i[k] < 0) continue;
    const int64_t o = i[k] + P.delta;
    if (P.node == kNoNode || o < P.lo || o >= P.hi || o >= A.e_raw) {
      atomicOr(A.err, kNetErrIndex);
      continue;
    }
    const uint32_t c = cn[k] + P.base;
    const bool in = (P.g_dir & 1u) != 0u;
    uint32_t u = in ? c : P.node, v = in ? P.node : c;
    if (cn[k] == kNoNode) {
      u = v = kNoNode;  // the grid end is not a hidden node: dropped
    } else if (cn[k] >= P.n) {
      atomicOr(A.err, kNetErrIndex);
      u = v = kNoNode;
    }
    A.eu[o] = u;
    A.ev[o] = v;
    A.ew[o] = w[k];
  }
}

// Wave w takes the phase's connections [w span, (w + 1) span), 64 at a time. While they belong to
// one pair (most do: a few heavy genomes hold most connections, hundreds per pair) the pair is the
// wave's and only the grid end is looked up per lane; else each lane finds its pair from the step's
// first on. (A search of all pairs and genomes per connection: 455 us for 16.8M.)
__global__ void __launch_bounds__(kNetThreads) k_net_edges(NetEdgeArgs A, int64_t span) {
  const uint32_t lane = threadIdx.x % kWave;
  const int64_t wave = (int64_t)blockIdx.x * (kNetThreads / kWave) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t base = wave * span, end = base + span < A.total ? base + span : A.total;
  if (base >= end) return;
  uint32_t r = __builtin_amdgcn_readfirstlane(
      (uint32_t)find_segment(A.conn_offset, A.n_pairs, base));  // (pairs number below 2^32)
  int64_t r1 = A.conn_offset[r + 1];
  NetPair P = A.pairs[r];
  for (int64_t b = base; b < end; b += kWave) {
    if (b >= r1) {
      r = __builtin_amdgcn_readfirstlane(
          (uint32_t)find_segment_from(A.conn_offset, A.n_pairs, r, b));
      r1 = A.conn_offset[r + 1];
      P = A.pairs[r];
    }
    const int64_t i = b + lane;
    if (b + 4 * kWave <= r1 && b + 4 * kWave <= end) {
      const int64_t four[4] = {i, i + kWave, i + 2 * kWave, i + 3 * kWave};
      net_edges<4>(A, P, four);
      b += 3 * kWave;
      continue;
    }
    const int64_t one[1] = {i < end ? i : -1};
    if (i < r1 || i >= end)
      net_edges<1>(A, P, one);
    else
      net_edges<1>(A, A.pairs[find_segment_from(A.conn_offset, A.n_pairs, r, i)], one);
  }
}

// ------------------------------------------------------------------------ pruning
// Flags of every raw node before the passes: substrate inputs reach themselves, substrate
// outputs reach an output. One workgroup per genome (its nodes).
constexpr uint32_t kFwd = 1u, kBwd = 0x100u;  // a byte each: stored by themselves, read together
__global__ void __launch_bounds__(kNetThreads) k_net_flags(NetFlagArgs A) {
  for (uint32_t g = blockIdx.x; g < A.n_genomes; g += gridDim.x) {
    const int64_t nb = A.raw_node[g], n = A.raw_node[g + 1] - nb;
    for (int64_t j = threadIdx.x; j < n; j += blockDim.x)
      A.flags[nb + j] =
          (uint16_t)(j >= (int64_t)A.n_sub ? 0u : (A.sub_dir[j] == 0u ? kFwd : kBwd));
  }
}

// One pass over every raw edge of the population: u -> v carries reachability from an input
// forward (fwd[u] -> fwd[v]) and reachability of an output backward (bwd[v] -> bwd[u]). Flags only
// go from 0 to 1, so a thread reading a flag another thread is setting sees either value; a pass
// that changes nothing saw only values fixed since the launch began (every write of the previous
// pass is visible at launch), which is the fixed point. The host enqueues kNetPasses passes at a
// time (a wait for each costs more than the pass) and goes on until the last one changed nothing;
// a pass after one that changed nothing returns at once. Four edges per thread: the edges in two
// 16-byte loads, eight flag reads in flight.
__device__ __forceinline__ bool reach_edge(const NetReachArgs& A, uint32_t u, uint32_t v,
                                           uint32_t fu, uint32_t fv) {
  bool ch = false;
  uint8_t* bytes = reinterpret_cast<uint8_t*>(A.flags);
  if ((fu & kFwd) != 0u && (fv & kFwd) == 0u) {
    bytes[2 * (int64_t)v] = 1;
    ch = true;
  }
  if ((fv & kBwd) != 0u && (fu & kBwd) == 0u) {
    bytes[2 * (int64_t)u + 1] = 1;
    ch = true;
  }
  return ch;
}
__global__ void __launch_bounds__(kNetThreads) k_net_reach(NetReachArgs A) {
  if (A.pass > 0u && A.changed[A.pass - 1u] == 0u) return;
  bool ch = false;
  const int64_t quads = (A.edges + 3) / 4;
  for (int64_t q = grid_thread(); q < quads; q += grid_threads()) {
    uint32_t u[4], v[4], fu[4], fv[4];
    if (4 * q + 4 <= A.edges) {
      const uint4 a = reinterpret_cast<const uint4*>(A.eu)[q];
      const uint4 b = reinterpret_cast<const uint4*>(A.ev)[q];
      u[0] = a.x, u[1] = a.y, u[2] = a.z, u[3] = a.w;
      v[0] = b.x, v[1] = b.y, v[2] = b.z, v[3] = b.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        u[k] = 4 * q + k < A.edges ? A.eu[4 * q + k] : kNoNode;
        v[k] = 4 * q + k < A.edges ? A.ev[4 * q + k] : kNoNode;
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool ok = (int64_t)u[k] < A.nodes && (int64_t)v[k] < A.nodes;  // else a dropped edge
      fu[k] = ok ? A.flags[u[k]] : 0u;
      fv[k] = ok ? A.flags[v[k]] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) ch |= reach_edge(A, u[k], v[k], fu[k], fv[k]);
  }
  if (__ballot(ch) != 0ull && (threadIdx.x % kWave) == 0) A.changed[A.pass] = 1u;
}

__device__ __forceinline__ bool node_kept(uint32_t flags) {
  return flags == (kFwd | kBwd);
}

// Per genome: kept nodes (substrate nodes, and hidden ones reached from an input and reaching an
// output). One workgroup per genome (its nodes).
__global__ void __launch_bounds__(kNetThreads) k_net_kept(NetFlagArgs A) {
  __shared__ uint32_t part[kNetThreads / kWave];
  for (uint32_t g = blockIdx.x; g < A.n_genomes; g += gridDim.x) {
    const int64_t nb = A.raw_node[g], n = A.raw_node[g + 1] - nb;
    uint32_t kn = 0u;
    for (int64_t j = threadIdx.x; j < n; j += blockDim.x)
      if (j < (int64_t)A.n_sub || node_kept(A.flags[nb + j])) ++kn;
    uint32_t tn;
    block_excl_scan(kn, part, &tn);
    if (threadIdx.x == 0) A.kept_nodes[g] = tn;
  }
}

// One workgroup: the kept nodes' exclusive sums.
__global__ void __launch_bounds__(kNetThreads) k_net_number(NetFlagArgs A) {
  __shared__ uint32_t part[kNetThreads / kWave];
  int64_t run = 0;
  for (uint32_t base = 0; base < A.n_genomes; base += kNetThreads) {
    const uint32_t g = base + threadIdx.x;
    uint32_t t;
    const uint32_t e = block_excl_scan(g < A.n_genomes ? A.kept_nodes[g] : 0u, part, &t);
    if (g < A.n_genomes) A.node_offset[g] = run + e;
    run += t;
  }
  if (threadIdx.x == 0) {
    A.node_offset[A.n_genomes] = run;
    *A.total = run;
  }
}

// ------------------------------------------------------------------------ kept nodes
// One workgroup per genome: kept numbers in raw order and the input numbers, then the kept hidden
// nodes' heap cells.
__global__ void __launch_bounds__(kNetThreads) k_net_nodes(NetNodeArgs A) {
  __shared__ uint32_t part[kNetThreads / kWave];
  for (uint32_t g = blockIdx.x; g < A.n_genomes; g += gridDim.x) {
    const int64_t nb = A.raw_node[g], n = A.raw_node[g + 1] - nb;
    const int64_t NB = A.node_offset[g], NE = A.node_offset[g + 1];
    uint32_t run_id = 0u;
    for (int64_t base = 0; base < n; base += kNetThreads) {
      const int64_t j = base + threadIdx.x;
      const uint32_t keep =
          j < n && (j < (int64_t)A.n_sub || node_kept(A.flags[nb + j])) ? 1u : 0u;
      uint32_t tk;
      const uint32_t ek = block_excl_scan(keep, part, &tk);
      if (j < n) {
        const uint32_t id = run_id + ek;
        uint32_t gl = kNoNode;
        if (keep) {
          if (NB + id >= NE) {
            atomicOr(A.err, kNetErrIndex);
          } else {
            gl = (uint32_t)(NB + id);  // (at most the raw nodes, which stay below kNoNode)
            const bool sub = j < (int64_t)A.n_sub;
            A.node_in[NB + id] = sub ? A.in_slot[j] : -1;
            if (sub) A.node_cell[NB + id] = kNoNode;
          }
        }
        A.gid[nb + j] = gl;
      }
      run_id += tk;
    }
    if (threadIdx.x == 0 && NB + run_id != NE) atomicOr(A.err, kNetErrIndex);
    __syncthreads();  // gid of the whole genome before the cell pass
    const uint32_t* kw = A.known + (int64_t)g * A.words;
    const uint32_t* rk = A.rank + (int64_t)g * A.words;
    for (int64_t w = threadIdx.x; w < A.words; w += blockDim.x) {
      uint32_t word = kw[w];
      uint32_t raw = A.n_sub + rk[w];
      while (word != 0u) {
        const uint32_t b = (uint32_t)__builtin_ctz(word);
        word &= word - 1u;
        if ((int64_t)raw >= n) {
          atomicOr(A.err, kNetErrIndex);
          break;
        }
        const uint32_t id = A.gid[nb + raw];
        if (id != kNoNode && (int64_t)id >= NB && (int64_t)id < NE)
          A.node_cell[id] = 32u * (uint32_t)w + b + 1u;
        ++raw;
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------ incoming edges
// An edge u -> v is kept when an input reaches u and v reaches an output (then both ends are kept
// nodes). Sort keys of the raw edges: a kept edge's destination's kept number (sentinel: dropped);
// the values carry its source and weight, so that nothing is gathered after the sort (a gather of
// 15M edges by their raw index took 250 us).
__global__ void __launch_bounds__(kNetThreads) k_net_keys(NetKeyArgs A) {
  for (int64_t e = grid_thread(); e < A.edges; e += grid_threads()) {
    const uint32_t u = A.eu[e], v = A.ev[e];
    const uint32_t w = __float_as_uint(A.ew[e]);
    uint32_t key = A.sentinel, gu = 0u;
    if ((int64_t)u < A.nodes && (int64_t)v < A.nodes && (A.flags[u] & kFwd) != 0u &&
        (A.flags[v] & kBwd) != 0u) {
      gu = A.gid[u];
      const uint32_t gv = A.gid[v];
      if (gu >= A.sentinel || gv >= A.sentinel) atomicOr(A.err, kNetErrIndex);
      else key = gv;
    }
    A.key[e] = key;
    A.val[e] = (uint64_t)w << 32 | gu;
  }
}

// The first i with key[i] >= k (n: none).
__device__ __forceinline__ int64_t first_key(const uint32_t* key, int64_t n, uint32_t k) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (key[mid] < k) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// in_offset of every kept node (and one past the last), and the genomes' first edges, by searches of
// the sorted keys. (Counting the in-degrees instead took an atomic per edge: 190 us for 15M.)
__global__ void __launch_bounds__(kNetThreads) k_net_offsets(NetSplitArgs A) {
  const int64_t nodes = A.node_offset[A.n_genomes], G1 = (int64_t)A.n_genomes + 1;
  if (nodes > A.raw_nodes) {  // (never: k_net_number sums k_net_kept's counts)
    if (grid_thread() == 0) atomicOr(A.err, kNetErrIndex);
    return;
  }
  for (int64_t t = grid_thread(); t <= nodes + G1; t += grid_threads()) {
    const int64_t k = t <= nodes ? t : A.node_offset[t - nodes - 1];
    const int64_t e = first_key(A.key, A.raw_edges, k < nodes ? (uint32_t)k : A.sentinel);
    if (t <= nodes) {
      A.in_offset[t] = e;
    } else {
      A.summary[t - nodes - 1] = k;
      A.summary[G1 + t - nodes - 1] = e;
    }
  }
}

// The sorted kept edges' sources and weights.
__global__ void __launch_bounds__(kNetThreads) k_net_split(NetSplitArgs A) {
  const int64_t nodes = A.node_offset[A.n_genomes];
  for (int64_t i = grid_thread(); i < A.raw_edges; i += grid_threads()) {
    if (A.key[i] >= A.sentinel) return;  // (the dropped edges are the last)
    const uint64_t v = A.val[i];
    if ((int64_t)(uint32_t)v >= nodes) {
      atomicOr(A.err, kNetErrIndex);
      continue;
    }
    A.in_src[i] = (uint32_t)v;
    A.in_w[i] = __uint_as_float((uint32_t)(v >> 32));
  }
}

// ------------------------------------------------------------------------ activation
__global__ void __launch_bounds__(kNetThreads) k_net_stage(NetStageArgs A) {
  if (threadIdx.x < A.n) A.dst[threadIdx.x] = A.v[threadIdx.x];
}

// Four patterns (block pb) of input slot `slot`, of values at(i).
template <typename P>
__device__ __forceinline__ float4 pattern4(P&& at, uint32_t n_patterns, uint32_t n_inputs, int32_t slot,
                                           uint32_t pb) {
  float c[4] = {0.f, 0.f, 0.f, 0.f};
  if (slot >= 0 && (uint32_t)slot < n_inputs) {
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      const uint32_t p = 4u * pb + k;
      c[k] = p < n_patterns ? at((int64_t)p * n_inputs + (uint32_t)slot) : 0.0f;
    }
  }
  return make_float4(c[0], c[1], c[2], c[3]);
}

__device__ __forceinline__ void add4(float4& a, const float4& b) {
  a.x += b.x;
  a.y += b.y;
  a.z += b.z;
  a.w += b.w;
}
// a and b exchanged between lane halves (rows of 16 in swap16) so that the sum of the two results
// is, in the lower half (even rows), a plus its partner 32 (16) lanes away, and in the upper half
// (odd rows) the same of b: one butterfly stage of two values in two instructions.
__device__ __forceinline__ float swap_add32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_add16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// v plus v of the lane that the DPP control names.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(
                 0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, true));
}
constexpr int kDppRor8 = 0x128, kDppRor4 = 0x124, kDppXor2 = 0x4E, kDppXor1 = 0xB1;

// A node's incoming sum over one wave, for the 4 Q patterns whose states are x[source * Q + q]
// (q = lane % Q). The sum is always the same 64 partial sums, partial k an fmaf chain over edges
// k, k + 64, ... in list order, added in a fixed butterfly, so its bits depend neither on Q nor on
// the run: lane group t = lane / Q holds partials t, t + S, t + 2 S, ... (S = 64 / Q), the high
// bits of k are folded inside the lane and the low ones across lanes. The stages over 32 and 16
// lanes leave one of the four patterns per row of 16 lanes, so the rest and the sigmoid run once
// for all four: the lane returns the sum of pattern 4 q + lane / 16.
//
// The vector unit is what bounds these kernels, so the loop over whole batches of 64 edges holds
// only the multiply-adds and one address each: no bounds (x(s) reads the state of node s for the
// lane's q: from LDS, where an index outside would read zero, or checked, from memory) and no
// selects. AHEAD loads the next batch's sources and weights into a second register set: the
// stepwise kernel, whose batches wait for two trips to memory, needs it (55 -> 38 us a step); 32
// waves per CU hide the fused kernel's loads, and there the second set spilled (396 against 366
// us). The last, partial batch masks its lanes.
template <int Q, bool AHEAD, typename X>
__device__ __forceinline__ float node_sum(X&& x, const uint32_t* __restrict__ src,
                                          const float* __restrict__ wt, uint32_t deg,
                                          uint32_t lane) {
  constexpr uint32_t S = kWave / Q;
  const uint32_t t = lane / Q;
  float4 acc[Q];
#pragma unroll
  for (int j = 0; j < Q; ++j) acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](const uint32_t (&s)[Q], const float (&w)[Q]) {
    float4 v[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) v[j] = x(s[j]);
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      acc[j].x = fmaf(w[j], v[j].x, acc[j].x);
      acc[j].y = fmaf(w[j], v[j].y, acc[j].y);
      acc[j].z = fmaf(w[j], v[j].z, acc[j].z);
      acc[j].w = fmaf(w[j], v[j].w, acc[j].w);
    }
  };
  // (src and wt step along the list, so a lane's offsets from them stay constant)
  auto load = [&](uint32_t (&s)[Q], float (&w)[Q]) {
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      s[j] = src[S * (uint32_t)j + t];
      w[j] = wt[S * (uint32_t)j + t];
    }
    src += kWave;
    wt += kWave;
  };
  uint32_t s0[Q], s1[Q];
  float w0[Q], w1[Q];
  uint32_t whole = deg / kWave;
  if constexpr (AHEAD) {
    if (whole != 0u) load(s0, w0);
    while (whole >= 2u) {
      load(s1, w1);
      add(s0, w0);
      if (whole >= 3u) load(s0, w0);
      add(s1, w1);
      whole -= 2u;
    }
    if (whole != 0u) add(s0, w0);
  } else {
    for (; whole != 0u; --whole) {
      load(s0, w0);
      add(s0, w0);
    }
  }
  const uint32_t left = deg % kWave;
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    if (S * (uint32_t)j >= left) break;  // (the wave's)
    const uint32_t k = S * (uint32_t)j + t;
    if (k < left) {
      const float4 v = x(src[k]);
      const float w = wt[k];
      acc[j].x = fmaf(w, v.x, acc[j].x);
      acc[j].y = fmaf(w, v.y, acc[j].y);
      acc[j].z = fmaf(w, v.z, acc[j].z);
      acc[j].w = fmaf(w, v.w, acc[j].w);
    }
  }
#pragma unroll
  for (int h = Q / 2; h >= 1; h >>= 1)
#pragma unroll
    for (int j = 0; j < h; ++j) add4(acc[j], acc[j + h]);
  float z = swap_add16(swap_add32(acc[0].x, acc[0].z), swap_add32(acc[0].y, acc[0].w));
  static_assert(Q <= 4, "the stages over 8 and 4 lanes are always needed");
  z = dpp_add<kDppRor8>(z);  // (a rotation by 8 of 16 lanes; by 4 of values of period 8)
  z = dpp_add<kDppRor4>(z);
  if constexpr (Q <= 2) z = dpp_add<kDppXor2>(z);
  if constexpr (Q <= 1) z = dpp_add<kDppXor1>(z);
  return z;
}

// All steps of one genome for one block of 4 Q patterns. One launch per step over global states
// gathers 16 bytes per edge and four patterns from L2 (150 networks, 0.51M edges, 1000 patterns, 4
// steps: 2560 us); here the gathers are LDS reads, the edges are read once per 4 Q patterns and
// the steps need no launches between them (366 us; bound by the vector instructions: a node's sum
// and sigmoid beside its few edges). The states of its nodes live in two LDS
// buffers (swapped by each step), one wave per node and step, the edges read from L2. An input
// node holds its pattern values in both buffers. The node's first edge (bit 31: an input node) is
// kept in LDS after the states.
template <int Q>
__device__ __forceinline__ void net_run(const NetRunArgs& A, uint32_t g, uint32_t block,
                                        float4* lds) {
  const int64_t n0 = A.node_offset[g];
  const uint32_t n = (uint32_t)(A.node_offset[g + 1] - n0);
  if (n0 < 0 || n0 + (int64_t)n > A.nodes || net_run_lds(n, Q) > A.lds_bytes) return;  // (never)
  const int64_t e0 = A.in_offset[n0], e1 = A.in_offset[n0 + n];
  if (e0 < 0 || e1 < e0 || e1 > A.edges || e1 - e0 > 0x7FFFFFFF) return;  // (host-checked)
  const uint32_t edges = (uint32_t)(e1 - e0);
  const uint32_t lane = threadIdx.x % kWave;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  float4* cur = lds;
  float4* nxt = lds + n * Q;
  uint32_t* first = reinterpret_cast<uint32_t*>(lds + 2u * n * Q);
  for (uint32_t i = threadIdx.x; i < n * Q; i += kNetRunThreads) {
    const float4 v =
        pattern4([p = A.patterns](int64_t j) { return p[j]; }, A.n_patterns, A.n_inputs,
                 A.node_in[n0 + i / Q], block * Q + i % Q);
    cur[i] = v;
    nxt[i] = v;
  }
  for (uint32_t i = threadIdx.x; i <= n; i += kNetRunThreads) {
    const int64_t e = A.in_offset[n0 + i] - e0;
    const uint32_t f = e < 0 ? 0u : (e > (int64_t)edges ? edges : (uint32_t)e);
    first[i] = f | (i < n && A.node_in[n0 + i] >= 0 ? 0x80000000u : 0u);
  }
  __syncthreads();
  for (uint32_t step = 0; step < A.steps; ++step) {
    const float4* mine = cur + lane % Q;  // the lane's patterns
    for (uint32_t i = wave; i < n; i += kNetRunThreads / kWave) {
      const uint32_t f = __builtin_amdgcn_readfirstlane(first[i]);
      if (f >> 31) continue;
      const uint32_t l = __builtin_amdgcn_readfirstlane(first[i + 1]) & 0x7FFFFFFFu;
      const float z = node_sum<Q, false>([&](uint32_t s) { return mine[(s - (uint32_t)n0) * Q]; },
                                  A.in_src + e0 + f, A.in_w + e0 + f, l > f ? l - f : 0u, lane);
      if (lane % 16u < (uint32_t)Q)
        reinterpret_cast<float*>(nxt + i * Q + lane % 16u)[lane / 16u] = sigmoid_f(z);
    }
    __syncthreads();
    float4* s = cur;
    cur = nxt;
    nxt = s;
  }
  const float* c = reinterpret_cast<const float*>(cur);
  if (A.outputs) {
    const uint32_t np = min(A.n_patterns - block * 4u * Q, 4u * Q);
    for (uint32_t i = threadIdx.x; i < np * A.n_outputs; i += kNetRunThreads) {
      const uint32_t p = i / A.n_outputs, o = i % A.n_outputs;
      const uint32_t node = (uint32_t)A.out_node[o];
      if (node >= n) continue;  // (host-checked)
      A.outputs[((int64_t)g * A.n_patterns + block * 4u * Q + p) * A.n_outputs + o] =
          c[node * 4u * Q + p];
    }
  }
  if (A.fitness && threadIdx.x == 0 && (uint32_t)A.out_node[0] < n) {
    float se = 0.0f;
    for (uint32_t k = 0; k < A.n_patterns && k < 4u; ++k) {
      const float d = c[(uint32_t)A.out_node[0] * 4u * Q + k] - A.targets[k];
      se = fmaf(d, d, se);
    }
    A.fitness[g] = 1.0f - se / (float)A.n_patterns;
  }
}

__global__ void __launch_bounds__(kNetRunThreads, 8) k_net_run(NetRunArgs A) {
  extern __shared__ float4 net_lds[];
  uint32_t at = blockIdx.x;
#pragma unroll
  for (int r = 0; r < kNetRanges; ++r) {
    const uint32_t blocks = A.blocks[r], all = A.count[r] * blocks;
    if (at < all) {
      const uint32_t g = A.order[A.first[r] + at / blocks], block = at % blocks;
      if (g >= A.n_genomes) return;
      switch (A.q[r]) {
        case 1: net_run<1>(A, g, block, net_lds); break;
        case 2: net_run<2>(A, g, block, net_lds); break;
        default: net_run<4>(A, g, block, net_lds); break;
      }
      return;
    }
    at -= all;
  }
}

// The k-th genome of a list (k < total).
__device__ __forceinline__ uint32_t list_genome(const NetList& L, uint32_t k) {
  if (L.order == nullptr) return k;
#pragma unroll
  for (int r = 0; r < kNetRanges; ++r) {
    if (k < L.count[r]) return L.order[L.first[r] + k];
    k -= L.count[r];
  }
  return L.n_genomes;
}

// The stepwise kernels: blockIdx.y is the list's genome (0: all nodes as they lie, when the list is
// every genome: a step then waits for no list, order and offset; 4.8 -> 4.2 us), blockIdx.z the block
// of four patterns.
// Initial state: input nodes hold their pattern values, every other node 0.
__global__ void __launch_bounds__(kNetThreads) k_net_state(NetStateArgs A) {
  const bool all = A.list.order == nullptr;
  const uint32_t g = all ? 0u : list_genome(A.list, blockIdx.y);
  if (g >= A.list.n_genomes) return;
  float4* st = reinterpret_cast<float4*>(A.state);
  const int64_t n0 = all ? 0 : A.node_offset[g], n1 = all ? A.nodes : A.node_offset[g + 1];
  for (int64_t i = n0 + grid_thread(); i < n1; i += grid_threads())
    for (uint32_t pb = blockIdx.z; pb < A.pblocks; pb += gridDim.z)
      st[(int64_t)pb * A.nodes + i] = pattern4(
          [&](int64_t j) { return A.patterns ? A.patterns[j] : A.v[j]; }, A.n_patterns, A.n_inputs,
          A.node_in[i], pb);
}

// One synchronous step: one wave per (node, pattern block).
__global__ void __launch_bounds__(kNetThreads) k_net_step(NetStepArgs A) {
  const bool all = A.list.order == nullptr;
  const uint32_t g = all ? 0u : list_genome(A.list, blockIdx.y);
  if (g >= A.list.n_genomes) return;
  const uint32_t lane = threadIdx.x % kWave;
  const int64_t n0 = all ? 0 : A.node_offset[g];
  const int64_t n = (all ? A.nodes : A.node_offset[g + 1]) - n0;
  const int64_t waves = (int64_t)gridDim.x * (kNetThreads / kWave);
  for (int64_t k = (int64_t)blockIdx.x * (kNetThreads / kWave) +
                   __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
       k < n; k += waves) {
    const int64_t i = n0 + k;
    for (uint32_t pb = blockIdx.z; pb < A.pblocks; pb += gridDim.z) {
      const float4* cur = reinterpret_cast<const float4*>(A.cur) + (int64_t)pb * A.nodes;
      float4* nxt = reinterpret_cast<float4*>(A.nxt) + (int64_t)pb * A.nodes;
      if (A.node_in[i] >= 0) {
        if (lane == 0) nxt[i] = cur[i];
        continue;
      }
      const int64_t e0 = A.in_offset[i];
      const float z = node_sum<1, true>(
          [&](uint32_t s) {
            return (int64_t)s < A.nodes ? cur[s] : make_float4(0.f, 0.f, 0.f, 0.f);
          },
          A.in_src + e0, A.in_w + e0, (uint32_t)(A.in_offset[i + 1] - e0), lane);
      if (lane % 16u == 0u) reinterpret_cast<float*>(nxt + i)[lane / 16u] = sigmoid_f(z);
    }
  }
}

// Outputs of the list's (genome, pattern, output), or their XOR fitness (one output, four
// patterns: 1 - the mean squared error against the targets).
__global__ void __launch_bounds__(kNetThreads) k_net_out(NetOutArgs A) {
  const uint32_t g = list_genome(A.list, blockIdx.y);
  if (g >= A.list.n_genomes) return;
  const float4* st = reinterpret_cast<const float4*>(A.state);
  if (A.outputs) {
    const int64_t per_g = (int64_t)A.n_patterns * A.n_outputs;
    for (int64_t r = grid_thread(); r < per_g; r += grid_threads()) {
      const uint32_t p = (uint32_t)(r / A.n_outputs), o = (uint32_t)(r % A.n_outputs);
      const int64_t node = A.node_offset[g] + A.out_node[o];
      if (node >= A.node_offset[g + 1] || node >= A.nodes) continue;  // (host-checked)
      A.outputs[(int64_t)g * per_g + r] = comp(st[(int64_t)(p / 4u) * A.nodes + node], p % 4u);
    }
  }
  if (A.fitness && grid_thread() == 0) {
    const int64_t node = A.node_offset[g] + A.out_node[0];
    if (node >= A.node_offset[g + 1] || node >= A.nodes) return;
    const float4 v = st[node];
    float se = 0.0f;
    for (uint32_t q = 0; q < A.n_patterns && q < 4u; ++q) {
      const float d = comp(v, q) - A.target[q];
      se = fmaf(d, d, se);
    }
    A.fitness[g] = 1.0f - se / (float)A.n_patterns;
  }
}

// The copies of a build's buffers to buffers of their contents' size, a row of workgroups each
// (a copy call per buffer held the host for 8 to 15 us each).
__global__ void __launch_bounds__(kNetThreads) k_net_fit(NetFitArgs A) {
  const uint4* src = static_cast<const uint4*>(A.src[blockIdx.y]);
  uint4* dst = static_cast<uint4*>(A.dst[blockIdx.y]);
  const int64_t n = A.units[blockIdx.y];
  for (int64_t i = grid_thread(); i < n; i += grid_threads()) dst[i] = src[i];
}

// After every other kernel of the build: the error word to the host's summary.
__global__ void k_net_end(NetSplitArgs A) { A.summary[2 * ((int64_t)A.n_genomes + 1)] = *A.err; }

}  // namespace emr

namespace {
uint32_t genome_blocks(uint32_t n) { return n == 0 ? 1u : (n > 65535u ? 65535u : n); }
// Workgroups for a grid-stride loop over n items (at least one, at most 16384).
uint32_t stride_blocks(int64_t n) {
  int64_t b = (n + emr::kNetThreads - 1) / emr::kNetThreads;
  return (uint32_t)(b < 1 ? 1 : (b > 16384 ? 16384 : b));
}
// (x: the caller's, y: the list's genomes, z: pattern blocks, at most 65535 with a stride loop)
dim3 list_grid(const emr::NetList& L, uint32_t x, uint32_t pblocks) {
  return dim3(x < 1 ? 1 : x, L.total, pblocks < 65535u ? pblocks : 65535u);
}
// Workgroups of `per` nodes each over the nodes of a list's genomes (a row each), or over all nodes; the
// kernels stride over what 2^22 of them leave.
dim3 node_grid(const emr::NetList& L, int64_t nodes, uint32_t per, uint32_t pblocks) {
  const int64_t n = L.order ? (int64_t)L.max_nodes : nodes, x = (n + per - 1) / per;
  return dim3((uint32_t)(x < 1 ? 1 : (x > (1 << 22) ? 1 << 22 : x)), L.order ? L.total : 1u,
              pblocks < 65535u ? pblocks : 65535u);
}
}  // namespace

// Steps: 0 rank, 1 layout, 2 pairs of a phase, 3 its edges, 4 flags, 5 reach pass, 6 kept counts
// and their sums, 7 nodes, 8 keys; after the sort, 14 offsets and edges. Activation: 9 initial
// state, 10 one step, 11 outputs / fitness (stepwise), 12 patterns by value, 13 all steps in LDS. 15
// copies into buffers of the contents' size.
extern "C" hipError_t emr_launch_net(int step, const void* args, hipStream_t s) {
  using namespace emr;
  const dim3 blk(kNetThreads);
  switch (step) {
    case 0: {
      const auto& A = *static_cast<const NetRankArgs*>(args);
      hipLaunchKernelGGL(k_net_rank, dim3(genome_blocks(A.n_genomes)), blk, 0, s, A);
      break;
    }
    case 1: {
      const auto& A = *static_cast<const NetLayoutArgs*>(args);
      hipLaunchKernelGGL(k_net_layout, dim3(1), blk, 0, s, A);
      break;
    }
    case 2: {
      const auto& A = *static_cast<const NetEdgeArgs*>(args);
      if (A.n_pairs <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_net_pairs, dim3(stride_blocks(A.n_pairs)), blk, 0, s, A);
      break;
    }
    case 3: {
      const auto& A = *static_cast<const NetEdgeArgs*>(args);
      if (A.total <= 0) return hipSuccess;
      // 16384 waves at most (two rounds of the chip's wave slots), whole steps of 64 connections
      const int64_t steps = (A.total + kWave - 1) / kWave;
      const int64_t span = (steps + 16383) / 16384 * kWave;
      const int64_t waves = (A.total + span - 1) / span;
      constexpr int64_t per = kNetThreads / kWave;
      hipLaunchKernelGGL(k_net_edges, dim3((uint32_t)((waves + per - 1) / per)), blk, 0, s, A, span);
      break;
    }
    case 4: {
      const auto& A = *static_cast<const NetFlagArgs*>(args);
      hipLaunchKernelGGL(k_net_flags, dim3(genome_blocks(A.n_genomes)), blk, 0, s, A);
      break;
    }
    case 5: {
      const auto& A = *static_cast<const NetReachArgs*>(args);
      if (A.pass >= (uint32_t)kNetPasses || ((uintptr_t)A.eu & 15) != 0 || ((uintptr_t)A.ev & 15) != 0)
        return hipErrorInvalidValue;
      hipLaunchKernelGGL(k_net_reach, dim3(stride_blocks((A.edges + 3) / 4)), blk, 0, s, A);
      break;
    }
    case 6: {
      const auto& A = *static_cast<const NetFlagArgs*>(args);
      hipLaunchKernelGGL(k_net_kept, dim3(genome_blocks(A.n_genomes)), blk, 0, s, A);
      hipLaunchKernelGGL(k_net_number, dim3(1), blk, 0, s, A);
      break;
    }
    case 7: {
      const auto& A = *static_cast<const NetNodeArgs*>(args);
      hipLaunchKernelGGL(k_net_nodes, dim3(genome_blocks(A.n_genomes)), blk, 0, s, A);
      break;
    }
    case 8: {
      const auto& A = *static_cast<const NetKeyArgs*>(args);
      if (A.edges <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_net_keys, dim3(stride_blocks(A.edges)), blk, 0, s, A);
      break;
    }
    case 14: {
      const auto& A = *static_cast<const NetSplitArgs*>(args);
      hipLaunchKernelGGL(k_net_offsets, dim3(stride_blocks(A.raw_nodes + A.n_genomes + 2)), blk, 0,
                         s, A);
      if (A.raw_edges > 0)
        hipLaunchKernelGGL(k_net_split, dim3(stride_blocks(A.raw_edges)), blk, 0, s, A);
      hipLaunchKernelGGL(k_net_end, dim3(1), dim3(1), 0, s, A);
      break;
    }
    case 9: {
      const auto& A = *static_cast<const NetStateArgs*>(args);
      hipLaunchKernelGGL(k_net_state, node_grid(A.list, A.nodes, kNetThreads, A.pblocks), blk, 0, s, A);
      break;
    }
    case 10: {
      const auto& A = *static_cast<const NetStepArgs*>(args);
      constexpr uint32_t waves = kNetThreads / kWave;
      hipLaunchKernelGGL(k_net_step, node_grid(A.list, A.nodes, waves, A.pblocks), blk, 0, s, A);
      break;
    }
    case 11: {
      const auto& A = *static_cast<const NetOutArgs*>(args);
      const uint32_t items = A.outputs ? A.n_patterns * A.n_outputs : 1u;
      const uint32_t b = (items + kNetThreads - 1) / kNetThreads;
      hipLaunchKernelGGL(k_net_out, list_grid(A.list, b < 256u ? b : 256u, 1u), blk, 0, s, A);
      break;
    }
    case 12: {
      const auto& A = *static_cast<const NetStageArgs*>(args);
      if (A.n > kNetStageFloats || kNetStageFloats > (uint32_t)kNetThreads)
        return hipErrorInvalidValue;
      hipLaunchKernelGGL(k_net_stage, dim3(1), blk, 0, s, A);
      break;
    }
    case 13: {
      const auto& A = *static_cast<const NetRunArgs*>(args);
      uint64_t b = 0;
      for (int r = 0; r < kNetRanges; ++r) {
        if (A.count[r] == 0) continue;
        if ((A.q[r] & (A.q[r] - 1)) != 0 || A.q[r] == 0 || A.q[r] > kNetRunMaxQ ||
            A.blocks[r] == 0)
          return hipErrorInvalidValue;
        b += (uint64_t)A.count[r] * A.blocks[r];
      }
      if (b == 0) return hipSuccess;
      if (b > 0x7FFFFFFFull || A.lds_bytes > kNetRunLds) return hipErrorInvalidValue;
      hipLaunchKernelGGL(k_net_run, dim3((uint32_t)b), dim3(kNetRunThreads), A.lds_bytes, s, A);
      break;
    }
    case 15: {
      const auto& A = *static_cast<const NetFitArgs*>(args);
      int64_t most = 0;
      for (uint32_t k = 0; k < A.count && k < (uint32_t)kNetFits; ++k)
        most = A.units[k] > most ? A.units[k] : most;
      if (most == 0) return hipSuccess;
      const uint32_t b = stride_blocks(most);
      hipLaunchKernelGGL(k_net_fit, dim3(b < 2048u ? b : 2048u, A.count), blk, 0, s, A);
      break;
    }
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
