// gfx950 kernels that work on the CSR output of a discover call.
//
//   hidden nodes (Section 2, Phase 1 feeding Phase 2): per genome, the children of the kept cells of
//     its outgoing pairs as a bitmap over grid positions (a parent's four children are one aligned
//     nibble), counted, offset by k_scan and emitted in ascending heap order as outgoing sources at
//     their cell centres (Eq. 1);
//   connections (Section 4's types, Section 3.3's weight filter): each child of a kept parent as a
//     connection, kept by its type and weight magnitude;
//   Eq. 2 read literally: a record stays when every ancestor of its cell is a record of the pair;
//   the band filter: the connections whose band value (band.hip) exceeds a threshold.
// Each output is CSR. A pair's entries number from none to hundreds of thousands (a high-frequency
// CPPN keeps every cell), so no kernel gives a pair to a wave: entries go to the waves in spans.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/emr.h"
#include "band.h"
#include "discover.h"
#include "emr_internal.h"

namespace emr {

// Centre of grid position p (heap cell p + 1), Eq. 1: level l, Morton index within the level.
__device__ __forceinline__ void cell_centre(uint32_t p, float* x, float* y) {
  const int l = level_of(p);
  const uint32_t m = p - (uint32_t)level_offset(l);
  const float sc = pow2_neg(l);
  *x = __builtin_fmaf((float)(2u * compact_even(m) + 1u), sc, -1.0f);
  *y = __builtin_fmaf((float)(2u * compact_even(m >> 1) + 1u), sc, -1.0f);
}

// ------------------------------------------------------------------------ spans of entries
// The last q in [lo, hi) with off[q] <= r, given off[lo] <= r and (hi = n or off[hi] > r).
__device__ __forceinline__ uint32_t last_at_most(const int64_t* off, uint32_t lo, uint32_t hi,
                                                 int64_t r) {
  while (hi - lo > 1u) {
    const uint32_t mid = lo + (hi - lo) / 2u;
    if (off[mid] <= r)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}
// The same for an r of the whole wave, 64 places at a time: two or three trips to memory where the
// halving above takes 13 (5000 pairs), each of them most of a microsecond.
__device__ __forceinline__ uint32_t wave_last(const int64_t* off, uint32_t lo, uint32_t hi, int64_t r,
                                              uint32_t lane) {
  while (hi - lo > 1u) {
    const uint32_t step = (hi - lo - 1u) / kWave + 1u;
    const uint64_t q = (uint64_t)lo + (uint64_t)lane * step;
    const uint32_t le = popc64(ballot(q < hi && (lane == 0u || off[q] <= r)));
    lo += (le - 1u) * step;
    hi = hi - lo > step ? lo + step : hi;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}
// The last q >= lo with off[q] <= r (the wave's), given off[lo] <= r: mostly close to lo.
__device__ __forceinline__ uint32_t wave_last_from(const int64_t* off, uint32_t lo, uint32_t n,
                                                   int64_t r, uint32_t lane) {
  const uint64_t q = (uint64_t)lo + lane;
  const uint32_t le = popc64(ballot(q < n && (lane == 0u || off[q] <= r)));
  return le < (uint32_t)kWave ? __builtin_amdgcn_readfirstlane(lo + le - 1u)
                              : wave_last(off, lo + kWave - 1u, n, r, lane);
}
// Each lane's last q with off[q] <= r (off[p] <= r <= the last lane's r), v being off[p + lane]: 64
// places between p and the last lane's q are searched between the lanes; only where there are more
// (a step of 64 entries over many empty pairs) does a lane then halve the rest in memory.
__device__ __forceinline__ uint32_t lane_last(const int64_t* off, uint32_t p, uint32_t n, int64_t v,
                                              int64_t r, int64_t r_last, uint32_t lane) {
  uint32_t step = 1u, hi = n;
  if (ballot(v > r_last) == 0ull) {
    hi = wave_last(off, p + kWave - 1u, n, r_last, lane) + 1u;
    step = (hi - p - 1u) / kWave + 1u;
    const uint64_t q = (uint64_t)p + (uint64_t)lane * step;
    v = q < hi ? off[q] : INT64_MAX;
  }
  uint32_t k = 0;  // the last place with v <= r
#pragma unroll
  for (uint32_t d = kWave / 2; d >= 1u; d >>= 1) {
    const int64_t u = __shfl(v, (int)(k + d), kWave);
    if (u <= r) k += d;
  }
  const uint32_t lo = p + k * step;
  return step == 1u ? lo : last_at_most(off, lo, hi - lo > step ? lo + step : hi, r);
}

// The entries of a CSR table that the buffers hold: from the first pair's offset (a caller may pass
// the pairs from some k on: the offsets' tail over the same entries) to the last one's.
struct Held {
  int64_t first, end;
};
__device__ __forceinline__ Held held_entries(const int64_t* off, uint32_t n, int64_t cap) {
  const int64_t first = min(max(off[0], (int64_t)0), cap);
  return {first, min(max(off[n], first), cap)};
}

// Entries per span when `held` entries go to n_spans spans: a multiple of 64.
__device__ __forceinline__ int64_t span_length(int64_t held, uint32_t n_spans) {
  const int64_t steps = (held + kWave - 1) / kWave;
  return (steps + n_spans - 1) / n_spans * kWave;
}

// 64 of the n offsets, spread over all of them: the first round of a span's search, read before its
// first entry is known.
__device__ __forceinline__ int64_t span_pivot(const int64_t* off, uint32_t n, uint32_t lane) {
  const uint64_t q = (uint64_t)lane * ((n - 1u) / kWave + 1u);
  return q < n ? off[q] : INT64_MAX;
}

// Calls f(i, pair, ctx) for the wave's entries [base, end) of a CSR table (off[n + 1], n > 0), 64 at
// a time, every lane of the wave taking part (i < end is the lane's own test): pair is the entry's
// and ctx = make(pair) what its entries need of it. The wave holds the offsets of 64 pairs, from
// its step's first on. Most steps lie inside one pair, which the wave then follows without a search
// or another load of its context; in the others each lane finds its pair among the 64. (What bounds
// a call of few entries is the trips to memory, one after the other: with a search by halves here,
// a gallop per lane and a fence in k_filter_end, the filters of 432 records took 56 / 40 / 65 us,
// expression / band / chain, now 51 / 36 / 57; of 63,000 records 64 / 49 / 75, now 57 / 42 / 67.)
template <typename M, typename F>
__device__ __forceinline__ void for_span(const int64_t* off, uint32_t n, int64_t pivot, int64_t base,
                                         int64_t end, uint32_t lane, M&& make, F&& f) {
  if (base >= end) return;
  const uint32_t step = (n - 1u) / kWave + 1u;
  uint32_t p = (popc64(ballot(lane == 0u || pivot <= base)) - 1u) * step;
  p = wave_last(off, p, n - p > step ? p + step : n, base, lane);
  auto window = [&] {
    const uint64_t q = (uint64_t)p + lane;
    return q < n ? off[q] : INT64_MAX;
  };
  int64_t v = window(), p1 = __shfl(v, 1, kWave);
  bool have = false;
  decltype(make(p)) ctx{};
  for (int64_t b = base; b < end; b += kWave) {
    if (b >= p1) {
      const uint32_t le = popc64(ballot(lane == 0u || v <= b));
      p = le < (uint32_t)kWave ? __builtin_amdgcn_readfirstlane(p + le - 1u)
                               : wave_last(off, p + kWave - 1u, n, b, lane);
      v = window();
      p1 = __shfl(v, 1, kWave);
      have = false;
    }
    const int64_t i = b + lane, last = min(b + kWave, end) - 1;
    if (p1 > last) {
      if (!have) ctx = make(p);
      have = true;
      f(i, p, ctx);
    } else {
      const uint32_t q = lane_last(off, p, n, v, i < last ? i : last, last, lane);
      f(i, q, make(q));
    }
  }
}

// The wave's span index, and the launches' workgroups: 4 spans each.
__device__ __forceinline__ uint32_t span_index() {
  return __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
}

// Sum over the wave of a per-lane count c < 8 (bit-sliced ballots).
__device__ __forceinline__ uint32_t wave_sum3(uint32_t c) {
  uint32_t t = 0;
#pragma unroll
  for (int b = 0; b < 3; ++b) t += popc64(ballot((c >> b) & 1u)) << b;
  return t;
}
__device__ __forceinline__ uint32_t wave_excl3(uint32_t c) {
  uint32_t t = 0;
#pragma unroll
  for (int b = 0; b < 3; ++b) t += mbcnt64(ballot((c >> b) & 1u)) << b;
  return t;
}

// A filter over a CSR table: Op has off() (the table's offsets), pairs(), cap() (entries held),
// context(pair) (with the pair's first entry in `start`), keep(entry, context) -> a mask of the
// entry's kept items (up to 4) and emit(entry, item, place).
template <typename Op>
__global__ void __launch_bounds__(256) k_filter_count(Op op) {
  const uint32_t lane = lane_id(), span = span_index();
  const uint32_t n = op.pairs(), n_spans = gridDim.x * (blockDim.x / kWave);
  const int64_t pivot = span_pivot(op.off(), n, lane);
  const Held held = held_entries(op.off(), n, op.cap());
  const int64_t len = span_length(held.end - held.first, n_spans);
  const int64_t base = held.first + (int64_t)span * len, end = min(base + len, held.end);
  uint32_t total = 0;
  for_span(
      op.off(), n, pivot, base, end, lane, [&](uint32_t pair) { return op.context(pair); },
      [&](int64_t i, uint32_t, const auto& c) {
        const uint32_t m = i < end ? op.keep(i, c) : 0u;
        total += wave_sum3((uint32_t)__builtin_popcount(m));
      });
  if (lane == 0) op.spans.kept[span] = total;
  if (span == 0 && lane == 0) op.spans.kept[kFilterSpans] = 0u;  // k_filter_end's counter
}

// The kept entries of the spans before this one (n_spans at most kFilterSpans, read by the
// workgroup: 32 loads per thread at most; the spans from `used` on hold no entries).
constexpr uint32_t kFilterWaves = 4;  // of the counting and emitting workgroups
__device__ __forceinline__ uint64_t spans_before(const uint32_t* kept, uint32_t used,
                                                 uint64_t* wsum) {
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  const uint32_t first = blockIdx.x * kFilterWaves, read = min(first, used);
  const uint4 own = *reinterpret_cast<const uint4*>(kept + first);
  uint64_t sum = 0;
  for (uint32_t k = threadIdx.x; k < read; k += kFilterWaves * kWave) sum += kept[k];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, kWave);
  if (lane == 0) wsum[wv] = sum;
  __syncthreads();
  uint64_t t = 0;
#pragma unroll
  for (uint32_t k = 0; k < kFilterWaves; ++k) t += wsum[k];
  return t + (wv > 0u ? own.x : 0u) + (wv > 1u ? own.y : 0u) + (wv > 2u ? own.z : 0u);
}

// Writes the kept items in order, and the offset of every pair whose first entry the span holds.
template <typename Op>
__global__ void __launch_bounds__(256) k_filter_emit(Op op) {
  __shared__ uint64_t wsum[kFilterWaves];
  const uint32_t lane = lane_id(), span = span_index();
  const uint32_t n = op.pairs(), n_spans = gridDim.x * (blockDim.x / kWave);
  const int64_t pivot = span_pivot(op.off(), n, lane);
  const Held held = held_entries(op.off(), n, op.cap());
  const int64_t entries = held.end - held.first, len = span_length(entries, n_spans);
  const int64_t base = held.first + (int64_t)span * len, end = min(base + len, held.end);
  // The spans are those of the capacity: of a light call's, most workgroups have no entries and
  // leave before the sums (the last one writes the total).
  const uint32_t used = len > 0 ? (uint32_t)((entries + len - 1) / len) : 0u;
  if (blockIdx.x + 1 < gridDim.x && blockIdx.x * kFilterWaves >= used) return;
  // (few spans are summed whole: these reads then go out with the offsets', not after them)
  int64_t at0 = (int64_t)spans_before(op.spans.kept, n_spans <= 1024u ? n_spans : used, wsum);
  for_span(
      op.off(), n, pivot, base, end, lane, [&](uint32_t pair) { return op.context(pair); },
      [&](int64_t i, uint32_t pair, const auto& ctx) {
        const bool mine = i < end;
        const uint32_t m = mine ? op.keep(i, ctx) : 0u;
        const uint32_t c = (uint32_t)__builtin_popcount(m);
        int64_t at = at0 + wave_excl3(c);
        if (mine && i == ctx.start) op.spans.out_offset[pair] = at;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if ((m >> k) & 1u) op.emit(i, k, at++);
        at0 += wave_sum3(c);
      });
  if (span == n_spans - 1 && lane == 0)
    *reinterpret_cast<uint64_t*>(op.spans.kept + kFilterSpans + 2) = (uint64_t)at0;  // the total
}

// After k_filter_emit: the offsets of the empty pairs (their next pair's that has an entry) and of
// those whose entries lie beyond the ones held (the total), and every pair's count, 64 consecutive
// pairs per wave; the workgroup that ends last hands the call's flags over (see k_scan).
constexpr int kEndThreads = 1024;
template <typename Op>
__global__ void __launch_bounds__(kEndThreads) k_filter_end(Op op) {
  __shared__ uint32_t wmax[kEndThreads / kWave];
  const uint32_t n = op.pairs(), lane = lane_id();
  const FilterSpans& F = op.spans;
  const int64_t* off = op.off();
  const uint32_t err = __hip_atomic_load(F.flags + kFlagErr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t held = held_entries(off, n, op.cap()).end;
  const int64_t total = (int64_t)*reinterpret_cast<const uint64_t*>(F.kept + kFilterSpans + 2);
  uint32_t mx = 0;
  const uint32_t waves = gridDim.x * (kEndThreads / kWave);
  for (uint32_t w = span_index(); w <= (n - 1u) / kWave; w += waves) {
    const uint32_t p0 = w * kWave, p = p0 + lane;
    const uint32_t p1 = n - p0 > (uint32_t)kWave ? p0 + kWave : n;  // the wave's pairs end here
    const int64_t i0 = p < p1 ? off[p] : 0, i1 = p < p1 ? off[p + 1] : 0, i_end = off[p1];
    const bool has = i0 < i1 && i0 < held;
    const uint64_t m = ballot(has);
    int64_t o = has ? F.out_offset[p] : 0;
    // the offset of the first entry after the wave's pairs
    int64_t after = total;
    if (i_end < held) after = F.out_offset[wave_last_from(off, p1 - 1u, n, i_end, lane)];
    const uint64_t later = lane == kWave - 1 ? 0ull : m >> (lane + 1u);
    const int64_t ahead = __shfl(o, later ? (int)(lane + 1u + (uint32_t)__builtin_ctzll(later)) : 0, kWave);
    const int64_t next = later ? ahead : after;
    if (p < p1) {
      if (!has) F.out_offset[p] = next;
      const int64_t c = has && next > o ? next - o : 0;
      F.out_count[p] = c;
      mx = max(mx, (uint32_t)min(c, (int64_t)0xFFFFFFFFll));
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o, kWave));
  if (lane == 0) wmax[threadIdx.x / kWave] = mx;
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int k = 1; k < kEndThreads / kWave; ++k) mx = max(mx, wmax[k]);
  if (gridDim.x > 1u) {
    // the workgroup's largest is raised before the workgroup is counted: the value that the first
    // atomic returns has to be there before the second (a fence would write the L2 back)
    const uint32_t before = atomicMax(F.flags + kFlagMax, mx);
    asm volatile("" ::"v"(before) : "memory");
    if (atomicAdd(F.kept + kFilterSpans, 1u) != gridDim.x - 1u) return;
    mx = __hip_atomic_load(F.flags + kFlagMax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  F.out_offset[n] = total;
  F.host[kFlagErr] = err;
  F.host[kFlagMax] = mx;
  F.host[kFlagTotal] = (uint32_t)total;
  F.host[kFlagTotal + 1] = (uint32_t)((uint64_t)total >> 32);
#pragma unroll
  for (int k = 0; k < kFlagWords; ++k)
    __hip_atomic_store(F.flags + k, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What a record's entry needs of its pair.
struct RecordPair {
  int64_t start, end;  // its records
  uint32_t info;       // genome << 1 | direction
  float sx, sy;        // its source
};

// ------------------------------------------------------------------------ hidden nodes
// Each record's four cells. A record outside the range of the pair found (offsets out of order)
// marks nothing. (One lane per record with a search of its own took 261 us for 6M records.)
__global__ void __launch_bounds__(256) k_hidden_mark(HiddenArgs A) {
  const uint32_t lane = lane_id();
  const int64_t Q = n_parents(A.rec.depth);
  const uint32_t np = A.rec.n_pairs;
  if (np == 0u) return;
  const int64_t* off = A.rec.offset;
  const int64_t held = min(max(off[np], (int64_t)0), A.rec.cap);  // the call's records held
  if (off[0] > 0) return;                                          // not a CSR offset table
  const int64_t len = span_length(held, gridDim.x * (blockDim.x / kWave));
  const int64_t base = (int64_t)span_index() * len, end = min(base + len, held);
  for_span(
      off, np, span_pivot(off, np, lane), base, end, lane,
      [&](uint32_t p) {
        return RecordPair{off[p], off[p] + A.rec.count[p], A.rec.pair_info[2 * p], 0.0f, 0.0f};
      },
      [&](int64_t i, uint32_t, const RecordPair& c) {
        // grid positions 4P .. 4P+3 (incoming pairs add no hidden node)
        const uint32_t g = c.info >> 1;
        const bool mine = i < end && i >= c.start && i < c.end && (c.info & 1u) == 0u &&
                          g < A.n_genomes;
        const uint32_t P = mine ? A.rec.parent[i] : 0u;
        const bool ok = mine && (int64_t)P < Q;
        int64_t key = ok ? (int64_t)g * A.words + P / 8u : -1 - (int64_t)lane;
        uint32_t m = 0xFu << (4u * (P % 8u));
        // A pair's parents ascend, so the lanes of one bitmap word follow each other: the first of
        // them (and every eighth lane: small pairs' runs can be longer) takes the bits of up to
        // eight. Bits already marked by the genome's other pairs (most are)
        // cost a read only; the read and the atomic both go to the memory side, past the L2s.
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
          const int64_t k2 = __shfl_down(key, d, kWave);
          const uint32_t m2 = (uint32_t)__shfl_down((int)m, d, kWave);
          if (lane + (uint32_t)d < (uint32_t)kWave && k2 == key) m |= m2;
        }
        const int64_t before = __shfl_up(key, 1, kWave);
        if (!ok || (lane % 8u != 0u && before == key)) return;
        uint32_t* bits = A.fresh + key;
        if ((__hip_atomic_load(bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & m) != m)
          atomicOr(bits, m);
      });
}

// One workgroup of 16 waves per genome: its new cells (found now, not known before). A deep grid's
// bitmap is long (43,691 words at depth 10) and a call's genomes may be few.
constexpr int kHiddenThreads = 1024;
__global__ void __launch_bounds__(kHiddenThreads) k_hidden_count(HiddenArgs A) {
  __shared__ uint32_t part[kHiddenThreads / kWave];
  constexpr uint32_t waves = kHiddenThreads / kWave;
  for (uint32_t g = blockIdx.x; g < A.n_genomes; g += gridDim.x) {
    const uint32_t* f = A.fresh + (int64_t)g * A.words;
    const uint32_t* k = A.known ? A.known + (int64_t)g * A.words : nullptr;
    uint32_t c = 0;
#pragma unroll 4
    for (int64_t w = threadIdx.x; w < A.words; w += blockDim.x)
      c += __builtin_popcount(f[w] & (k ? ~k[w] : ~0u));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) c += (uint32_t)__shfl_xor((int)c, off, kWave);
    if (lane_id() == 0) part[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t t = 0;
      for (uint32_t i = 0; i < waves; ++i) t += part[i];
      A.totals[g] = t;
    }
    __syncthreads();
  }
}

// One workgroup per genome, four consecutive bitmap items per thread and round: the genome's new
// cells come out in ascending order at offsets[g] + (cells of the rounds and threads before) + rank
// in the thread's items; then the genome's known bits take the new cells. An item is a word of a
// long bitmap, which is sparse, and a nibble (the four children of one parent) of a short one,
// where a thread with four dense words would write 128 cells one after the other (26 us for 43
// words). (A thread per run of words / 256, scanned by one thread: 280 to 650 us for 100 genomes
// at depth 10.)
constexpr int64_t kShortWords = 1024;
template <int BITS>
__global__ void __launch_bounds__(kHiddenThreads) k_hidden_emit(HiddenArgs A) {
  constexpr int PER = 32 / BITS;  // items per word
  constexpr int ITEMS = BITS == 32 ? 4 : 1;
  __shared__ uint32_t part[kHiddenThreads / kWave];
  const int64_t n_pos = n_positions(A.rec.depth), items = A.words * PER;
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  for (uint32_t g = blockIdx.x; g < A.n_genomes; g += gridDim.x) {
    const uint32_t* f = A.fresh + (int64_t)g * A.words;
    uint32_t* k = A.known ? A.known + (int64_t)g * A.words : nullptr;
    int64_t at0 = A.offsets[g];
    for (int64_t round = 0; round < items; round += ITEMS * kHiddenThreads) {
      const int64_t i0 = round + ITEMS * (int64_t)threadIdx.x;
      uint32_t fresh[ITEMS], c = 0;
#pragma unroll
      for (int q = 0; q < ITEMS; ++q) {
        const int64_t w = (i0 + q) / PER;
        fresh[q] = w < A.words ? f[w] & (k ? ~k[w] : ~0u) : 0u;
        if constexpr (BITS < 32)
          fresh[q] = (fresh[q] >> (BITS * (uint32_t)((i0 + q) % PER))) & ((1u << BITS) - 1u);
        c += __builtin_popcount(fresh[q]);
      }
      uint32_t incl = c;
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, off, kWave);
        if (lane >= (uint32_t)off) incl += v;
      }
      if (lane == kWave - 1) part[wv] = incl;
      __syncthreads();
      uint32_t before = 0, total = 0;
#pragma unroll
      for (int i = 0; i < kHiddenThreads / kWave; ++i) {
        before += (uint32_t)i < wv ? part[i] : 0u;
        total += part[i];
      }
      int64_t at = at0 + before + incl - c;
#pragma unroll
      for (int q = 0; q < ITEMS; ++q)
        for (uint32_t b = fresh[q]; b != 0u; b &= b - 1u) {
          const int64_t p = (i0 + q) * BITS + __builtin_ctz(b);
          if (p < n_pos && at < A.cap) {
            float x, y;
            cell_centre((uint32_t)p, &x, &y);
            A.out_src[3 * at] = __float_as_uint(x);
            A.out_src[3 * at + 1] = __float_as_uint(y);
            A.out_src[3 * at + 2] = (uint32_t)EMR_DIR_OUT;
            if (A.out_cell) A.out_cell[at] = (uint32_t)(p + 1);
          }
          ++at;
        }
      at0 += total;
      __syncthreads();  // part is rewritten for the next round, and every known word was read
      if (k && c != 0u) {
        if constexpr (BITS == 32) {
#pragma unroll
          for (int q = 0; q < ITEMS; ++q)
            if (fresh[q] != 0u) k[i0 + q] |= fresh[q];
        } else {
          atomicOr(k + i0 / PER, fresh[0] << (BITS * (uint32_t)(i0 % PER)));
        }
      }
    }
  }
}

// ------------------------------------------------------------------------ connections
// Type of a connection from (ax, ay) to (bx, by) (Section 4).
__device__ __forceinline__ uint32_t conn_type(float ax, float ay, float bx, float by) {
  if (ax == bx && ay == by) return EMR_CONN_SELF;
  if (ay < by) return EMR_CONN_FORWARD;
  if (ay > by) return EMR_CONN_BACKWARD;
  return EMR_CONN_LATERAL;
}

// The children of a pair's record that are expressed connections.
struct ExpressOp : ExpressArgs {
  __device__ const int64_t* off() const { return rec.offset; }
  __host__ __device__ uint32_t pairs() const { return rec.n_pairs; }
  __device__ int64_t cap() const { return rec.cap; }
  __device__ RecordPair context(uint32_t pair) const {
    const uint32_t j = rec.pair_info[2 * pair + 1];
    const int64_t start = rec.offset[pair];
    return {start, start + rec.count[pair], rec.pair_info[2 * pair], rec.src_xy[2 * j],
            rec.src_xy[2 * j + 1]};
  }
  __device__ uint32_t keep(int64_t i, const RecordPair& c) const {
    const uint32_t P = rec.parent[i];  // (these reads go out with the pair's)
    const float4 w = reinterpret_cast<const float4*>(rec.w4)[i];
    if (i < c.start || i >= c.end || (int64_t)P >= n_parents(rec.depth)) return 0u;
    const bool incoming = (c.info & 1u) != 0u;
    const float sx = c.sx, sy = c.sy;
    const float wk[4] = {w.x, w.y, w.z, w.w};
    // Eq. 1: the four children are one aligned quad of their level
    float x0, y0;
    cell_centre(4u * P, &x0, &y0);
    const float side = 2.0f * pow2_neg(level_of(4u * P));  // (exact: so are the centres)
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float cx = (k & 1) ? x0 + side : x0, cy = (k & 2) ? y0 + side : y0;
      const uint32_t t = incoming ? conn_type(cx, cy, sx, sy) : conn_type(sx, sy, cx, cy);
      if ((t & type_mask) != 0u && __builtin_fabsf(wk[k]) > w_min) m |= 1u << k;
    }
    return m;
  }
  __device__ void emit(int64_t i, int k, int64_t at) const {
    if (at >= ExpressArgs::cap) return;
    out_cell[at] = 4u * rec.parent[i] + 1u + (uint32_t)k;
    out_w[at] = rec.w4[4 * i + k];
  }
};

// ------------------------------------------------------------------------ band filter
// The connections with band > theta_band (strict; a NaN band never passes), in order.
struct BandOp : BandSelectArgs {
  __device__ const int64_t* off() const { return in_offset; }
  __host__ __device__ uint32_t pairs() const { return n_pairs; }
  __device__ int64_t cap() const { return in_cap; }
  __device__ RecordPair context(uint32_t pair) const { return {in_offset[pair], 0, 0u, 0.0f, 0.0f}; }
  __device__ uint32_t keep(int64_t i, const RecordPair&) const {
    return band[i] > theta_band ? 1u : 0u;
  }
  __device__ void emit(int64_t i, int, int64_t at) const {
    if (at >= out_cap) return;
    out_cell[at] = in_cell[i];
    out_w[at] = in_w[i];
  }
};

// ------------------------------------------------------------------------ Eq. 2 chain rule
__global__ void __launch_bounds__(256) k_chain_mark(ChainArgs A) {
  const uint32_t lane = lane_id();
  const int64_t Q = n_parents(A.rec.depth);
  const uint32_t np = A.rec.n_pairs;
  const int64_t* off = A.rec.offset;
  const Held held = held_entries(off, np, A.rec.cap);
  const int64_t len = span_length(held.end - held.first, gridDim.x * (blockDim.x / kWave));
  const int64_t base = held.first + (int64_t)span_index() * len, end = min(base + len, held.end);
  for_span(
      off, np, span_pivot(off, np, lane), base, end, lane,
      [&](uint32_t p) { return RecordPair{off[p], off[p] + A.rec.count[p], 0u, 0.0f, 0.0f}; },
      [&](int64_t i, uint32_t p, const RecordPair& c) {
        const uint32_t P = i < end ? A.rec.parent[i] : 0u;
        if (i < c.end && i >= c.start && i < end && (int64_t)P < Q)
          atomicOr(A.member + (int64_t)p * A.qwords + P / 32u, 1u << (P % 32u));
      });
}

// A pair's record (its members: the pair's bitmap) stays when every ancestor of its cell is a record
// of the pair (the root is its own ancestor line's start).
struct ChainOp : ChainArgs {
  __device__ const int64_t* off() const { return rec.offset; }
  __host__ __device__ uint32_t pairs() const { return rec.n_pairs; }
  __device__ int64_t cap() const { return rec.cap; }
  __device__ RecordPair context(uint32_t pair) const {
    const int64_t start = rec.offset[pair];
    return {start, start + rec.count[pair], pair, 0.0f, 0.0f};  // (info: the pair itself)
  }
  __device__ uint32_t keep(int64_t i, const RecordPair& c) const {
    uint32_t P = rec.parent[i];
    if (i < c.start || i >= c.end || (int64_t)P >= n_parents(rec.depth)) return 0u;
    const uint32_t* bits = member + (int64_t)c.info * qwords;
    while (P > 0u) {  // four ancestors at a time, their reads in flight together (the root: its own)
      uint32_t all = 1u;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        P = P > 0u ? (P - 1u) / 4u : 0u;
        all &= bits[P / 32u] >> (P % 32u);
      }
      if ((all & 1u) == 0u) return 0u;
    }
    return 1u;
  }
  __device__ void emit(int64_t i, int, int64_t at) const {
    if (at >= ChainArgs::cap) return;
    out_parent[at] = rec.parent[i];
    reinterpret_cast<float4*>(out_w4)[at] = reinterpret_cast<const float4*>(rec.w4)[i];
  }
};

}  // namespace emr

// ------------------------------------------------------------------------ launchers
// Workgroups of 4 waves, one span each, for at most `cap` entries (the entries are counted on the
// device: spans beyond them do nothing).
static uint32_t span_blocks(int64_t cap) {
  const int64_t steps = (cap + emr::kWave - 1) / emr::kWave;
  return (uint32_t)((std::min<int64_t>(std::max<int64_t>(steps, 1), emr::kFilterSpans) + 3) / 4);
}

extern "C" hipError_t emr_launch_hidden(const emr::HiddenArgs* A, int step, hipStream_t s) {
  const uint32_t gb = A->n_genomes == 0 ? 1 : (A->n_genomes > 65535 ? 65535 : A->n_genomes);
  switch (step) {
    case 0:
      hipLaunchKernelGGL(emr::k_hidden_mark, dim3(span_blocks(A->rec.cap)), dim3(256), 0, s, *A);
      break;
    case 1:
      hipLaunchKernelGGL(emr::k_hidden_count, dim3(gb), dim3(emr::kHiddenThreads), 0, s, *A);
      break;
    case 2:
      if (A->words <= emr::kShortWords)
        hipLaunchKernelGGL(emr::k_hidden_emit<4>, dim3(gb), dim3(emr::kHiddenThreads), 0, s, *A);
      else
        hipLaunchKernelGGL(emr::k_hidden_emit<32>, dim3(gb), dim3(emr::kHiddenThreads), 0, s, *A);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

namespace {
template <typename Op>
hipError_t launch_filter(const Op& op, int64_t cap, hipStream_t s) {
  const uint32_t blocks = span_blocks(cap);
  hipLaunchKernelGGL(emr::k_filter_count<Op>, dim3(blocks), dim3(256), 0, s, op);
  hipLaunchKernelGGL(emr::k_filter_emit<Op>, dim3(blocks), dim3(256), 0, s, op);
  const uint32_t ends = (op.pairs() + emr::kEndThreads - 1) / emr::kEndThreads;
  hipLaunchKernelGGL(emr::k_filter_end<Op>, dim3(ends < 64u ? ends : 64u), dim3(emr::kEndThreads), 0,
                     s, op);
  return hipGetLastError();
}
}  // namespace

// The filters over at least one pair.
extern "C" hipError_t emr_launch_express(const emr::ExpressArgs* A, hipStream_t s) {
  return launch_filter(emr::ExpressOp{*A}, A->rec.cap, s);
}

extern "C" hipError_t emr_launch_band_select(const emr::BandSelectArgs* A, hipStream_t s) {
  return launch_filter(emr::BandOp{*A}, A->in_cap, s);
}

extern "C" hipError_t emr_launch_chain(const emr::ChainArgs* A, hipStream_t s) {
  hipLaunchKernelGGL(emr::k_chain_mark, dim3(span_blocks(A->rec.cap)), dim3(256), 0, s, *A);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_filter(emr::ChainOp{*A}, A->rec.cap, s);
}
