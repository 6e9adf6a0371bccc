// gfx950 kernel of ES-HyperNEAT's band values of expressed connections (the band threshold that
// Theorem 1 names beside the variance threshold; ES-HyperNEAT's pruning step defines it): for
// connection (pair, cell C, weight w), the pair's CPPN at the four same-level neighbour centres
// of C, one cell side d away along x and y, and band = max(min(|w - left|, |w - right|),
// min(|w - down|, |w - up|)). The pair's program runs through the interpreter's record step (one
// source per walk), each lane holding P / 4 connections and their 4 neighbours each. kBandParts waves
// share a pair, each taking every kBandParts-th walk: a high-frequency CPPN's pair has thousands of
// connections (one wave per pair: 131 us for 300,000 connections of 4950 pairs, the heaviest
// pair's wave). Most pairs have one walk at most, so the waves past a pair's first look at several
// pairs at once and run those that have a walk for them (a wave per pair and part: 29,894 connections
// of 4000 pairs 17 us, 240,075 of 4950 45 us).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/emr.h"
#include "band.h"
#include "discover.h"
#include "emr_internal.h"

namespace emr {

// The walks of one pair over its connections [lo, hi): connection i = b + 64 k + lane holds
// instances 4k .. 4k + 3 (left, right, down, up).
constexpr uint32_t kBandParts = 8;
template <int W>
__device__ __forceinline__ void band_walks(const BandArgs& A, const BandPair& bp, int64_t lo,
                                           int64_t hi, uint32_t part, uint32_t lane) {
  constexpr int P = positions_per_lane(1, W);
  constexpr int C = P / 4;
  const int64_t n_pos = n_positions(A.depth);
  for (int64_t b = lo + (int64_t)part * kWave * C; b < hi; b += (int64_t)kBandParts * kWave * C) {
    float px[P], py[P], wc[C];
    bool live[C];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      const int64_t i = b + (int64_t)k * kWave + lane;
      live[k] = i < hi;
      uint32_t F = live[k] ? A.conn_cell[i] : 1u;
      wc[k] = live[k] ? A.conn_w[i] : 0.0f;
      if (F == 0u || (int64_t)F > n_pos) {  // not a cell of this grid
        if (live[k]) atomicOr(A.err, kErrTable);
        live[k] = false;
        F = 1u;
      }
      // Eq. 1: the centre of grid position F - 1 (level l, Morton index m), side d = 2^(1-l)
      const uint32_t p = F - 1u;
      const int l = level_of(p);
      const uint32_t m = p - (uint32_t)level_offset(l);
      const float sc = pow2_neg(l);
      const float x = __builtin_fmaf((float)(2u * compact_even(m) + 1u), sc, -1.0f);
      const float y = __builtin_fmaf((float)(2u * compact_even(m >> 1) + 1u), sc, -1.0f);
      const float d = 2.0f * sc;
      px[4 * k + 0] = x - d;
      py[4 * k + 0] = y;
      px[4 * k + 1] = x + d;
      py[4 * k + 1] = y;
      px[4 * k + 2] = x;
      py[4 * k + 2] = y - d;
      px[4 * k + 3] = x;
      py[4 * k + 3] = y + d;
    }
    Walker<1, P, W> R;
    R.def();
    R.walk((uint64_t)(A.blob + bp.var_off), (uint64_t)(A.bias + bp.bias_base), bp.n_rec, px, py);
#pragma unroll
    for (int k = 0; k < C; ++k) {
      if (!live[k]) continue;
      const float* a = R.acc + 4 * k;
      const float dl = __builtin_fabsf(wc[k] - a[0]), dr = __builtin_fabsf(wc[k] - a[1]);
      const float dd = __builtin_fabsf(wc[k] - a[2]), du = __builtin_fabsf(wc[k] - a[3]);
      A.band[b + (int64_t)k * kWave + lane] =
          __builtin_fmaxf(__builtin_fminf(dl, dr), __builtin_fminf(dd, du));
    }
  }
}

// Part `part` of the pair's walks.
__device__ __forceinline__ void band_pair(const BandArgs& A, uint32_t pair, uint32_t part,
                                          uint32_t lane) {
  const BandPair bp = A.pairs[pair];
  // The pair's records, rows and window must lie inside their tables (the walk reads one record
  // and one row past the last, and a row as four floats).
  const uint32_t rec_words = kRecWords * (bp.n_rec + 1), row_floats = 4u * (bp.n_rec + 2);
  const bool ok = bp.n_rec <= kMaxRecords && (bp.var_off & (kRecWords - 1)) == 0 &&
                  rec_words <= A.blob_words && bp.var_off <= A.blob_words - rec_words &&
                  row_floats <= A.bias_floats && bp.bias_base <= A.bias_floats - row_floats &&
                  (bp.window == 4u || bp.window == 8u || bp.window == 16u || bp.window == 32u);
  if (!ok) {
    if (lane == 0) atomicOr(A.err, kErrTable);
    return;
  }
  int64_t lo = A.conn_offset[pair], hi = A.conn_offset[pair + 1];
  lo = lo < 0 ? 0 : (lo > A.cap ? A.cap : lo);
  hi = hi > A.cap ? A.cap : (hi < lo ? lo : hi);
  switch (bp.window) {
    case 4u: band_walks<4>(A, bp, lo, hi, part, lane); break;
    case 8u: band_walks<8>(A, bp, lo, hi, part, lane); break;
    case 16u: band_walks<16>(A, bp, lo, hi, part, lane); break;
    default: band_walks<32>(A, bp, lo, hi, part, lane); break;
  }
}

// The first `heads` workgroups run every pair's first part, a pair per wave; then `tails` workgroups
// each for the parts after it: their wave w takes the pairs w, w + W, ... (W waves: neighbours, the
// sources of one genome, go to different waves), 64 at a time. Up to kBandShared pairs the waves get a
// pair each (the launch is small, and a wave with several heavy pairs would outlast it: 900 pairs 38
// against 40 us with 8), above kBandPairs (4000 pairs 49 us, 4 each 51, 4950 pairs 62 and 67).
constexpr uint32_t kBandPairs = 8, kBandShared = 1024;
constexpr uint32_t kBandWaves = 4;
__global__ void __launch_bounds__(kBandWaves * kWave) k_band(BandArgs A, uint32_t heads, uint32_t tails) {
  const uint32_t lane = lane_id();
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (blockIdx.x < heads) {
    for (uint64_t pair = (uint64_t)blockIdx.x * kBandWaves + wv; pair < A.n_pairs;
         pair += (uint64_t)heads * kBandWaves)
      band_pair(A, (uint32_t)pair, 0u, lane);
    return;
  }
  const uint32_t part = 1u + (blockIdx.x - heads) / tails;
  const uint64_t w = (uint64_t)((blockIdx.x - heads) % tails) * kBandWaves + wv;
  const uint64_t waves = (uint64_t)tails * kBandWaves;
  for (uint64_t base = w; base < A.n_pairs; base += kWave * waves) {
    const uint64_t pair = base + lane * waves;
    bool more = false;
    if (pair < A.n_pairs) {
      const uint32_t window = A.pairs[pair].window;  // (any other value: band_pair reports it)
      const int64_t per = kWave * (window == 4u ? positions_per_lane(1, 4) / 4
                                   : window == 8u ? positions_per_lane(1, 8) / 4
                                   : window == 16u ? positions_per_lane(1, 16) / 4
                                                   : positions_per_lane(1, 32) / 4);
      more = A.conn_offset[pair + 1] - A.conn_offset[pair] > (int64_t)part * per;
    }
    for (uint64_t m = __ballot(more); m != 0ull; m &= m - 1ull)
      band_pair(A, (uint32_t)(base + (uint32_t)__builtin_ctzll(m) * waves), part, lane);
  }
}

}  // namespace emr

extern "C" hipError_t emr_launch_band(const emr::BandArgs* A, hipStream_t s) {
  using namespace emr;
  auto blocks = [&](uint32_t pairs) {
    const uint32_t b = (A->n_pairs + pairs - 1) / pairs;
    return b == 0 ? 1u : (b > 8192u ? 8192u : b);
  };
  const uint32_t heads = blocks(kBandWaves);
  const uint32_t tails = blocks(kBandWaves * (A->n_pairs > kBandShared ? kBandPairs : 1u));
  hipLaunchKernelGGL(k_band, dim3(heads + (kBandParts - 1) * tails), dim3(kBandWaves * kWave), 0, s, *A,
                     heads, tails);
  return hipGetLastError();
}
