// Device pieces shared by the sorts (flatten.hip) and the voxeliser (voxelize.hip).
#pragma once
#include "common.h"

namespace ff {
namespace {

// ---- block-wide exclusive scan of one uint32 per thread ---------------------------------------
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t t = __shfl_up(v, d, 64);
    if (lane >= d) v += t;
  }
  return v;
}

template <int THREADS>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wave_totals /*[THREADS/64]*/,
                                                         uint32_t* block_total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = wave_inclusive_scan(v);
  if (lane == 63) wave_totals[w] = inc;
  __syncthreads();
  uint32_t base = 0, total = 0;
#pragma unroll
  for (int i = 0; i < THREADS / 64; ++i) {
    uint32_t t = wave_totals[i];
    if (i < w) base += t;
    total += t;
  }
  if (block_total) *block_total = total;
  __syncthreads();
  return base + inc - v;
}

// Lanes with the same number (its lowest `bits` bits)
__device__ __forceinline__ uint64_t same_number(uint32_t v, int bits) {
  uint64_t m = ~0ull;
  for (int b = 0; b < bits; ++b) {
    const uint64_t set = __ballot((v >> b) & 1u);
    m &= (v >> b) & 1u ? set : ~set;
  }
  return m;
}
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// Rank of this lane's number among the wavefront's so far, whose counts of each number are counts[].
__device__ __forceinline__ uint32_t rank_in_wave(uint16_t* counts, uint32_t v, int bits, bool valid) {
  const uint64_t same = same_number(v, bits) & __ballot(valid);
  const uint32_t before = counts[v], below = lanes_below(same);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (all lanes have read)
  if (valid && below == 0u) counts[v] = (uint16_t)(before + (uint32_t)__popcll(same));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  return before + below;
}
// counts[wave][2 word], [.. + 1], packed, to the sums of the wavefronts before; returns the totals.
template <int WAVES>
__device__ __forceinline__ uint32_t sum_over_waves(uint32_t* words, int words_of_wave, int word) {
  uint32_t run = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const uint32_t c = words[w * words_of_wave + word];
    words[w * words_of_wave + word] = run;
    run += c;                                // (no carry from the lower half: at most 24,576 points are counted)
  }
  return run;
}

// Cell of point i (see PointCells).  Comparisons with NaN fail, so such a point is dropped.
__device__ __forceinline__ void point_cell(const PointCells& pt, int64_t i, int32_t* c) {
  const float cx = floorf((pt.xy[2 * i] - pt.x_min) / pt.voxel_x), cy = floorf((pt.xy[2 * i + 1] - pt.y_min) / pt.voxel_y);
  const int b = pt.frame ? pt.frame[i] : 0;
  const bool keep = cx >= 0.f && cx < (float)pt.grid_x && cy >= 0.f && cy < (float)pt.grid_y && b >= 0 && b < pt.B;
  c[0] = keep ? b : pt.B;
  c[1] = keep ? (int)cx : 0;
  c[2] = keep ? (int)cy : 0;
  c[3] = 0;
}

}  // namespace
}  // namespace ff
