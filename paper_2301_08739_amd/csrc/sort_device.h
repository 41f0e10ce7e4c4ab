// Device pieces shared by the sorts (flatten.hip) and the voxeliser (voxelize.hip).
#pragma once
#include "common.h"

namespace ff {
namespace {

// ---- sums over the lanes of a wavefront ---------------------------------------------------------
// Lanes read each other through the data-parallel primitives of the vector unit: six dependent additions of eight clocks, where
// the same by __shfl_up is six round trips to the LDS, 700 clocks.  Sorts are chains of such steps: 30,000 pillars, four sorts,
// k_split 5.8 -> 4.9 and k_buckets 9.2 -> 7.7 us, 12,345 pillars k_direct 8.8 -> 7.6, with what these no longer wait for before
// their first load.
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t dpp_or_0(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  v += dpp_or_0<0x111, 0xf>(v);              // the lane 1, 2, 4, 8 to the left, within rows of 16
  v += dpp_or_0<0x112, 0xf>(v);
  v += dpp_or_0<0x114, 0xf>(v);
  v += dpp_or_0<0x118, 0xf>(v);
  v += dpp_or_0<0x142, 0xa>(v);              // the last lane of rows 0 and 2 to all of rows 1 and 3,
  v += dpp_or_0<0x143, 0xc>(v);              // and of the lower half to all of the upper
  return v;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(v), 63);
}

// ---- block-wide exclusive scan of one uint32 per thread ---------------------------------------

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

// The same, with the sum of w over the block, in the barriers of one scan.  totals: [THREADS / 64][2]
template <int THREADS>
__device__ __forceinline__ uint32_t block_exclusive_scan_and_sum(uint32_t v, uint32_t w, uint32_t* totals, uint32_t* sum_v,
                                                                 uint32_t* sum_w) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_inclusive_scan(v), all_w = wave_inclusive_scan(w);
  if (lane == 63) {
    totals[2 * wave] = inc;
    totals[2 * wave + 1] = all_w;
  }
  __syncthreads();
  uint32_t base = 0, tv = 0, tw = 0;
#pragma unroll
  for (int i = 0; i < THREADS / 64; ++i) {
    const uint32_t t = totals[2 * i];
    if (i < wave) base += t;
    tv += t;
    tw += totals[2 * i + 1];
  }
  *sum_v = tv;
  *sum_w = tw;
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
