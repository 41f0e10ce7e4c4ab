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
