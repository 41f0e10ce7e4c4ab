// Row gather / scatter between pillar order and the flattened (sorted) order: the explicit form
// of the reshape [N, C] -> [N/G, G, C] of paper Sec. 4.2.1.  Pure data movement, HBM-bound:
// every thread moves 16-byte pieces, consecutive threads move consecutive pieces of a row.
#include "common.h"

namespace ff {
namespace {

typedef uint32_t piece_t __attribute__((ext_vector_type(4)));

// Pieces of 16 bytes that lie side by side in the order of the rows of one side: which row a piece is of.
struct RowPieces { int64_t total; int32_t per_row, log; };  // log: of per_row if that is a power of two, else -1
RowPieces row_pieces(int64_t n, int per_row) {
  int log = 0;
  while ((1 << log) < per_row) ++log;
  return {n * per_row, per_row, 1 << log == per_row ? log : -1};
}
__device__ __forceinline__ int64_t row_of(const RowPieces& rp, int64_t i) {
  return rp.log >= 0 ? i >> rp.log : i / rp.per_row;  // the same way for every thread
}

// What bounds it: memory, and with few rows the launch.  Rows of 2^k pieces (all feature counts of the layers) take shifts: a 64-bit
// division for every piece was most of the instructions.  Up to kRowsShort a thread takes one piece: the pieces of a workgroup then
// lie as in the launches on either side, whose lines its L2 has.  Beyond, two are in flight.  What is read once passes the 256 MB
// memory-side cache by; what is written does so only where the next launch would hardly find it there.  Measured from graphs, 128 or
// 256 bfloat16, buffers that no cache holds / that the launches before left there, us:
//   a launch that writes the rows, scatter, a launch that reads them: two pieces and non-temporal stores 3.7 MiB 12.1 / 11.5, 7 MiB 12.4
//   / 14.8, 15 MiB 20.6 / 18.7, 29 MiB 34.4 / 32.0, 59 MiB 64.3 / 57.8, 88 MiB 93.9 / 83.0, 117 MiB 121 / 111; two pieces, plain stores
//   11.2 / 10.9, 12.5 / 15.5, 20.1 / 17.7, 34.3 / 30.6, 63.7 / 55.9, 93.3 / 81.7, 123 / 113; one 11.0 / 9.9, 12.5 / 12.5, 20.4 / 17.5.
//   The same around gather, two pieces / one: 3.7 MiB 11.7, 11.4 / 11.5, 9.5, 7 MiB 13.1, 15.9 / 13.0, 12.8, 11 MiB 17.2, 18.6 / 17.5, 16.4.
//   Plain loads in scatter: 29 MiB 36.1 / 30.7 instead of 34.2 / 30.6.
//   Scatter of rows that were written long before, and a launch that reads the result, non-temporal stores / plain ones: 3.7 MiB 8.3, 7.9
//   / 6.7, 7.0, 15 MiB 15.6, 16.0 / 13.3, 15.4, 59 MiB 48.4, 44.0 / 43.8, 40.6.
// Without a reader the stores of 7 to 64 MiB look 4 to 12 % faster non-temporal (gather and scatter alone, 59 MiB 42.4 / 45.1): the
// reader pays for it.  A gather's loads are non-temporal where its source would push out what it writes (gather and scatter, 117 MiB
// 76 us so and plain, 234 MiB 144 / 169).
constexpr int64_t kRowsShort = (int64_t)14 << 20, kScatterStreamed = (int64_t)64 << 20;  // bytes of the rows of one side
constexpr int64_t kGatherStreamed = (int64_t)128 << 20;

// U: pieces of a thread.  LOADS, STORES: those that are non-temporal
template <bool SCATTER, int U, bool LOADS, bool STORES>
__global__ __launch_bounds__(256) void k_rows(const piece_t* __restrict__ src, piece_t* __restrict__ dst,
                                               const int32_t* __restrict__ perm, RowPieces rp) {
  for (int64_t i0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x; i0 < rp.total; i0 += (int64_t)gridDim.x * (256 * U)) {
    int64_t here[U], there[U];               // of the side in sorted order, and of the other
    piece_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * 256;
      here[u] = i < rp.total ? i : i0;
      const int64_t p = row_of(rp, here[u]);
      there[u] = here[u] + ((int64_t)perm[p] - p) * rp.per_row;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const piece_t* const from = src + (SCATTER ? here[u] : there[u]);
      v[u] = LOADS ? __builtin_nontemporal_load(from) : *from;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * 256 >= rp.total) continue;
      piece_t* const to = dst + (SCATTER ? there[u] : here[u]);
      if (STORES) __builtin_nontemporal_store(v[u], to);
      else        *to = v[u];
    }
  }
}

// Rows of sorted positions outside every group skip the layer ('Drop Residual', Sec. 4.3): for a
// residual layer that means out = feats.  A workgroup looks at 64 consecutive sorted positions; a
// position p is grouped when the last group start at or before p lies less than G before it.
template <typename T, typename TO>
__global__ __launch_bounds__(256) void k_copy_ungrouped(const T* __restrict__ feats, TO* __restrict__ out,
                                                         const int32_t* __restrict__ perm,
                                                         const int32_t* __restrict__ group_offsets,
                                                         const int32_t* __restrict__ num_groups, int max_groups,
                                                         int64_t n, int C, int G) {
  __shared__ int32_t row_of[64];
  const int64_t p0 = (int64_t)blockIdx.x * 64;
  if (threadIdx.x < 64) {
    const int64_t p = p0 + threadIdx.x;
    int32_t row = -1;
    if (p < n) {
      const int listed = num_groups ? *num_groups : 0, ng = listed < max_groups ? listed : max_groups;
      int lo = 0, hi = ng;  // first group start beyond p
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (group_offsets[mid] <= p) lo = mid + 1; else hi = mid;
      }
      if (ng >= 0 && (lo == 0 || p >= (int64_t)group_offsets[lo - 1] + G)) row = perm[p];  // (negative: no list)
    }
    row_of[threadIdx.x] = row;
  }
  __syncthreads();
  for (int r = 0; r < 64; ++r) {
    const int32_t row = row_of[r];
    if (row < 0) continue;
    for (int k = threadIdx.x; k < C; k += blockDim.x)
      Elem<TO>::store(out + (int64_t)row * C + k, Elem<T>::load(feats + (int64_t)row * C + k));
  }
}

// ---- sparse pillars -> dense bird's-eye-view map (the step after the FWA blocks, Sec. 5.1 'Model') -----
// bev[b][y][x][:] = feats[i][:] for pillar i = (b, x, y), zero elsewhere; channels last, so that a
// pillar's features stay one contiguous row.  Two launches: zero fill (the map is mostly empty:
// 30k of 219k cells at the paper's resolution), then the rows, a 16-byte piece per thread.
// What bounds it: memory, 37 of 48 us for four 468 x 468 maps of 128 bfloat16 (214 MiB) the fill's writes.  Non-temporal ones leave the
// memory-side cache to the rows that come after it, and the map to whoever reads it next in memory.  30,000 pillars a frame, from
// graphs, buffers that no cache holds, plain / non-temporal, us: the map alone 107 MiB 28.4 / 26.6, 160 MiB 40.9 / 38.4, 214 MiB 52.8 /
// 51.3, 428 MiB 105.4 / 96.9; with a launch behind it that reads the map 54 MiB 32.8 / 36.2, 107 MiB 62.7 / 66.7, 160 MiB 92.6 / 97.8, 187 MiB
// 111.1 / 114.1, 214 MiB 128.4 / 129.7, 267 MiB 160.1 / 159.5, 428 MiB 252.9 / 247.3.  Writing each cell once, with the pillars' numbers
// left in the map's last rows by a launch of their own and checked against the coordinates, was slower (52.9 to 74 us: the rows'
// addresses hang on two trips to memory).
constexpr int64_t kFillStreamed = (int64_t)200 << 20;  // bytes of a map

template <bool STREAM>
__global__ __launch_bounds__(256) void k_fill_zero(piece_t* __restrict__ dst, int64_t pieces) {
  const piece_t z = {0u, 0u, 0u, 0u};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < pieces; i += (int64_t)gridDim.x * blockDim.x) {
    if (STREAM) __builtin_nontemporal_store(z, dst + i);
    else        dst[i] = z;
  }
}

__global__ __launch_bounds__(256) void k_bev_scatter(const piece_t* __restrict__ feats, const int32_t* __restrict__ coords,
                                                      RowPieces rp, int B, int gx, int gy, piece_t* __restrict__ bev) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rp.total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = row_of(rp, i);
    const int32_t b = coords[3 * p], x = coords[3 * p + 1], y = coords[3 * p + 2];
    if ((uint32_t)b >= (uint32_t)B || (uint32_t)x >= (uint32_t)gx || (uint32_t)y >= (uint32_t)gy) continue;  // outside the map
    bev[(((int64_t)b * gy + y) * gx + x - p) * rp.per_row + i] = feats[i];
  }
}

}  // namespace

int bev_scatter_launch(const void* feats, const int32_t* coords, int64_t n, const ff_geom* g, int C, int dtype,
                       void* bev, hipStream_t stream) {
  if (!g || n < 0 || C < 1 || (dtype != FF_F32 && dtype != FF_BF16 && dtype != FF_F16)) return FF_ERR_ARG;
  if (g->num_frames < 1 || g->grid_x < 1 || g->grid_y < 1 || !bev) return FF_ERR_ARG;
  const size_t row_bytes = (size_t)C * (dtype == FF_F32 ? 4 : 2);
  if (row_bytes % 16) return FF_ERR_UNSUPPORTED;
  if (((uintptr_t)bev & 15) || ((uintptr_t)feats & 15)) return FF_ERR_ARG;
  if (n > 0 && (!feats || !coords)) return FF_ERR_ARG;
  const RowPieces rp = row_pieces(n, (int)(row_bytes / 16));
  const int64_t pieces = (int64_t)g->num_frames * g->grid_x * g->grid_y * rp.per_row;
  int64_t fb = ceil_div(pieces, 256 * 8);
  if (fb > 256 * 64) fb = 256 * 64;
  if (pieces * 16 > kFillStreamed) hipLaunchKernelGGL(k_fill_zero<true>, dim3((unsigned)fb), dim3(256), 0, stream, (piece_t*)bev, pieces);
  else hipLaunchKernelGGL(k_fill_zero<false>, dim3((unsigned)fb), dim3(256), 0, stream, (piece_t*)bev, pieces);
  if (n > 0) {
    const int64_t blocks = ceil_div(rp.total, 256);
    hipLaunchKernelGGL(k_bev_scatter, dim3((unsigned)(blocks < (1 << 20) ? blocks : 1 << 20)), dim3(256), 0, stream,
                       (const piece_t*)feats, coords, rp, g->num_frames, g->grid_x, g->grid_y, (piece_t*)bev);
  }
  return launch_status();
}

// ---- coordinate check: how many rows of coords lie outside the geometry -------------------------------------
// result[0] = rows with a frame, x or y outside [0, num_frames) x [0, grid_x) x [0, grid_y), result[1] = index of
// the first such row (n if there is none).  Two launches: the two words are set, then every workgroup adds its
// count (and lowers the index) with one atomic each.
__global__ void k_check_init(int32_t* __restrict__ result, int32_t n) { result[0] = 0; result[1] = n; }

__global__ __launch_bounds__(256) void k_check_coords(const int32_t* __restrict__ coords, int64_t n, int B, int gx, int gy,
                                                       int32_t* __restrict__ result) {
  __shared__ uint32_t bad_s;
  __shared__ int32_t first_s;
  if (threadIdx.x == 0) { bad_s = 0u; first_s = 0x7fffffff; }
  __syncthreads();
  uint32_t bad = 0;
  int32_t first = 0x7fffffff;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t b = coords[3 * i], x = coords[3 * i + 1], y = coords[3 * i + 2];
    if ((uint32_t)b >= (uint32_t)B || (uint32_t)x >= (uint32_t)gx || (uint32_t)y >= (uint32_t)gy) {
      ++bad;
      if ((int32_t)i < first) first = (int32_t)i;
    }
  }
  if (bad) { atomicAdd(&bad_s, bad); atomicMin(&first_s, first); }
  __syncthreads();
  if (threadIdx.x == 0 && bad_s) { atomicAdd(&result[0], (int32_t)bad_s); atomicMin(&result[1], first_s); }
}

int check_coords_launch(const int32_t* coords, int64_t n, const ff_geom* g, int32_t* result, hipStream_t stream) {
  if (!g || n < 0 || n > 0x7fffffffLL || !result || (n > 0 && !coords)) return FF_ERR_ARG;
  if (g->num_frames < 1 || g->grid_x < 1 || g->grid_y < 1) return FF_ERR_ARG;
  hipLaunchKernelGGL(k_check_init, dim3(1), dim3(1), 0, stream, result, (int32_t)n);
  if (n > 0) {
    int64_t blocks = ceil_div(n, 256 * 4);
    if (blocks > 256 * 8) blocks = 256 * 8;
    hipLaunchKernelGGL(k_check_coords, dim3((unsigned)blocks), dim3(256), 0, stream, coords, n, g->num_frames, g->grid_x,
                       g->grid_y, result);
  }
  return launch_status();
}

int rows_copy_ungrouped_launch(const void* feats, void* out, int64_t n, const int32_t* perm,
                               const int32_t* group_offsets, const int32_t* num_groups, int32_t max_groups, int C,
                               int G, int dtype, bool out_f32, hipStream_t stream) {
  if (n < 0 || C < 1 || G < 1 || max_groups < 0 || (dtype != FF_F32 && dtype != FF_BF16 && dtype != FF_F16)) return FF_ERR_ARG;
  if (n == 0) return FF_OK;
  if (!feats || !out || !perm || (max_groups > 0 && (!group_offsets || !num_groups))) return FF_ERR_ARG;
  const dim3 grid((unsigned)ceil_div(n, 64)), block(256);
  if (dtype == FF_F32)
    hipLaunchKernelGGL((k_copy_ungrouped<float, float>), grid, block, 0, stream, (const float*)feats, (float*)out,
                       perm, group_offsets, num_groups, (int)max_groups, n, C, G);
  else if (out_f32 && dtype == FF_F16)
    hipLaunchKernelGGL((k_copy_ungrouped<f16_t, float>), grid, block, 0, stream, (const f16_t*)feats, (float*)out,
                       perm, group_offsets, num_groups, (int)max_groups, n, C, G);
  else if (out_f32)
    hipLaunchKernelGGL((k_copy_ungrouped<bf16_t, float>), grid, block, 0, stream, (const bf16_t*)feats, (float*)out,
                       perm, group_offsets, num_groups, (int)max_groups, n, C, G);
  else  // 16 bits to the same 16 bits: a bit copy for either format
    hipLaunchKernelGGL((k_copy_ungrouped<bf16_t, bf16_t>), grid, block, 0, stream, (const bf16_t*)feats,
                       (bf16_t*)out, perm, group_offsets, num_groups, (int)max_groups, n, C, G);
  return launch_status();
}

int rows_launch(bool scatter, const void* src, void* dst, const int32_t* perm, int64_t n, int C,
                int dtype, hipStream_t stream) {
  if (n < 0 || C < 1 || (dtype != FF_F32 && dtype != FF_BF16 && dtype != FF_F16)) return FF_ERR_ARG;
  const size_t row_bytes = (size_t)C * (dtype == FF_F32 ? 4 : 2);
  if (row_bytes % 16) return FF_ERR_UNSUPPORTED;
  if (n == 0) return FF_OK;
  if (!src || !dst || !perm || src == dst) return FF_ERR_ARG;
  if (((uintptr_t)src | (uintptr_t)dst) & 15) return FF_ERR_ARG;
  const RowPieces rp = row_pieces(n, (int)(row_bytes / 16));
  auto go = [&](auto kern, int pieces) {
    const int64_t blocks = ceil_div(rp.total, (int64_t)256 * pieces);
    hipLaunchKernelGGL(kern, dim3((unsigned)(blocks < (1 << 20) ? blocks : 1 << 20)), dim3(256), 0, stream, (const piece_t*)src,
                       (piece_t*)dst, perm, rp);
  };
  const int64_t bytes = rp.total * 16;
  if (scatter) {
    if (bytes <= kRowsShort) go(k_rows<true, 1, true, false>, 1);
    else if (bytes <= kScatterStreamed) go(k_rows<true, 2, true, false>, 2);
    else go(k_rows<true, 2, true, true>, 2);
  } else {
    if (bytes <= kRowsShort) go(k_rows<false, 1, false, false>, 1);
    else if (bytes <= kGatherStreamed) go(k_rows<false, 2, false, false>, 2);
    else go(k_rows<false, 2, true, false>, 2);
  }
  return launch_status();
}

}  // namespace ff
