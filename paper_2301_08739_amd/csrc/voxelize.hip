// Pillar voxelisation, the step in front of the FWA blocks (paper Sec. 5.1 'Model': the point cloud
// is voxelised into sparse bird's-eye-view pillars of 0.32 m x 0.32 m).  Here in its plain form: a
// pillar is a non-empty cell, its feature vector the mean of its points' feature vectors, pillars
// come out in ascending (frame, x, y) order; the learned per-point network of PointPillars is not
// part of it.  HBM/latency bound integer work that reuses the window sort:
//   flatten         the radix argsort of flatten.hip with 1 x 1 windows, its key generation fed by the points:
//                   cell of every point (float32: floor((x - x_min) / voxel)), dropped points -> frame B,
//                   points ordered by (frame, x, y)
//   k_seg_count     per 1024 sorted points: how many cells start there
//   k_seg_scan      exclusive prefix over those counts, total = number of pillars (above 262,144 points only)
//   k_seg_starts    numbers the cell starts: start position and cell of every pillar
//   k_seg_mean      means of the pillars' points' features, point -> pillar
// Grids of up to half a million cells take three launches instead (k_vox_split, k_vox_order, k_vox_mean below).
#include "common.h"
#include "sort_device.h"
#include <type_traits>

namespace ff {
namespace {

constexpr int kSegBlock = 1024;
constexpr int kPointsInFlight = 8;  // per lane of pillar_mean
constexpr int kSegDirectBlocks = 256;  // up to 262,144 points the blocks' prefixes need no launch of their own

// exported key of the sort: frame << 48 | x << 32 | y << 16 (window 1 x 1: no local fields)
// The key at sorted position p and the one before it, loaded without conditions (positions clamped
// into the array) so that a thread's loads travel together; starts_cell then tells whether p is the
// first point of a cell inside the grid.
struct KeyPair { uint64_t k, before; };
__device__ __forceinline__ KeyPair load_pair(const uint64_t* __restrict__ keys, int64_t p, int64_t m) {
  const int64_t pc = p < m ? p : m - 1;
  return {keys[pc], keys[pc > 0 ? pc - 1 : 0]};
}
__device__ __forceinline__ bool starts_cell(const KeyPair& kp, int64_t p, int64_t m, int B) {
  return p < m && (int)(kp.k >> 48) < B && (p == 0 || kp.before != kp.k);
}

__global__ __launch_bounds__(256) void k_seg_count(const uint64_t* __restrict__ keys, int64_t m, int B,
                                                    uint32_t* __restrict__ block_counts, int32_t* __restrict__ kept) {
  __shared__ uint32_t wave_sums[4];
  if (blockIdx.x == 0 && threadIdx.x == 0) *kept = (int32_t)m;  // lowered by k_seg_starts
  const int64_t p0 = (int64_t)blockIdx.x * kSegBlock;
  uint32_t c = 0;
  if (m > 0) {  // the same for every thread
    KeyPair kp[kSegBlock / 256];
#pragma unroll
    for (int r = 0; r < kSegBlock / 256; ++r) kp[r] = load_pair(keys, p0 + r * 256 + threadIdx.x, m);
#pragma unroll
    for (int r = 0; r < kSegBlock / 256; ++r)
      if (starts_cell(kp[r], p0 + r * 256 + threadIdx.x, m, B)) ++c;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
  if ((threadIdx.x & 63) == 0) wave_sums[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) block_counts[blockIdx.x] = wave_sums[0] + wave_sums[1] + wave_sums[2] + wave_sums[3];
}

// One workgroup: block_counts -> exclusive prefixes in place, total -> *num_pillars.  Only for more
// blocks than k_seg_starts adds up by itself.
__global__ __launch_bounds__(1024) void k_seg_scan(uint32_t* __restrict__ block_counts, int64_t nb,
                                                    int32_t* __restrict__ num_pillars) {
  __shared__ uint32_t wave_sums[16];
  __shared__ uint32_t carry_s;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int64_t base = 0; base < nb; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const uint32_t v = i < nb ? block_counts[i] : 0u;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t t = __shfl_up(inc, d, 64);
      if (lane >= d) inc += t;
    }
    if (lane == 63) wave_sums[w] = inc;
    __syncthreads();
    uint32_t before = carry_s, total = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const uint32_t t = wave_sums[k];
      if (k < w) before += t;
      total += t;
    }
    if (i < nb) block_counts[i] = before + inc - v;
    __syncthreads();
    if (threadIdx.x == 0) carry_s += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) *num_pillars = (int32_t)carry_s;
}

// Cell starts get their pillar numbers (block-local scan on top of the block's prefix): writes where
// each pillar's run of sorted points starts, its cell, and -1 for the points that were dropped.
// SCANNED: block_base holds exclusive prefixes (k_seg_scan ran).  Otherwise it holds the blocks'
// counts and every workgroup adds up the ones before it (a few KB from L2: cheaper than a dependent
// launch); workgroup 0 also writes the total.
template <bool SCANNED>
__global__ __launch_bounds__(256) void k_seg_starts(const uint64_t* __restrict__ keys, const int32_t* __restrict__ perm,
                                                     int64_t m, int B, const uint32_t* __restrict__ block_base, int nb,
                                                     int32_t* __restrict__ num_pillars,
                                                     int32_t* __restrict__ starts, int32_t* __restrict__ kept,
                                                     int32_t* __restrict__ coords, int32_t* __restrict__ point_to_pillar) {
  __shared__ uint32_t wave_sums[4];
  __shared__ uint32_t base_sums[4][2];
  uint32_t base = 0;
  if (SCANNED) {
    base = block_base[blockIdx.x];
  } else {
    uint32_t before = 0, all = 0;
    for (int i = threadIdx.x; i < nb; i += 256) {
      const uint32_t c = block_base[i];
      all += c;
      if (i < (int)blockIdx.x) before += c;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) { before += __shfl_xor(before, d, 64); all += __shfl_xor(all, d, 64); }
    if ((threadIdx.x & 63) == 0) { base_sums[threadIdx.x >> 6][0] = before; base_sums[threadIdx.x >> 6][1] = all; }
    __syncthreads();
    base = base_sums[0][0] + base_sums[1][0] + base_sums[2][0] + base_sums[3][0];
    if (blockIdx.x == 0 && threadIdx.x == 0)
      *num_pillars = (int32_t)(base_sums[0][1] + base_sums[1][1] + base_sums[2][1] + base_sums[3][1]);
  }
  const int64_t p0 = (int64_t)blockIdx.x * kSegBlock;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // thread t owns positions p0 + 4t .. p0 + 4t + 3, so that cell starts are numbered in sorted order
  bool head[4];
  KeyPair kp[4];
  uint32_t mine = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) kp[r] = m > 0 ? load_pair(keys, p0 + 4 * threadIdx.x + r, m) : KeyPair{0, 0};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    head[r] = starts_cell(kp[r], p0 + 4 * threadIdx.x + r, m, B);
    mine += head[r] ? 1u : 0u;
  }
  uint32_t inc = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(inc, d, 64);
    if (lane >= d) inc += t;
  }
  if (lane == 63) wave_sums[w] = inc;
  __syncthreads();
  uint32_t pid = base + inc - mine;
  for (int k = 0; k < w; ++k) pid += wave_sums[k];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t p = p0 + 4 * threadIdx.x + r;
    if (p >= m) continue;
    const uint64_t k = kp[r].k;
    if ((int)(k >> 48) >= B) {  // dropped points sort behind all pillars
      if (point_to_pillar) point_to_pillar[perm[p]] = -1;
      if (p == 0 || (int)(kp[r].before >> 48) < B) *kept = (int32_t)p;
    }
    if (!head[r]) continue;
    starts[pid] = (int32_t)p;
    coords[3 * (int64_t)pid + 0] = (int32_t)(k >> 48);
    coords[3 * (int64_t)pid + 1] = (int32_t)((k >> 32) & 0xffffu);
    coords[3 * (int64_t)pid + 2] = (int32_t)((k >> 16) & 0xffffu);
    ++pid;
  }
}

// v of the lane D further in its row of sixteen
template <int D> __device__ __forceinline__ float row_turned(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x120 + D, 0xf, 0xf, false));
}

// Sixteen lanes per pillar: lane l adds the points l, l + 16, ... of the pillar's run lo .. hi of perm in float32, the
// sixteen partial sums are combined in a fixed tree, so the result does not depend on timing.  vec4: rows of four features
// in one 16-byte load.
__device__ __forceinline__ void pillar_mean(int64_t pid, int lo, int hi, const int32_t* __restrict__ perm,
                                            const float* __restrict__ pfeats, int Cp, bool vec4, float* __restrict__ feats,
                                            int32_t* __restrict__ point_to_pillar) {
  const int sub = threadIdx.x & 15;
  const float inv = 1.0f / (float)(hi - lo);
  for (int c0 = 0; c0 < Cp; c0 += 4) {  // four features at a time
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    auto points = [&](int q, auto in_flight, int32_t (&src)[kPointsInFlight]) {  // q, q + 16, .. of the pillar, -1: none
      constexpr int U = decltype(in_flight)::value;
#pragma unroll
      for (int u = 0; u < U; ++u) src[u] = q + 16 * u < hi ? perm[q + 16 * u] : -1;
    };
    auto add = [&](const int32_t (&src)[kPointsInFlight], auto in_flight) {  // their loads in flight together
      constexpr int U = decltype(in_flight)::value;
      if (point_to_pillar && c0 == 0) {  // the point indices are at hand here (Cp >= 1: this round always runs)
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (src[u] >= 0) point_to_pillar[src[u]] = (int32_t)pid;
      }
      float v[U][4];
      if (vec4) {  // four features of a point in one 16-byte load (the same for every thread)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float4 t = *reinterpret_cast<const float4*>(pfeats + (int64_t)(src[u] >= 0 ? src[u] : 0) * Cp + c0);
          v[u][0] = src[u] >= 0 ? t.x : 0.f; v[u][1] = src[u] >= 0 ? t.y : 0.f;
          v[u][2] = src[u] >= 0 ? t.z : 0.f; v[u][3] = src[u] >= 0 ? t.w : 0.f;
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            v[u][j] = src[u] >= 0 && c0 + j < Cp ? pfeats[(int64_t)src[u] * Cp + c0 + j] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] += v[u][j];
    };
    // Most pillars hold a few points: one point per lane then, where eight rounds of masked loads were issued before.
    // Eight in flight for the others: a pillar of several hundred points (a dense object, the cell under the sensor)
    // is a chain of dependent round trips otherwise (sixteen were no faster).  The four pillars of a wavefront go the
    // same way: with one of them long, the others' single round would come on top of its rounds.  The whole call, us,
    // eight rounds for all / each pillar its own way / this: 180,000 points of 3, 4, 5 and 8 features 62 / 63 / 57, 60 /
    // 53 / 53, 71 / 74 / 67, 67 / 60 / 60; 1.44 M of 3 and 5 155 / 157 / 148 and 191 / 187 / 177; 60,000 of 5 50 / 52 / 51.
    // The same bits.
    constexpr auto one = std::integral_constant<int, 1>();
    constexpr auto many = std::integral_constant<int, kPointsInFlight>();
    int32_t src[kPointsInFlight];
    if (!__builtin_amdgcn_ballot_w64(hi - lo > 16)) {
      if (lo + sub < hi) {
        points(lo + sub, one, src);
        add(src, one);
      }
    } else {                             // (the next round's points are fetched beside this one's features)
      points(lo + sub, many, src);
      for (int q = lo + sub; q < hi; q += 16 * kPointsInFlight) {
        int32_t next[kPointsInFlight];
        points(q + 16 * kPointsInFlight, many, next);
        add(src, many);
#pragma unroll
        for (int u = 0; u < kPointsInFlight; ++u) src[u] = next[u];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int d = 0; d < 4; ++d) acc[j] += d == 0 ? row_turned<8>(acc[j]) : d == 1 ? row_turned<4>(acc[j]) : d == 2 ? row_turned<2>(acc[j]) : row_turned<1>(acc[j]);
      if (sub == 0 && c0 + j < Cp) feats[pid * Cp + c0 + j] = acc[j] * inv;
    }
  }
}
__device__ __forceinline__ bool rows_of_four(const float* pfeats, int Cp) {
  return Cp % 4 == 0 && (reinterpret_cast<uintptr_t>(pfeats) & 15) == 0;
}

__global__ __launch_bounds__(256) void k_seg_mean(const int32_t* __restrict__ perm, const float* __restrict__ pfeats,
                                                   int Cp, const int32_t* __restrict__ num_pillars,
                                                   const int32_t* __restrict__ starts, const int32_t* __restrict__ kept,
                                                   float* __restrict__ feats, int32_t* __restrict__ point_to_pillar) {
  const int np = *num_pillars;
  const bool vec4 = rows_of_four(pfeats, Cp);
  const int64_t stride = (int64_t)gridDim.x * (blockDim.x / 16);
  for (int64_t pid = (int64_t)blockIdx.x * (blockDim.x / 16) + (threadIdx.x >> 4); pid < np; pid += stride)
    pillar_mean(pid, starts[pid], pid + 1 < np ? starts[pid + 1] : *kept, perm, pfeats, Cp, vec4, feats, point_to_pillar);
}

// ---- grids of up to kVoxMaxRanges * 256 cells in three launches -----------------------------------------------------
// The cells, in the order (frame, x, y), are cut into ranges of 256.  k_vox_split sorts each tile of the points by range, in
// place of a key: the table of where a range begins in a tile says all that the next launch needs, and the sums of a column
// how many points lie in front of the range.  k_vox_order, a workgroup per range, brings its pieces of all tiles into LDS and
// sorts them by cell.  k_vox_mean, with the pillars in front of each range known, numbers them and takes the means.  Both
// sorts keep the order of the points (ranks of equal numbers in a wavefront, counters of its own for each wavefront), so a
// pillar's points come in the order of their indices.
//
// What bounds it: three dependent launches, each a chain of four to six round trips to memory (8.4 + 10.2 + 19 us for 180,000
// points of one frame, 4 of each the launch itself), not the 7 MB moved.  In front of them were nine launches, keys of 64 bits
// through two radix passes.  The call, us, before / this: 2,000 points 31 / 17, 20,000 36 / 20, 60,000 of 5 features 48 / 28,
// 180,000 of 4 50.5 / 34.7, of 8 56.3 / 41, 262,144 of two frames 55 / 50.  Ranges of 1024 cells, which cover four times the
// grid: 180,000 47.9 us, and 1.44 M points of eight frames 177, which the general path takes 137 for.  Rows brought into LDS by
// the whole workgroup before they are added up, or four lanes to a short pillar: k_vox_mean 19 to 40 us instead of 17.
// Thousands of points in a single cell are one workgroup's, and one chain of sums as ever: 60,000 of 4 features 505 / 620 us, 180,000
// 1.63 / 1.95 ms, of 5 features 4.8 / 6.5 (the general path's radix passes spread them over the chip).
constexpr int kVoxThreads = 1024, kVoxWaves = kVoxThreads / 64;              // of k_vox_split
constexpr int kVoxOrderThreads = 512, kVoxOrderWaves = kVoxOrderThreads / 64;
constexpr int kVoxCellBits = 8;             // cells of a range: 256
constexpr int kVoxMaxRanges = 1983;         // with one more bin for the points that are dropped, the counters of k_vox_split take 62 KB
constexpr int kVoxPoints = 2;               // points of a thread of k_vox_split
constexpr int kVoxTile = kVoxThreads * kVoxPoints, kVoxLocalBits = 11;
constexpr int kVoxMaxTiles = 248;           // (as many points as cells)
constexpr uint32_t kVoxMaxTilesPow = 256;
constexpr int kVoxIndexBits = 19;           // points: index and cell of the range share a word of 32 bits
constexpr int kVoxList = 4096;              // points in LDS at a time
constexpr int kVoxInFlight = 8;            // points of a lane on their way there
constexpr int kVoxManyRanges = 256;         // more than this many have four workgroups each in k_vox_mean (180,000 points in
                                            // 855 ranges: two 23 us, four 17, six 20), fewer sixteen
static_assert(kVoxTile == 1 << kVoxLocalBits && kVoxMaxTiles <= kVoxOrderThreads && kVoxMaxTiles * kVoxTile <= 1 << kVoxIndexBits &&
              kVoxMaxRanges << kVoxCellBits <= kVoxMaxTiles * kVoxTile && kVoxMaxTiles <= (int)kVoxMaxTilesPow, "");

// entries: of tile t, at t * kVoxTile, its points sorted by range: cell of the range << 13 | point of the tile.
// table[t][bin]: where the range begins there; the bin behind the last range is that of the dropped points.
__global__ __launch_bounds__(kVoxThreads) void k_vox_split(PointCells pts, int m, int bins, int bin_bits,
                                                            uint32_t* __restrict__ entries, uint32_t* __restrict__ table,
                                                            int32_t* __restrict__ point_to_pillar) {
  extern __shared__ uint32_t words[];        // [kVoxWaves][bins / 2]: counts of two bins
  __shared__ uint32_t wave_totals[kVoxWaves];
  const int tid = threadIdx.x, lane = tid & 63, half = bins >> 1, dropped_bin = bins - 1;
  const int tile0 = blockIdx.x * kVoxTile, local0 = (tid >> 6) * 64 * kVoxPoints + lane;
  uint16_t* const mine = reinterpret_cast<uint16_t*>(words + (tid >> 6) * half);
  uint32_t id[kVoxPoints], rank[kVoxPoints];                 // cell of all frames
#pragma unroll
  for (int u = 0; u < kVoxPoints; ++u) {
    const int i = tile0 + local0 + u * 64;
    int32_t c[4];
    point_cell(pts, i < m ? i : m - 1, c);
    id[u] = c[0] < pts.B ? ((uint32_t)c[0] * (uint32_t)pts.grid_x + (uint32_t)c[1]) * (uint32_t)pts.grid_y + (uint32_t)c[2]
                         : (uint32_t)dropped_bin << kVoxCellBits;
    if (i >= m) id[u] = (uint32_t)dropped_bin << kVoxCellBits;
    else if (c[0] >= pts.B && point_to_pillar) point_to_pillar[i] = -1;
  }
  for (int w = tid; w < kVoxWaves * half; w += kVoxThreads) words[w] = 0u;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kVoxPoints; ++u) rank[u] = rank_in_wave(mine, id[u] >> kVoxCellBits, bin_bits, true);
  __syncthreads();
  const uint32_t total = tid < half ? sum_over_waves<kVoxWaves>(words, half, tid) : 0u;
  const uint32_t first = block_exclusive_scan<kVoxThreads>((total & 0xffffu) + (total >> 16), wave_totals, nullptr);
  if (tid < half) {
    const uint32_t both = first | (first + (total & 0xffffu)) << 16;
    table[blockIdx.x * half + tid] = both;
#pragma unroll
    for (int w = 0; w < kVoxWaves; ++w) words[w * half + tid] += both;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kVoxPoints; ++u) {
    const uint32_t bin = id[u] >> kVoxCellBits;
    if (bin != (uint32_t)dropped_bin)
      entries[tile0 + mine[bin] + rank[u]] = (id[u] & ((1u << kVoxCellBits) - 1u)) << kVoxLocalBits | (uint32_t)(local0 + u * 64);
  }
}

// order: the points, sorted by cell.  The pillars of a range, from where its points begin: starts (in order) and cells.
__global__ __launch_bounds__(kVoxOrderThreads) void k_vox_order(const uint32_t* __restrict__ entries, const uint16_t* __restrict__ table,
                                                            int tiles, int bins, int32_t* __restrict__ order,
                                                            int32_t* __restrict__ starts, uint32_t* __restrict__ cells,
                                                            uint32_t* __restrict__ range_pillars, uint32_t* __restrict__ range_end) {
  constexpr int CELLS = 1 << kVoxCellBits, ROUNDS = kVoxList / kVoxOrderThreads;
  extern __shared__ uint32_t list[];                       // [kVoxList] cell of the range << 22 | point
  uint32_t* const words = list + kVoxList;                 // [kVoxOrderWaves][CELLS / 2]: counts of two cells
  uint32_t* const place = words + kVoxOrderWaves * CELLS / 2;   // [CELLS] where the cell's next point goes
  uint32_t* const cum = place + CELLS;                     // [kVoxMaxTiles + 1] the range's points in the tiles before,
  uint32_t* const from = cum + kVoxMaxTiles + 1;           // [kVoxMaxTiles] and where those of a tile are
  __shared__ uint32_t wave_totals[2 * kVoxOrderWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, range = blockIdx.x;
  uint32_t s = 0, e = 0, T, base;
  if (tid < tiles) {
    s = table[(size_t)tid * bins + range];
    e = table[(size_t)tid * bins + range + 1];
  }
  const uint32_t before = block_exclusive_scan_and_sum<kVoxOrderThreads>(e - s, s, wave_totals, &T, &base);
  if (tid == 0) {
    range_end[range] = base + T;
    if (T == 0u) range_pillars[range] = 0u;
  }
  if (T == 0u) return;
  if (tid < tiles) {
    cum[tid] = before;
    from[tid] = (uint32_t)tid * (uint32_t)kVoxTile + s;
  }
  if (tid == 0) cum[tiles] = T;
  uint16_t* const mine = reinterpret_cast<uint16_t*>(words + wave * (CELLS / 2));
  // lanes that bring a tile's points: few, for as many tiles at a time, unless there are many points
  const int lane_bits = T <= 64u * (uint32_t)tiles ? 2 : T <= 512u * (uint32_t)tiles ? 4 : 6;
  const uint32_t lanes = 1u << lane_bits;
  uint32_t rank[ROUNDS];
  int chunks = 0, at = 0;
  uint32_t len = 0;
  // Points list0 .. list0 + kVoxList of the range: into the list, their ranks, the counts of cells 2 tid and 2 tid + 1.
  auto take = [&](uint32_t list0) -> uint32_t {
    __syncthreads();
    len = T - list0 < (uint32_t)kVoxList ? T - list0 : (uint32_t)kVoxList;
    for (int w = tid; w < kVoxOrderWaves * CELLS / 2; w += kVoxOrderThreads) words[w] = 0u;
    if (lane_bits == 6 && T > (uint32_t)kVoxList) {  // a few tiles' pieces, too few for the wavefronts: each point finds its tile, the last that
      uint32_t tile[ROUNDS] = {}, v[ROUNDS]; // begins no later
#pragma unroll
      for (uint32_t step = kVoxMaxTilesPow / 2; step > 0; step >>= 1)
#pragma unroll
        for (int u = 0; u < ROUNDS; ++u) {
          const uint32_t p = (uint32_t)(tid + u * kVoxOrderThreads) < len ? list0 + tid + u * kVoxOrderThreads : list0;
          tile[u] += tile[u] + step < (uint32_t)tiles && cum[tile[u] + step] <= p ? step : 0u;
        }
#pragma unroll
      for (int u = 0; u < ROUNDS; ++u) {
        const uint32_t p = (uint32_t)(tid + u * kVoxOrderThreads) < len ? list0 + tid + u * kVoxOrderThreads : list0;
        v[u] = entries[from[tile[u]] + p - cum[tile[u]]];
      }
#pragma unroll
      for (int u = 0; u < ROUNDS; ++u)
        if ((uint32_t)(tid + u * kVoxOrderThreads) < len)
          list[tid + u * kVoxOrderThreads] = v[u] >> kVoxLocalBits << kVoxIndexBits |
                                             (tile[u] * (uint32_t)kVoxTile + (v[u] & ((1u << kVoxLocalBits) - 1u)));
    } else {
      for (int t = tid >> lane_bits; t < tiles; t += kVoxOrderThreads >> lane_bits) {
        const uint32_t c0 = cum[t], c1 = cum[t + 1], src = from[t] - c0;
        const uint32_t stop = c1 < list0 + len ? c1 : list0 + len;
        for (uint32_t p = (c0 > list0 ? c0 : list0) + (tid & (lanes - 1u)); p < stop; p += lanes * kVoxInFlight) {
          uint32_t v[kVoxInFlight];
#pragma unroll
          for (int u = 0; u < kVoxInFlight; ++u) v[u] = entries[src + (p + lanes * u < stop ? p + lanes * u : p)];
#pragma unroll
          for (int u = 0; u < kVoxInFlight; ++u)
            if (p + lanes * u < stop)
              list[p + lanes * u - list0] = v[u] >> kVoxLocalBits << kVoxIndexBits |
                                         ((uint32_t)t * (uint32_t)kVoxTile + (v[u] & ((1u << kVoxLocalBits) - 1u)));
        }
      }
    }
    __syncthreads();
    chunks = (int)((len + kVoxOrderThreads - 1u) / kVoxOrderThreads);   // of 64 points, of each wavefront
    at = wave * chunks * 64 + lane;
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
      if (u < chunks) {
        const bool valid = (uint32_t)(at + u * 64) < len;
        rank[u] = rank_in_wave(mine, valid ? list[at + u * 64] >> kVoxIndexBits : 0u, kVoxCellBits, valid);
      }
    __syncthreads();
    return tid < CELLS / 2 ? sum_over_waves<kVoxOrderWaves>(words, CELLS / 2, tid) : 0u;
  };
  auto put = [&] {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
      if (u < chunks && (uint32_t)(at + u * 64) < len) {
        const uint32_t v = list[at + u * 64], cell = v >> kVoxIndexBits;
        order[base + place[cell] + mine[cell] + rank[u]] = (int32_t)(v & ((1u << kVoxIndexBits) - 1u));
      }
  };
  uint32_t total, c0 = 0, c1 = 0;
  if (T <= (uint32_t)kVoxList) {
    total = take(0u);
    c0 = total & 0xffffu;
    c1 = total >> 16;
  } else {                                   // several lists: the cells' points are counted in front of them
    for (int c = tid; c < CELLS; c += kVoxOrderThreads) place[c] = 0u;
    __syncthreads();
    for (int t = tid >> lane_bits; t < tiles; t += kVoxOrderThreads >> lane_bits) {
      const uint32_t n = cum[t + 1] - cum[t];
      for (uint32_t p = tid & (lanes - 1u); p < n; p += lanes * kVoxInFlight) {
        uint32_t v[kVoxInFlight];
#pragma unroll
        for (int u = 0; u < kVoxInFlight; ++u) v[u] = entries[from[t] + (p + lanes * u < n ? p + lanes * u : p)];
#pragma unroll
        for (int u = 0; u < kVoxInFlight; ++u)
          if (p + lanes * u < n) {           // (all of one cell: one addition, where they would wait for each other)
            const uint32_t cell = v[u] >> kVoxLocalBits, of_first = (uint32_t)__builtin_amdgcn_readfirstlane((int)cell);
            const uint64_t here = __ballot(true);
            if (__ballot(cell != of_first) == 0ull) {
              if (lanes_below(here) == 0u) atomicAdd(&place[cell], (uint32_t)__popcll(here));
            } else {
              atomicAdd(&place[cell], 1u);
            }
          }
      }
    }
    __syncthreads();
    if (tid < CELLS / 2) {
      c0 = place[2 * tid];
      c1 = place[2 * tid + 1];
    }
  }
  uint32_t np;                               // points and pillars in one scan
  const uint32_t both = block_exclusive_scan<kVoxOrderThreads>((c0 + c1) | ((c0 ? 1u : 0u) + (c1 ? 1u : 0u)) << kVoxIndexBits, wave_totals, &np);
  const uint32_t pos = both & ((1u << kVoxIndexBits) - 1u);
  uint32_t pillar = both >> kVoxIndexBits;
  np >>= kVoxIndexBits;
  if (tid < CELLS / 2) {
    place[2 * tid] = pos;
    place[2 * tid + 1] = pos + c0;
    if (c0) {
      starts[base + pillar] = (int32_t)(base + pos);
      cells[base + pillar] = (uint32_t)(range * CELLS + 2 * tid);
      ++pillar;
    }
    if (c1) {
      starts[base + pillar] = (int32_t)(base + pos + c0);
      cells[base + pillar] = (uint32_t)(range * CELLS + 2 * tid + 1);
    }
  }
  if (tid == 0) range_pillars[range] = np;
  if (T <= (uint32_t)kVoxList) {
    put();
    return;
  }
  for (uint32_t list0 = 0; list0 < T; list0 += kVoxList) {
    total = take(list0);
    put();
    __syncthreads();
    if (tid < CELLS / 2) {
      place[2 * tid] += total & 0xffffu;
      place[2 * tid + 1] += total >> 16;
    }
  }
}

__global__ __launch_bounds__(256) void k_vox_mean(const int32_t* __restrict__ order, const int32_t* __restrict__ starts,
                                                   const uint32_t* __restrict__ cells, const uint32_t* __restrict__ range_pillars,
                                                   const uint32_t* __restrict__ range_end, int ranges, int parts, int grid_x, int grid_y,
                                                   const float* __restrict__ pfeats, int Cp, int32_t* __restrict__ coords,
                                                   float* __restrict__ feats, int32_t* __restrict__ num_pillars,
                                                   int32_t* __restrict__ point_to_pillar) {
  __shared__ uint32_t sums[4];
  const int range = blockIdx.x / (unsigned)parts, part = blockIdx.x % (unsigned)parts, tid = threadIdx.x;
  // All that does not depend on anything, together
  constexpr int LOOKS = (kVoxMaxRanges + 255) / 256;
  uint32_t look[LOOKS], front = 0;
#pragma unroll
  for (int u = 0; u < LOOKS; ++u) look[u] = tid + 256 * u < range ? range_pillars[tid + 256 * u] : 0u;
  const int np = (int)range_pillars[range], end = (int)range_end[range], base = range > 0 ? (int)range_end[range - 1] : 0;
  if (part * 16 >= np && (range != ranges - 1 || part > 0)) return;
#pragma unroll
  for (int u = 0; u < LOOKS; ++u) front += look[u];
  front = wave_sum(front);
  if ((tid & 63) == 0) sums[tid >> 6] = front;
  __syncthreads();
  front = sums[0] + sums[1] + sums[2] + sums[3];
  if (range == ranges - 1 && part == 0 && tid == 0) *num_pillars = (int32_t)front + np;
  const bool vec4 = rows_of_four(pfeats, Cp);
  for (int k = part * 16 + (tid >> 4); k < np; k += parts * 16) {
    const int64_t pid = (int64_t)front + k;
    const int lo = starts[base + k], hi = k + 1 < np ? starts[base + k + 1] : end;
    if ((tid & 15) == 0) {
      const uint32_t cell = cells[base + k], row = cell / (uint32_t)grid_y, frame = row / (uint32_t)grid_x;
      coords[3 * pid + 0] = (int32_t)frame;
      coords[3 * pid + 1] = (int32_t)(row - frame * (uint32_t)grid_x);
      coords[3 * pid + 2] = (int32_t)(cell - row * (uint32_t)grid_y);
    }
    pillar_mean(pid, lo, hi, order, pfeats, Cp, vec4, feats, point_to_pillar);
  }
}

struct VoxLayout {
  ff_geom geom;  // the geometry the sort sees: one extra frame, 1 x 1 windows
  size_t off_perm, off_keys, off_goff, off_ng, off_blocks, off_starts, off_flat, flat_bytes, total;
  int64_t nb;
};

int make_vox_layout(int64_t m, const ff_geom* g, VoxLayout* L) {
  if (!g || m < 0 || m > 0x7fffffffLL) return FF_ERR_ARG;
  if (g->num_frames < 1 || g->num_frames > 65534 || g->grid_x < 1 || g->grid_x > 65535 || g->grid_y < 1 ||
      g->grid_y > 65535)
    return FF_ERR_ARG;
  L->geom = *g;
  L->geom.num_frames = g->num_frames + 1;
  L->geom.win_x = L->geom.win_y = 1;
  L->flat_bytes = flatten_workspace_bytes(m, &L->geom, 1);
  if (L->flat_bytes == 0) return FF_ERR_UNSUPPORTED;
  L->nb = ceil_div(m > 0 ? m : 1, kSegBlock);
  size_t off = 0;
  L->off_perm = off;   off += align_up((size_t)m * 4, 256);
  L->off_keys = off;   off += align_up((size_t)m * 8, 256);
  L->off_goff = off;   off += align_up((size_t)(L->geom.num_frames + 2) * 4, 256);  // one group per frame
  L->off_ng = off;     off += 256;
  L->off_blocks = off; off += align_up((size_t)L->nb * 4, 256);
  L->off_starts = off; off += align_up((size_t)(m + 1) * 4, 256);
  L->off_flat = off;   off += align_up(L->flat_bytes, 256);
  L->total = off;
  return FF_OK;
}

}  // namespace

size_t voxelize_workspace_bytes(int64_t m, const ff_geom* g) {
  VoxLayout L;
  return make_vox_layout(m, g, &L) == FF_OK ? L.total : 0;
}

int voxelize_launch(const float* xy, const int32_t* frame, const float* pfeats, int64_t m, int Cp, const ff_geom* g,
                    const ff_voxel_grid* v, int32_t* coords, float* feats, int32_t* num_pillars,
                    int32_t* point_to_pillar, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  VoxLayout L;
  int st = make_vox_layout(m, g, &L);
  if (st != FF_OK) return st;
  if (!v || !(v->voxel_x > 0.f) || !(v->voxel_y > 0.f) || Cp < 1 || !num_pillars) return FF_ERR_ARG;
  if (m > 0 && (!xy || !pfeats || !coords || !feats)) return FF_ERR_ARG;
  if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < L.total) return FF_ERR_WORKSPACE;
  char* ws = (char*)workspace;
  int32_t* perm = (int32_t*)(ws + L.off_perm);
  uint64_t* keys = (uint64_t*)(ws + L.off_keys);
  int32_t* goff = (int32_t*)(ws + L.off_goff);
  int32_t* ng = (int32_t*)(ws + L.off_ng);
  uint32_t* blocks = (uint32_t*)(ws + L.off_blocks);
  int32_t* starts = (int32_t*)(ws + L.off_starts);
  // Three launches: for no more points than cells (beyond, single ranges, or a grid's few, have too much of the work: 500,000
  // points around the centre of 468 x 468 cells 93 us by the general path, 108 by this, 60,000 of 100 x 100 48 and 58; 180,000
  // and 5,000 of them 55 / 50 and 31 / 18), and where the tables fit into the memory of the sort that they replace, as they do
  // unless there are far fewer points than ranges.
  const int64_t grid_cells = (int64_t)g->num_frames * g->grid_x * g->grid_y, ranges = ceil_div(grid_cells, (int64_t)1 << kVoxCellBits);
  if (m > 0 && m <= grid_cells && ranges <= kVoxMaxRanges) {
    const int tiles = (int)ceil_div(m, (int64_t)kVoxTile);
    const int bins = (int)(ranges + 2) & ~1;  // (at least one more than ranges)
    int bin_bits = 1;
    while ((1 << bin_bits) < bins) ++bin_bits;
    const size_t table_bytes = align_up((size_t)tiles * bins * 2, 256), range_bytes = align_up((size_t)ranges * 4, 256);
    if (table_bytes + 2 * range_bytes <= L.flat_bytes) {
      char* flat = ws + L.off_flat;
      uint32_t* table = (uint32_t*)flat;
      uint32_t* range_pillars = (uint32_t*)(flat + table_bytes);
      uint32_t* range_end = (uint32_t*)(flat + table_bytes + range_bytes);
      uint32_t* entries = (uint32_t*)perm;
      int32_t* order = (int32_t*)keys;
      uint32_t* cells = (uint32_t*)keys + m;
      const PointCells pts{xy, frame, g->num_frames, g->grid_x, g->grid_y, v->x_min, v->y_min, v->voxel_x, v->voxel_y};
      hipLaunchKernelGGL(k_vox_split, dim3((unsigned)tiles), dim3(kVoxThreads), (size_t)kVoxWaves * bins * 2, stream, pts, (int)m,
                         bins, bin_bits, entries, table, point_to_pillar);
      constexpr size_t order_lds = (size_t)(kVoxList + kVoxOrderWaves * (1 << kVoxCellBits) / 2 + (1 << kVoxCellBits) + 2 * kVoxMaxTiles + 1) * 4;
      static_assert(order_lds <= 65536 - 256, "");
      hipLaunchKernelGGL(k_vox_order, dim3((unsigned)ranges), dim3(kVoxOrderThreads), order_lds, stream, entries,
                         (const uint16_t*)table, tiles, bins, order, starts, cells, range_pillars, range_end);
      const int parts = ranges > kVoxManyRanges ? 4 : 16;
      hipLaunchKernelGGL(k_vox_mean, dim3((unsigned)(ranges * parts)), dim3(256), 0, stream, order, starts, cells,
                         range_pillars, range_end, (int)ranges, parts, g->grid_x, g->grid_y, pfeats, Cp, coords, feats, num_pillars,
                         point_to_pillar);
      return launch_status();
    }
  }
  // key generation computes the cells itself: no array of cells, no launch for it
  const PointCells pts{xy, frame, g->num_frames, g->grid_x, g->grid_y, v->x_min, v->y_min, v->voxel_x, v->voxel_y};
  st = flatten_launch_points(&pts, m, &L.geom, perm, goff, ng, keys, ws + L.off_flat, L.flat_bytes, stream);
  if (st != FF_OK) return st;
  int32_t* kept = ng + 1;  // number of points inside the grid (a spare word beside the sort's group count)
  hipLaunchKernelGGL(k_seg_count, dim3((unsigned)L.nb), dim3(256), 0, stream, keys, m, g->num_frames, blocks, kept);
  if (L.nb <= kSegDirectBlocks) {
    hipLaunchKernelGGL(k_seg_starts<false>, dim3((unsigned)L.nb), dim3(256), 0, stream, keys, perm, m, g->num_frames,
                       blocks, (int)L.nb, num_pillars, starts, kept, coords, point_to_pillar);
  } else {
    hipLaunchKernelGGL(k_seg_scan, dim3(1), dim3(1024), 0, stream, blocks, L.nb, num_pillars);
    hipLaunchKernelGGL(k_seg_starts<true>, dim3((unsigned)L.nb), dim3(256), 0, stream, keys, perm, m, g->num_frames,
                       blocks, (int)L.nb, num_pillars, starts, kept, coords, point_to_pillar);
  }
  int64_t mean_blocks = ceil_div(m > 0 ? m : 1, 16);  // a pillar per sixteen lanes; there are at most m pillars
  if (mean_blocks > 256 * 32) mean_blocks = 256 * 32;
  hipLaunchKernelGGL(k_seg_mean, dim3((unsigned)mean_blocks), dim3(256), 0, stream, perm, pfeats, Cp, num_pillars, starts,
                     kept, feats, point_to_pillar);
  return launch_status();
}

}  // namespace ff
