// Window-based sorting and equal-size grouping (paper Sec. 4.2.1, Eq. (1); Sec. 4.2.2 'Window
// Shift'; Sec. 4.3 'Reuse Sorting' is the caller keeping the result).
//
// Each pillar becomes ONE 64-bit word  (compact_key << idx_bits) | original_index, where the
// compact key packs the tuple fields (b, W_major, W_minor, L_major, L_minor) using only as many
// bits as the geometry needs.  An LSD radix sort over the compact-key bits is stable, so equal
// tuples keep ascending original index.  The word carries the index, so a pass moves 8 bytes per
// pillar each way.
//
// S sort configurations of the same cloud are sorted together, one grid row each.  Workgroups on
// different XCDs of this chip talk through memory (two microseconds and more per flag round trip),
// so no kernel waits for another workgroup: everything a pass needs is in memory when it starts.
//   * A table counts[pass][tile][digit] says how many words with that digit of that pass the tile
//     holds in the order the pass reads them.  Key generation writes the rows of the first pass
//     (plain stores) and zeroes the others; each pass adds, for every word it places, one to the
//     row of the tile the word lands in for the next pass.  Nothing has to be cleared beforehand.
//   * Clouds over ordinary geometries take no such passes at all: up to 24,576 pillars one launch (k_direct below), up to
//     4 million two (k_split and k_buckets).
//   * Small clouds otherwise (at most 128 tiles of 1024 words, see kSmallMaxTiles: launch and latency bound): digits of up to 10
//     bits, and a pass reads the whole table of its pass itself (column sums = global digit
//     starts, rows of earlier tiles = its own offsets): key generation + one launch per pass.
//   * Larger clouds (bandwidth bound): per-word atomics would dominate, so passes after the first
//     count their tiles in a kernel of their own, and a small scan kernel turns the table of a pass
//     into exclusive prefixes over the tiles plus per-digit totals.  Tiles of 1024, 2048 or 4096
//     words by cloud size, so that clouds of a few hundred thousand words still fill the chip.
//   * A tile ranks its words with per-wavefront ballot matching and LDS counters and scatters
//     through an LDS stage so that global writes come out in runs.
//   * The last pass writes perm, exported keys and group offsets itself when its digit contains
//     the whole frame field; otherwise two small output kernels run.
#include "common.h"
#include "pack_weights.h"
#include "sort_device.h"
#include <atomic>
#include <type_traits>

namespace ff {

namespace {

constexpr int kMaxSorts = 4;
// Small clouds: tiles of 1024 words, up to 128 of them.  Inside a block the tiles of all its sorts count, because every
// workgroup of a pass reads the tables of its sort: with four sorts and four layers behind them (C = 128, us, small path
// against scanned tables) 30,000 words 93.5 / 95.3, 40,000 122 / 115, 80,000 216 / 202, 130,000 283 / 256; two sorts and
// layers 80,000 words 122 / 116, 120,000 153 / 141 (C = 64: 70,000 84.5 / 75.7); three 45,000 95.8 / 90.9, 100,000 203 /
// 190.  A batch of sorts by itself is bound by its launches, of which the scanned path has twice as many (50,000 words in
// two frames, four sorts: 66 / 79), so it counts like a single sort (80,000 words 37 / 39, 120,000 46 / 48).
constexpr int kSmallKpt = 4, kSmallMaxTiles = 128;
constexpr int kLargeKpt = 16;                       // larger clouds: tiles of 4096 words
// In between, the tables are scanned by their own kernel as for larger clouds, but tiles of 4096 words
// would leave most compute units without a workgroup.  Tiles of 1024 words up to 256 K words, of 2048
// words up to 1.5 M (measured: 140 K words 63 -> 52 us, 400 K 68 -> 58, 1 M 73 -> 67, 1.5 M 80 -> 75;
// from 2 M words on the large tiles are ahead).
constexpr int kMidKptA = 4, kMidMaxTilesA = 256;
constexpr int kMidKptB = 8, kMidMaxTilesB = 768;
constexpr int kScanThreads = 1024;
// Shape of the column scan: digits per workgroup (its 1024 threads cut the rows into 1024 / digits runs) and rows a
// thread keeps in registers between its two sweeps.  It is a chain of latencies, so what counts is few rows per thread:
// 64 digits and 16 rows up to 256 tiles, 16 digits and 16 rows up to 1024, 16 digits and 64 rows up to 4096.  Before,
// 64 rows everywhere and 64 digits up to 1024 tiles: sorts of 240,000 / 480,000 / 960,000 / 3.84 M words took 52 / 59 /
// 69 / 115 us, now 49 / 51 / 63 / 110.
constexpr int kScanWide = 64, kScanNarrow = 16;
constexpr int kScanFewRows = 16, kScanManyRows = 64;
constexpr int kScanWideTiles = kScanThreads / kScanWide * kScanFewRows;
constexpr int kScanFewRowsTiles = kScanThreads / kScanNarrow * kScanFewRows;

struct KeyParams {
  int32_t B, win_x, win_y, win_z;       // win_z = 1 and stride = 3 for bird's-eye-view pillars
  int32_t sx, sy, sz;                   // shift added to x / y / z
  int32_t axis, stride;                 // stride: int32 per row of coords (3: b,x,y; 4: b,x,y,z)
  int32_t bits_b, bits_w1, bits_w2, bits_w3, bits_l1, bits_l2, bits_l3;  // w3 / l3: the z fields (0 bits in 2-D)
  int32_t key_bits, idx_bits;
};

struct Batch {
  KeyParams kp[kMaxSorts];
  int32_t* perm[kMaxSorts];
  int32_t* inv_perm[kMaxSorts];  // nullptr, or sorted position of every pillar (inverse of perm)
  int32_t* group_offsets[kMaxSorts];
  int32_t* num_groups[kMaxSorts];
  uint64_t* keys_sorted[kMaxSorts];
};

// Groups a frame of `count` pillars is cut into: ceil(count / G), or floor when short groups are dropped.
// (count + G - 1 would overflow for a G near the top of the int range.)
__device__ __forceinline__ uint32_t groups_of(uint32_t count, int G, int drop) {
  const uint32_t full = count / (uint32_t)G;
  return drop || full * (uint32_t)G == count ? full : full + 1u;
}

__device__ __forceinline__ uint32_t field_mask(int bits) { return bits >= 32 ? 0xffffffffu : ((1u << bits) - 1u); }

__device__ __forceinline__ uint32_t digit_rb(uint64_t word, int idx_bits, int key_bits, int pass, int rb) {
  const int lo = pass * rb;
  const int nb = key_bits - lo < rb ? key_bits - lo : rb;
  if (nb <= 0) return 0u;
  return (uint32_t)(word >> (idx_bits + lo)) & ((1u << nb) - 1u);
}

__device__ __forceinline__ uint64_t make_word_at(const int32_t* __restrict__ c, int64_t i, const KeyParams& kp);
__device__ __forceinline__ uint64_t make_word(const int32_t* __restrict__ coords, int64_t i, const KeyParams& kp) {
  return make_word_at(coords + (int64_t)kp.stride * i, i, kp);
}
__device__ __forceinline__ uint64_t make_word_at(const int32_t* __restrict__ c, int64_t i, const KeyParams& kp) {
  const uint32_t b = (uint32_t)c[0];
  const uint32_t X = (uint32_t)(c[1] + kp.sx);
  const uint32_t Y = (uint32_t)(c[2] + kp.sy);
  const uint32_t Wx = X / (uint32_t)kp.win_x, Lx = X - Wx * (uint32_t)kp.win_x;
  const uint32_t Wy = Y / (uint32_t)kp.win_y, Ly = Y - Wy * (uint32_t)kp.win_y;
  uint32_t Wz = 0u, Lz = 0u;
  if (kp.stride > 3) {  // uniform: pillars pay for no third division
    const uint32_t Z = (uint32_t)(c[3] + kp.sz);
    Wz = Z / (uint32_t)kp.win_z;
    Lz = Z - Wz * (uint32_t)kp.win_z;
  }
  const uint32_t w1 = kp.axis == 0 ? Wx : Wy, w2 = kp.axis == 0 ? Wy : Wx;
  const uint32_t l1 = kp.axis == 0 ? Lx : Ly, l2 = kp.axis == 0 ? Ly : Lx;
  // Fields are masked to their widths so that a coordinate outside the geometry can only
  // disturb the order, never another field's bits or any index computed from them.
  uint64_t k = b & field_mask(kp.bits_b);
  k = (k << kp.bits_w1) | (w1 & field_mask(kp.bits_w1));
  k = (k << kp.bits_w2) | (w2 & field_mask(kp.bits_w2));
  k = (k << kp.bits_w3) | (Wz & field_mask(kp.bits_w3));  // 3-D windows: z is the last window and the last local field
  k = (k << kp.bits_l1) | (l1 & field_mask(kp.bits_l1));
  k = (k << kp.bits_l2) | (l2 & field_mask(kp.bits_l2));
  k = (k << kp.bits_l3) | (Lz & field_mask(kp.bits_l3));
  return (k << kp.idx_bits) | (uint64_t)i;
}

__device__ __forceinline__ uint64_t exported_key(uint64_t k, const KeyParams& kp, uint32_t* frame) {
  k >>= kp.bits_l3;  // the exported format has no z fields (it is only produced for 2-D keys)
  const uint64_t l2 = k & field_mask(kp.bits_l2); k >>= kp.bits_l2;
  const uint64_t l1 = k & field_mask(kp.bits_l1); k >>= kp.bits_l1;
  k >>= kp.bits_w3;
  const uint64_t w2 = k & field_mask(kp.bits_w2); k >>= kp.bits_w2;
  const uint64_t w1 = k & field_mask(kp.bits_w1); k >>= kp.bits_w1;
  const uint64_t b = k & field_mask(kp.bits_b);
  *frame = (uint32_t)b;
  return (b << 48) | (w1 << 32) | (w2 << 16) | (l1 << 8) | l2;
}

// ---- A1: coords -> sortable words, plus the digit counts of the first pass ---------------------------
// counts [S][P][tiles][BINS]
// A sort kernel can take workgroups along that do not sort: they re-tile layer weights for the fused
// attention kernels (pack_weights.h), work that does not depend on the sort and would otherwise cost
// a launch of its own in front of the first layer.  Such a launch has a wider grid; the workgroups
// are numbered in dispatch order, the first tiles * sorts of them sort, the rest pack.
// (id: of 256 threads, of which this is thread t)
__device__ __forceinline__ void pack_tail(const PackJob& pack, int id, int t) {
  int layer = id / pack.blocks;
  t += (id - layer * pack.blocks) * 256;
  if (layer >= pack.layers) return;
  layer += pack.first;
  if (pack.mode == kPackF32) pack_weights_f32_thread(pack.pb, layer, t, pack.C, pack.F, pack.total_frags);
  else if (pack.mode == kPackF16) pack_weights_thread<true>(pack.pb, layer, t, pack.C, pack.F, pack.total_frags);
  else pack_weights_thread<false>(pack.pb, layer, t, pack.C, pack.F, pack.total_frags);
}

template <int RB, int KPT>
__global__ __launch_bounds__(kSortThreads) void k_keygen(const int32_t* __restrict__ coords, int64_t n, Batch bt, int P,
                                                          int64_t tiles, uint64_t* __restrict__ words,
                                                          uint32_t* __restrict__ counts, PackJob pack, PointCells pts) {
  constexpr int BINS = 1 << RB, TILE = kSortThreads * KPT;
  static_assert(kSortThreads == 256, "pack_tail counts in 256 threads");
  const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;  // dispatch order
  if (wg >= tiles * gridDim.y) {  // the same for the whole workgroup
    pack_tail(pack, (int)(wg - tiles * gridDim.y), (int)threadIdx.x);
    return;
  }
  __shared__ uint32_t h[BINS];
  const int s = (int)(wg / tiles), tid = threadIdx.x;
  const int64_t tile = wg % tiles;
  const KeyParams kp = bt.kp[s];
  for (int t = tid; t < BINS; t += kSortThreads) h[t] = 0u;
  __syncthreads();
#pragma unroll 4
  for (int r = 0; r < KPT; ++r) {
    const int64_t i = tile * TILE + r * kSortThreads + tid;
    if (i < n) {
      uint64_t word;
      if (pts.xy) {  // the same for every thread
        int32_t cell[4];
        point_cell(pts, i, cell);
        word = make_word_at(cell, i, kp);
      } else {
        word = make_word(coords, i, kp);
      }
      words[(int64_t)s * n + i] = word;
      atomicAdd(&h[digit_rb(word, kp.idx_bits, kp.key_bits, 0, RB)], 1u);
    }
  }
  __syncthreads();
  for (int p = 0; p < P; ++p) {
    const size_t base = (((size_t)s * P + p) * tiles + tile) * BINS;
    for (int t = tid; t < BINS; t += kSortThreads) counts[base + t] = p == 0 ? h[t] : 0u;
  }
}

// ---- digit counts of one pass, one table row per tile (larger clouds, passes after the first) ---------
template <int RB, int KPT>
__global__ __launch_bounds__(kSortThreads) void k_tile_counts(const uint64_t* __restrict__ in_all, int64_t n, Batch bt, int pass,
                                                               int P, int64_t tiles, uint32_t* __restrict__ counts) {
  constexpr int BINS = 1 << RB, TILE = kSortThreads * KPT;
  __shared__ uint32_t h[BINS];
  const int s = blockIdx.y, tid = threadIdx.x;
  const int64_t tile = blockIdx.x;
  const int idx_bits = bt.kp[s].idx_bits, key_bits = bt.kp[s].key_bits;
  const uint64_t* in = in_all + (int64_t)s * n;
  for (int t = tid; t < BINS; t += kSortThreads) h[t] = 0u;
  __syncthreads();
  uint64_t key[KPT];
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const int64_t i = tile * TILE + r * kSortThreads + tid;
    key[r] = i < n ? in[i] : ~0ull;
  }
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const int64_t i = tile * TILE + r * kSortThreads + tid;
    if (i < n) atomicAdd(&h[digit_rb(key[r], idx_bits, key_bits, pass, RB)], 1u);
  }
  __syncthreads();
  const size_t base = (((size_t)s * P + pass) * tiles + tile) * BINS;
  for (int t = tid; t < BINS; t += kSortThreads) counts[base + t] = h[t];
}

// ---- exclusive prefixes of a pass's table over the tiles, and the per-digit totals ------------------
// One workgroup per W digits (a strip of the table, W * 4 bytes of every row).  The rows are cut into
// 1024 / W runs, W lanes take one run.  Up to ROWS rows per run are loaded at once and stay in
// registers between the two sweeps.
template <int RB, int W, int ROWS>
__global__ __launch_bounds__(kScanThreads) void k_scan_cols(uint32_t* __restrict__ counts, uint32_t* __restrict__ totals,
                                                             int pass, int P, int64_t tiles) {
  constexpr int BINS = 1 << RB, RUNS = kScanThreads / W;
  __shared__ uint32_t part[RUNS][W];
  const int s = blockIdx.y, dl = threadIdx.x % W, c = threadIdx.x / W;
  const int d = blockIdx.x * W + dl;
  uint32_t* tab = counts + ((size_t)s * P + pass) * tiles * BINS + d;
  const int64_t per = (tiles + RUNS - 1) / RUNS;
  const int64_t r0 = c * per, r1 = r0 + per < tiles ? r0 + per : tiles;
  const bool fits = per <= ROWS;  // the same for every thread
  uint32_t v[ROWS];
  uint32_t sum = 0;
  if (fits) {
#pragma unroll
    for (int u = 0; u < ROWS; ++u) v[u] = r0 + u < r1 ? tab[(size_t)(r0 + u) * BINS] : 0u;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) sum += v[u];
  } else {
    for (int64_t r = r0; r < r1; r += 8) {
      uint32_t t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = r + u < r1 ? tab[(size_t)(r + u) * BINS] : 0u;
#pragma unroll
      for (int u = 0; u < 8; ++u) sum += t[u];
    }
  }
  part[c][dl] = sum;
  __syncthreads();
  uint32_t run = 0, total = 0;
#pragma unroll 8
  for (int i = 0; i < RUNS; ++i) {
    const uint32_t t = part[i][dl];
    if (i < c) run += t;
    total += t;
  }
  if (c == 0) totals[((size_t)s * P + pass) * BINS + d] = total;
  if (fits) {
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      if (r0 + u < r1) tab[(size_t)(r0 + u) * BINS] = run;
      run += v[u];
    }
  } else {
    for (int64_t r = r0; r < r1; r += 8) {
      uint32_t t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = r + u < r1 ? tab[(size_t)(r + u) * BINS] : 0u;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (r + u < r1) tab[(size_t)(r + u) * BINS] = run;
        run += t[u];
      }
    }
  }
}

// ---- A2: one radix pass ----------------------------------------------------------------------------
// SCANNED: the table row of this tile already holds the counts of earlier tiles and `totals` the
// per-digit totals (k_scan_cols ran); otherwise the workgroup adds the table up itself.
template <int RB, int KPT, bool FUSE, bool SCANNED>
__global__ __launch_bounds__(kSortThreads) void k_pass(const uint64_t* __restrict__ in_all, uint64_t* __restrict__ out_all,
                                                        int64_t n, Batch bt, int pass, int P, int64_t tiles, int G,
                                                        int drop, uint32_t* __restrict__ counts,
                                                        const uint32_t* __restrict__ totals, PackJob pack) {
  constexpr int BINS = 1 << RB, BPT = BINS / kSortThreads, WAVES = kSortThreads / 64, TILE = kSortThreads * KPT;
  static_assert(BPT == 1 || BPT == 2 || BPT == 4, "digits of 8, 9 or 10 bits");
  // LDS is what limits the workgroups per compute unit (4 with 9-bit digits and 4096 words: 40 KB), so
  // the two arrays are reused: wave_cnt holds the per-wavefront digit counters until the words are
  // staged, then the output tables (row 0: gbase, output position of a word = gbase[digit] + its stage
  // slot; row 1: gdig, first output position of a digit over the whole array; rows 2 and 3: the frame
  // table of the last pass).  stage holds the per-wavefront match tables (one 64-bit lane mask per
  // digit), then the scratch of the block scans, then the words in output order.
  __shared__ uint32_t wave_cnt[WAVES][BINS];
  __shared__ uint64_t stage[TILE > WAVES * BINS ? TILE : WAVES * BINS];
  static_assert(WAVES >= 4, "rows of wave_cnt are reused for four tables");
  uint32_t* wave_totals = reinterpret_cast<uint32_t*>(stage);
  uint32_t* gbase = &wave_cnt[0][0];
  uint32_t* gdig = &wave_cnt[1][0];

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;  // dispatch order
  if (wg >= tiles * gridDim.y) {  // the same for the whole workgroup
    pack_tail(pack, (int)(wg - tiles * gridDim.y), (int)threadIdx.x);
    return;
  }
  const int s = (int)(wg / tiles);
  const int64_t tile = wg % tiles;
  const KeyParams kp = bt.kp[s];
  const int idx_bits = kp.idx_bits, key_bits = kp.key_bits;
  const uint64_t* in = in_all + (int64_t)s * n;
  uint64_t* out = out_all + (int64_t)s * n;
  const uint32_t* cnt_tab = counts + ((size_t)s * P + pass) * tiles * BINS;
  uint32_t* next_tab = counts + ((size_t)s * P + pass + 1) * tiles * BINS;
  const int64_t tile_start = tile * TILE;
  const int tile_count = (int)((n - tile_start) < (int64_t)TILE ? (n - tile_start) : (int64_t)TILE);
  // Element order inside the tile: wave-major, then round, then lane.  Each wave owns a contiguous
  // run of 64 * KPT words, so stability only needs (wave, round, lane) order.
  uint64_t key[KPT];
  uint32_t rank[KPT];
  const uint64_t lanes_below = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const int e = w * 64 * KPT + r * 64 + lane;
    key[r] = e < tile_count ? in[tile_start + e] : ~0ull;
  }

  // Thread t owns digits t * BPT ..: their counts over the whole array and over earlier tiles.
  uint32_t gtot[BPT], before[BPT];
  if (SCANNED) {
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
      gtot[k] = totals[((size_t)s * P + pass) * BINS + tid * BPT + k];
      before[k] = cnt_tab[(size_t)tile * BINS + tid * BPT + k];
    }
  } else {  // column sums, 32 rows per memory round trip
#pragma unroll
    for (int k = 0; k < BPT; ++k) { gtot[k] = 0; before[k] = 0; }
    for (int t0 = 0; t0 < tiles; t0 += 32) {
      uint32_t v[32][BPT];
#pragma unroll
      for (int u = 0; u < 32; ++u) {
        const int64_t t = t0 + u < tiles ? t0 + u : tiles - 1;
        if (BPT == 4) {
          const uint4 q = *reinterpret_cast<const uint4*>(cnt_tab + (size_t)t * BINS + tid * 4);
          v[u][0] = q.x; v[u][1 % BPT] = q.y; v[u][2 % BPT] = q.z; v[u][3 % BPT] = q.w;
        } else if (BPT == 2) {
          const uint2 q = *reinterpret_cast<const uint2*>(cnt_tab + (size_t)t * BINS + tid * 2);
          v[u][0] = q.x; v[u][1 % BPT] = q.y;
        } else {
          v[u][0] = cnt_tab[(size_t)t * BINS + tid];
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // all 32 in flight before the first is added
#pragma unroll
      for (int u = 0; u < 32; ++u)
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
          if (t0 + u < tiles) gtot[k] += v[u][k];
          if (t0 + u < tile) before[k] += v[u][k];
        }
    }
  }
#pragma unroll
  for (int i = 0; i < WAVES; ++i)
#pragma unroll
    for (int k = 0; k < BPT; ++k) { wave_cnt[i][tid + k * kSortThreads] = 0; stage[i * BINS + tid + k * kSortThreads] = 0ull; }
  __syncthreads();
  // Rank inside the wavefront's run: lanes with the same digit find each other through the match
  // table (every lane ORs its bit into the digit's entry; LDS instructions of a wavefront execute in
  // order, so the read that follows sees all of them), the first of them adds the count to the
  // wavefront's running digit counter and clears the entry for the next round.
  unsigned long long* match = reinterpret_cast<unsigned long long*>(stage) + w * BINS;
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const int e = w * 64 * KPT + r * 64 + lane;
    const bool valid = e < tile_count;
    const uint32_t d = digit_rb(key[r], idx_bits, key_bits, pass, RB);
    unsigned long long same = 0ull;
    uint32_t prev = 0;
    if (valid) atomicOr(&match[d], 1ull << lane);
    if (valid) { same = match[d]; prev = wave_cnt[w][d]; }
    const uint32_t below = __popcll(same & lanes_below);
    const uint32_t cnt = __popcll(same);
    if (valid && below == 0) { wave_cnt[w][d] = prev + cnt; match[d] = 0ull; }
    rank[r] = prev + below;
  }
  __syncthreads();

  uint32_t total[BPT];
  uint32_t tsum = 0, gsum = 0;
#pragma unroll
  for (int k = 0; k < BPT; ++k) {
    const int d = tid * BPT + k;
    uint32_t run = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
      const uint32_t c = wave_cnt[i][d];
      wave_cnt[i][d] = run;  // exclusive prefix over the tile's waves
      run += c;
    }
    total[k] = run;
    tsum += run;
    gsum += gtot[k];
  }
  const uint32_t gex = block_exclusive_scan<kSortThreads>(gsum, wave_totals, nullptr);
  const uint32_t tex = block_exclusive_scan<kSortThreads>(tsum, wave_totals, nullptr);
  uint32_t gb[BPT], gd[BPT];
  {
    uint32_t grun = gex, trun = tex;
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
      const int d = tid * BPT + k;
      gb[k] = grun + before[k] - trun;
      gd[k] = grun;
#pragma unroll
      for (int i = 0; i < WAVES; ++i) wave_cnt[i][d] += trun;  // first stage slot of (wave, digit)
      trun += total[k];
      grun += gtot[k];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const int e = w * 64 * KPT + r * 64 + lane;
    if (e < tile_count) {
      const uint32_t d = digit_rb(key[r], idx_bits, key_bits, pass, RB);
      stage[wave_cnt[w][d] + rank[r]] = key[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < BPT; ++k) {
    gbase[tid * BPT + k] = gb[k];
    if (FUSE) gdig[tid * BPT + k] = gd[k];
  }
  __syncthreads();

  if (!FUSE) {
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
      const int j = r * kSortThreads + tid;
      uint32_t slot = 0xffffffffu;  // table entry of the next pass this word counts for (none: no word here)
      if (j < tile_count) {
        const uint64_t k = stage[j];
        const uint32_t d = digit_rb(k, idx_bits, key_bits, pass, RB);
        const int64_t pos = (int64_t)(gbase[d] + (uint32_t)j);
        if (pos < n) {
          out[pos] = k;
          if (!SCANNED && pass + 1 < P)  // small clouds: the next pass finds this word in tile pos / TILE
            slot = (uint32_t)(pos / TILE) * BINS + digit_rb(k, idx_bits, key_bits, pass + 1, RB);
        }
      }
      if (!SCANNED && pass + 1 < P) {
        // One atomic per run of neighbouring lanes that count the same table entry.  Words next to each other in
        // the stage share this pass's digit and land side by side; when the cloud arrives in an order that
        // follows the grid (a voxeliser's row-major output) they mostly share the next digit as well, and
        // one atomic per word then queues up on a few addresses.
        const uint32_t prev = __shfl_up(slot, 1, 64);
        const bool head = lane == 0 || prev != slot;
        const uint64_t heads = __ballot(head);
        if (head && slot != 0xffffffffu) {
          const uint64_t later = lane == 63 ? 0ull : (heads >> (lane + 1));
          const uint32_t run = later ? (uint32_t)__builtin_ctzll(later) + 1u : 64u - (uint32_t)lane;
          atomicAdd(&next_tab[slot], run);
        }
      }
    }
    return;
  }

  // ---- last pass: the output position is final -------------------------------------------------------
  int32_t* __restrict__ const perm_s = bt.perm[s];  // read once: the stores below must not wait for them
  int32_t* __restrict__ const inv_s = bt.inv_perm[s];
  uint64_t* __restrict__ const keys_s = bt.keys_sorted[s];
  int32_t* __restrict__ const goff_s = bt.group_offsets[s];
  const uint32_t idx_mask = idx_bits >= 32 ? ~0u : (1u << idx_bits) - 1u;  // n < 2^31
  uint32_t pos_r[KPT], idx_r[KPT];
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const int j = r * kSortThreads + tid;
    const uint64_t word = stage[j < tile_count ? j : 0];
    const uint32_t d = digit_rb(word, idx_bits, key_bits, pass, RB);
    pos_r[r] = j < tile_count ? gbase[d] + (uint32_t)j : 0xffffffffu;
    idx_r[r] = (uint32_t)word & idx_mask;
  }
#pragma unroll
  for (int r = 0; r < KPT; ++r)
    if ((int64_t)pos_r[r] < n) perm_s[pos_r[r]] = (int32_t)idx_r[r];
  if (inv_s) {  // the same for the whole workgroup
#pragma unroll
    for (int r = 0; r < KPT; ++r)
      if ((int64_t)pos_r[r] < n) inv_s[idx_r[r]] = (int32_t)pos_r[r];
  }
  if (keys_s) {  // the same for the whole workgroup
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
      if ((int64_t)pos_r[r] < n) {
        uint32_t b;
        keys_s[pos_r[r]] = exported_key(stage[r * kSortThreads + tid] >> idx_bits, kp, &b);
      }
    }
  }
  // Frame b starts where the first last-pass digit of frame b starts; group bases are the running
  // sum of the frames' group counts, ceil(frame size / G), or floor when short groups are dropped.
  // The group list follows from that table alone: every workgroup builds the table and writes its
  // share of the list.
  __syncthreads();  // the stage has been read: its memory serves the block scan again
  uint32_t* fstart = &wave_cnt[2][0];
  uint32_t* fgroup = &wave_cnt[3][0];
  const int B = kp.B;
  const int nb_last = key_bits - pass * RB;       // bits of this digit (>= bits_b, checked by the host)
  const int fshift = nb_last - kp.bits_b;
  uint32_t gcount[BPT], fs[BPT], gs = 0;
#pragma unroll
  for (int k = 0; k < BPT; ++k) {
    const int b = tid * BPT + k;
    uint32_t c = 0, lo = 0;
    if (b < B) {
      lo = gdig[(uint32_t)b << fshift];
      const uint32_t hi = b + 1 < B ? gdig[(uint32_t)(b + 1) << fshift] : (uint32_t)n;
      c = groups_of(hi - lo, G, drop);
    }
    gcount[k] = c;
    fs[k] = lo;
    gs += c;
  }
  uint32_t ng_total = 0;
  uint32_t gexcl = block_exclusive_scan<kSortThreads>(gs, wave_totals, &ng_total);
#pragma unroll
  for (int k = 0; k < BPT; ++k) {
    const int b = tid * BPT + k;
    if (b < B) { fstart[b] = fs[k]; fgroup[b] = gexcl; }
    gexcl += gcount[k];
  }
  __syncthreads();
  for (int64_t gi = tile * kSortThreads + tid; gi < (int64_t)ng_total; gi += tiles * kSortThreads) {
    int lo = 0, hi = B;  // the last frame whose group base is at or below gi (empty frames share a base)
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (fgroup[mid] <= (uint32_t)gi) lo = mid; else hi = mid;
    }
    goff_s[gi] = (int32_t)(fstart[lo] + ((uint32_t)gi - fgroup[lo]) * (uint32_t)G);
  }
  if (tile == 0 && tid == 0) {
    *bt.num_groups[s] = (int32_t)ng_total;
    goff_s[ng_total] = (int32_t)n;
  }
}

// ---- A3: frame boundaries and group bases for many frames (num_frames > 256) ---------------------
__global__ __launch_bounds__(256) void k_frames(const uint64_t* __restrict__ sorted_all, int64_t n, Batch bt, int G,
                                                 int drop, int32_t* __restrict__ frame_tab /*[S][2][B+1]*/) {
  __shared__ uint32_t wave_totals[4];
  __shared__ uint32_t carry_s;
  const int s = blockIdx.x;
  const KeyParams kp = bt.kp[s];
  const int B = kp.B;
  const uint64_t* sorted = sorted_all + (int64_t)s * n;
  int32_t* frame_start = frame_tab + (int64_t)s * 2 * (B + 1);
  int32_t* group_base = frame_start + (B + 1);
  const int frame_shift = kp.idx_bits + kp.key_bits - kp.bits_b;
  const int tid = threadIdx.x;
  for (int b = tid; b <= B; b += 256) {
    int64_t lo = 0, hi = n;  // first position whose frame field is >= b
    if (b == B) lo = n;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      const uint32_t f = (uint32_t)(sorted[mid] >> frame_shift);
      if (f < (uint32_t)b) lo = mid + 1; else hi = mid;
    }
    frame_start[b] = (int32_t)lo;
  }
  if (tid == 0) carry_s = 0;
  __syncthreads();
  for (int base = 0; base < B; base += 256) {
    const int b = base + tid;
    uint32_t g = 0;
    if (b < B) g = groups_of((uint32_t)(frame_start[b + 1] - frame_start[b]), G, drop);
    uint32_t total;
    const uint32_t ex = block_exclusive_scan<256>(g, wave_totals, &total);
    const uint32_t carry = carry_s;
    if (b < B) group_base[b] = (int32_t)(carry + ex);
    __syncthreads();
    if (tid == 0) carry_s = carry + total;
    __syncthreads();
  }
  if (tid == 0) group_base[B] = (int32_t)carry_s;
}

// ---- outputs: perm, exported keys, group offsets, num_groups ----------------------------------------
// For a small cloud with at most 256 frames every block recomputes the frame table itself (B binary
// searches and one block scan); otherwise it reads the table k_frames wrote.
__global__ __launch_bounds__(256) void k_finalize(const uint64_t* __restrict__ sorted_all, int64_t n, Batch bt, int G,
                                                   int drop, const int32_t* __restrict__ frame_tab) {
  __shared__ int32_t fstart_s[257], gbase_s[257];
  __shared__ uint32_t wave_totals[4];
  const int s = blockIdx.y;
  const KeyParams kp = bt.kp[s];
  const int B = kp.B, tid = threadIdx.x;
  const uint64_t* sorted = sorted_all + (int64_t)s * n;
  const int frame_shift = kp.idx_bits + kp.key_bits - kp.bits_b;
  const int32_t* fstart = fstart_s;
  const int32_t* gbase = gbase_s;
  if (B == 1) {
    if (tid == 0) { fstart_s[0] = 0; fstart_s[1] = (int32_t)n; gbase_s[0] = 0; gbase_s[1] = (int32_t)groups_of((uint32_t)n, G, drop); }
    __syncthreads();
  } else if (B <= 256 && n <= 65536) {
    if (tid == 0) fstart_s[B] = (int32_t)n;
    if (tid < B) {
      int64_t lo = 0, hi = n;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        const uint32_t f = (uint32_t)(sorted[mid] >> frame_shift);
        if (f < (uint32_t)tid) lo = mid + 1; else hi = mid;
      }
      fstart_s[tid] = (int32_t)lo;
    }
    __syncthreads();
    uint32_t g = 0;
    if (tid < B) g = groups_of((uint32_t)(fstart_s[tid + 1] - fstart_s[tid]), G, drop);
    uint32_t total;
    const uint32_t ex = block_exclusive_scan<256>(g, wave_totals, &total);
    if (tid < B) gbase_s[tid] = (int32_t)ex;
    if (tid == 0) gbase_s[B] = (int32_t)total;
    __syncthreads();
  } else {
    fstart = frame_tab + (int64_t)s * 2 * (B + 1);
    gbase = fstart + (B + 1);
  }
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + tid;
  if (p == 0) {
    const int32_t ng = gbase[B];
    *bt.num_groups[s] = ng;
    bt.group_offsets[s][ng] = (int32_t)n;
  }
  if (p >= n) return;
  const uint64_t word = sorted[p];
  const uint64_t idx_mask = (1ull << kp.idx_bits) - 1ull;
  bt.perm[s][p] = (int32_t)(word & idx_mask);
  if (bt.inv_perm[s]) bt.inv_perm[s][word & idx_mask] = (int32_t)p;
  uint64_t k = word >> kp.idx_bits;
  k >>= kp.bits_l3;
  const uint64_t l2 = k & field_mask(kp.bits_l2); k >>= kp.bits_l2;
  const uint64_t l1 = k & field_mask(kp.bits_l1); k >>= kp.bits_l1;
  k >>= kp.bits_w3;
  const uint64_t w2 = k & field_mask(kp.bits_w2); k >>= kp.bits_w2;
  const uint64_t w1 = k & field_mask(kp.bits_w1); k >>= kp.bits_w1;
  const uint64_t b = k & field_mask(kp.bits_b);
  if (bt.keys_sorted[s]) bt.keys_sorted[s][p] = (b << 48) | (w1 << 32) | (w2 << 16) | (l1 << 8) | l2;
  const int fb = b < (uint64_t)B ? (int)b : B - 1;
  const int32_t rel = (int32_t)p - fstart[fb], gi = rel / G;
  if (rel == gi * G && gi < gbase[fb + 1] - gbase[fb]) bt.group_offsets[s][gbase[fb] + gi] = (int32_t)p;
}

// ---- small clouds in one launch ------------------------------------------------------------------------------------
// A workgroup owns a range of key values of one sort.  It looks at every pillar of the cloud, works out the key, counts the
// ones below its range (where its share of the output begins) and takes those inside: into a list, and as bits of a map with
// one bit per key value.  Prefix counts of the bits are the sorted positions: no digits, no passes, no other workgroup's
// results.  Fewer bits than pillars say that some share a cell: then the pillars are brought together by words of the map and
// ranked there, or, where there are many to a cell, counted by cell in the order in which they come.  Pillars that do not fit the
// lists are looked up in the cloud again.
//
// What bounds it: the look at all pillars, 12 bytes and some 20 vector instructions each in every workgroup, 0.23 us for
// every thousand of them, and 4 us for the launch, the scan and the way out; the radix path is three dependent launches of
// 5 to 12 us.  From a graph, without fills, radix path / this one, us: one sort, 2,000 pillars 17.6 / 4.8, 12,345 18.7 / 7.3, 24,576
// 18.9 / 9.6; four sorts, 2,000 18.9 / 4.9, 12,345 20.0 / 7.7, 24,576 21.9 / 10.2.  The line to the two launches of k_split was drawn
// when these took 2 to 3 us more (one sort and four as plain calls, 20,000 pillars of two frames 12.4 and 13.0 by this, 24 to 25 by
// those, 30,000 14.1 and 15.2 by this, 13.4 and 13.9 by those, 60,000 21.0 and 22.5, 14.6 and 16.4); from 18,000 on they are now
// up to 1 us ahead for clouds without crowds, and behind for crowds of few cells.
// Clouds whose pillars share a window's few cells, hundreds each, are one workgroup's, two more looks at the cloud: 20,000 on one,
// a hundred or a thousand cells 38, 44 and 49 us, radix path 20 to 26 (bitonic sorts of the lists: 106, 217, 130).
constexpr int kDirectThreads = 1024;
constexpr int kDirectWaves = kDirectThreads / 64;
constexpr int kDirectOwn = 1024;            // pillars of a range that a wavefront finds (4 bytes each),
constexpr int kDirectList = kDirectWaves * kDirectOwn;  // all together,
constexpr int kDirectShared = 8192;         // and when some share a cell and the wavefronts' lists have to be joined
constexpr int kDirectRanked = 256;          // pillars of 32 key values that are ranked by comparing them all
constexpr int kDirectMaxRows = 24576;       // pillars,
constexpr int kDirectCrowds = kDirectMaxRows / (kDirectRanked + 1);  // words that can have more
constexpr int kDirectDigits = 2 * (kDirectShared + kDirectList) / kDirectWaves;  // cells of a range that are counted at a time
static_assert(kDirectMaxRows <= kDirectShared + kDirectList && 32 * kDirectCrowds <= kDirectDigits && kDirectMaxRows < 1 << 16, "");
constexpr int kDirectMaxCodes = 131072;     // and key values of a workgroup's range; a list entry of 32 bits holds one of each
constexpr int kDirectMaxFrames = 16;
constexpr int kDirectMaxGrid = 4096;        // cells an axis, shift included: windows by a 24-bit multiplication

// How a sort makes its keys.  Window of a shifted coordinate X: w = (X * mul) >> 20, exact below 4096 for windows up to 256.
// With the local coordinate X - w win in its field, unit_l, and the window in its own, unit_w, an axis adds
// X unit_l + w (unit_w - win unit_l).
struct DirectAxis { int32_t shift; uint32_t max, mul, unit_l, rest_w; };  // max: largest shifted coordinate
struct DirectKeys { DirectAxis x, y, z; uint32_t unit_b; };
struct DirectBatch {
  DirectKeys k[kMaxSorts];
  uint32_t range;    // key values of a workgroup
  int32_t parts;     // workgroups of a sort
};

template <bool Z, bool FRAMES>
__device__ __forceinline__ uint32_t direct_key(const int32_t* c, const DirectKeys& k, uint32_t last_frame) {
  // A coordinate outside the geometry counts as the last cell: its key stays in range, whatever it is.
  auto axis = [](uint32_t key, int32_t v, const DirectAxis& a) -> uint32_t {
    const uint32_t at = (uint32_t)(v + a.shift), X = at < a.max ? at : a.max;
    return __umul24(__umul24(X, a.mul) >> 20, a.rest_w) + (__umul24(X, a.unit_l) + key);
  };
  uint32_t key = 0;
  if constexpr (FRAMES) {
    const uint32_t f = (uint32_t)c[0], b = f < last_frame ? f : last_frame;
    key = __umul24(b, k.unit_b);
  }
  key = axis(axis(key, c[1], k.x), c[2], k.y);
  if constexpr (Z) key = axis(key, c[3], k.z);
  return key;
}

// The group list of a sort from the frames' sizes alone, by one workgroup.
__device__ __forceinline__ void direct_groups(const int32_t* __restrict__ coords, int stride, int n, int B, int G, int drop,
                                              int32_t* __restrict__ goff, int32_t* __restrict__ num_groups,
                                              uint32_t* starts /*[kDirectMaxFrames]*/) {
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid < kDirectMaxFrames) starts[tid] = 0u;
  __syncthreads();
  if (B > 1) {
    uint32_t count = 0;                      // lane b: rows of frames below b that this wavefront has seen
    for (int i0 = 0; i0 < n; i0 += kDirectThreads * 8) {
      uint32_t f[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + u * kDirectThreads + tid;
        f[u] = i < n ? (uint32_t)coords[(uint32_t)(i * stride)] : ~0u;  // (nobody's, like ids outside, which count as the last frame)
      }
      for (int b = 1; b < B; ++b) {
        uint32_t c = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) c += (uint32_t)__popcll(__ballot(f[u] < (uint32_t)b));
        count += lane == b ? c : 0u;
      }
    }
    if (lane < B) atomicAdd(&starts[lane], count);
    __syncthreads();
  }
  uint32_t groups = 0;
  for (int b = 0; b < B; ++b) {
    const uint32_t from = starts[b], to = b + 1 < B ? starts[b + 1] : (uint32_t)n;
    const uint32_t g = groups_of(to - from, G, drop);
    for (uint32_t k = tid; k < g; k += kDirectThreads) goff[groups + k] = (int32_t)(from + k * (uint32_t)G);
    groups += g;
  }
  if (tid == 0) {
    *num_groups = (int32_t)groups;
    goff[groups] = n;
  }
}

// Position of v among a[q0 .. q1) in ascending order, counted from a[0].
__device__ __forceinline__ uint32_t rank_in_run(const uint32_t* a, uint32_t q0, uint32_t q1, uint32_t v) {
  uint32_t pos = q0, q = q0;
  for (; q + 4u <= q1; q += 4u) {
    const uint32_t x0 = a[q], x1 = a[q + 1u], x2 = a[q + 2u], x3 = a[q + 3u];
    pos += (x0 < v ? 1u : 0u) + (x1 < v ? 1u : 0u) + (x2 < v ? 1u : 0u) + (x3 < v ? 1u : 0u);
  }
  for (; q < q1; ++q) pos += a[q] < v ? 1u : 0u;
  return pos;
}

// a[0 .. T) in ascending order; a has room for the next power of two.  Pairs up to 64 apart stay within the 128 entries of a
// wavefront, whose LDS accesses are in order.
template <int THREADS>
__device__ __forceinline__ void direct_sort(uint32_t* a, uint32_t T) {
  uint32_t P = 128;
  while (P < T) P <<= 1;
  for (uint32_t e = T + threadIdx.x; e < P; e += THREADS) a[e] = 0xffffffffu;
  __syncthreads();
  for (uint32_t k = 2; k <= P; k <<= 1) {
    for (uint32_t j = k >> 1; j > 0; j >>= 1) {
      for (uint32_t t = threadIdx.x; t < P / 2; t += THREADS) {
        const uint32_t i = 2u * t - (t & (j - 1u)), x = a[i], y = a[i + j];
        if ((x > y) == ((i & k) == 0u)) { a[i] = y; a[i + j] = x; }
      }
      if (j > 64u) __syncthreads();
      else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (k > 64u) __syncthreads();            // (the next step pairs further than 64 apart)
  }
}

template <bool Z, bool FRAMES>
__global__ __launch_bounds__(kDirectThreads, 4) void k_direct(const int32_t* __restrict__ coords, int n, int S, int parts,
                                                               uint32_t range, int G, int drop, Batch bt, DirectBatch db,
                                                               PackJob pack) {
  constexpr int STRIDE = Z ? 4 : 3, ROWS = 4;  // rows of a thread in a round; the next round's are on their way meanwhile
  constexpr int ROUND = kDirectThreads * ROWS;
  __shared__ uint32_t wave_totals[kDirectWaves], starts[kDirectMaxFrames], crowd_start[kDirectCrowds];
  __shared__ uint32_t taken, below, full;
  extern __shared__ uint32_t bits[];                            // [range / 32]
  uint32_t* const first = bits + range / 32;                    // [range / 32] position of a word's first pillar
  uint32_t* const joined = first + range / 32;                  // [kDirectShared], or with the next kDirectMaxRows: pillars by word
  uint32_t* const list = joined + kDirectShared;                // [kDirectList] those of each wavefront: (key - lo) << idx_bits | index
  const int tid = threadIdx.x, lane = tid & 63;
  if ((int)blockIdx.x >= S * (parts + 1)) {
    pack_tail(pack, ((int)blockIdx.x - S * (parts + 1)) * (kDirectThreads / 256) + (tid >> 8), tid & 255);
    return;
  }
  if ((int)blockIdx.x >= S * parts) {
    const int s = blockIdx.x - S * parts;
    direct_groups(coords, STRIDE, n, bt.kp[s].B, G, drop, bt.group_offsets[s], bt.num_groups[s], starts);
    return;
  }

  const int s = blockIdx.x % S, part = blockIdx.x / S;
  const DirectKeys dk = db.k[s];
  const int idx_bits = bt.kp[s].idx_bits;
  const uint32_t idx_mask = (1u << idx_bits) - 1u;
  const uint32_t last_frame = (uint32_t)bt.kp[s].B - 1u, end = 1u << bt.kp[s].key_bits;
  const uint32_t lo = (uint32_t)part * range;
  if (lo >= end) return;
  const uint32_t hi = end - lo < range ? end : lo + range;
  int32_t* __restrict__ const perm_s = bt.perm[s];
  int32_t* __restrict__ const inv_s = bt.inv_perm[s];
  uint64_t* __restrict__ const keys_s = bt.keys_sorted[s];
  // (The looks at a cloud that changes under the call do not agree: no position is written that is none.)
  auto put = [&](uint32_t pos, uint32_t key, uint32_t i) {
    if (pos >= (uint32_t)n) return;
    perm_s[pos] = (int32_t)i;
    if (inv_s) inv_s[i] = (int32_t)pos;
    if (keys_s) {
      uint32_t b;
      keys_s[pos] = exported_key(key, bt.kp[s], &b);
    }
  };
  struct Row { int32_t c[STRIDE]; };
  auto fetch = [&](Row (&r)[ROWS], int i0) {
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int i = i0 + u * kDirectThreads + tid;
      const uint32_t at = __umul24((uint32_t)(i < n ? i : n - 1), (uint32_t)sizeof(Row));
      r[u] = *reinterpret_cast<const Row*>(reinterpret_cast<const char*>(coords) + at);
    }
  };
  const int wave = tid >> 6;
  uint32_t* const mine = list + wave * kDirectOwn;
  const uint32_t len = hi - lo, words = (len + 31u) >> 5;
  uint32_t less = 0, count = 0;              // count: of the wavefront
  {
    Row r[2][ROWS];
    int begin = 0;
    asm volatile("" : "+s"(begin));            // (or the addresses of the first round would be kept through everything that follows)
    fetch(r[0], begin);
    for (uint32_t w = tid; w < words; w += kDirectThreads) bits[w] = 0u;
    if (tid == 0) { taken = 0u; below = 0u; full = 0u; }
    __syncthreads();
    auto look = [&](Row (&now)[ROWS], int i0, auto whole) {
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        uint32_t key = direct_key<Z, FRAMES>(now[u].c, dk, last_frame);
        asm volatile("" : "+v"(key));          // (computed by every lane: under a condition its load would be waited for alone)
        const uint32_t i = (uint32_t)(i0 + u * kDirectThreads + tid);
        if (!decltype(whole)::value) key = i < (uint32_t)n ? key : 0xffffffffu;
        less += key < lo ? 1u : 0u;
        const uint32_t code = key - lo;
        const uint64_t in = __ballot(code < len);
        if (code < len) {
          const uint32_t at = count + lanes_below(in);
          if (at < (uint32_t)kDirectOwn) mine[at] = (code << idx_bits) | i;
          atomicOr(&bits[code >> 5], 1u << (code & 31u));
        }
        count += (uint32_t)__popcll(in);
      }
    };
    int i0 = begin;
    for (; i0 + 2 * ROUND <= n; i0 += 2 * ROUND) {
      fetch(r[1], i0 + ROUND);
      look(r[0], i0, std::true_type());
      fetch(r[0], i0 + 2 * ROUND);
      look(r[1], i0 + ROUND, std::true_type());
    }
    if (i0 + ROUND < n) {
      fetch(r[1], i0 + ROUND);
      look(r[0], i0, std::true_type());
      look(r[1], i0 + ROUND, std::false_type());
    } else if (i0 < n) {
      look(r[0], i0, std::false_type());
    }
  }
  less = wave_inclusive_scan(less);
  if (lane == 63) atomicAdd(&below, less);
  if (lane == 0) {
    atomicAdd(&taken, count);
    if (count > (uint32_t)kDirectOwn) full = 1u;
  }
  __syncthreads();
  const uint32_t T = taken, base = below;
  const uint32_t per = (words + kDirectThreads - 1u) / kDirectThreads, w0 = tid * per;
  uint32_t sum = 0, cells;
  for (uint32_t w = w0; w < w0 + per && w < words; ++w) sum += (uint32_t)__popc(bits[w]);
  uint32_t run = block_exclusive_scan<kDirectThreads>(sum, wave_totals, &cells);
  const bool plain = cells == T;             // no two pillars share a cell
  // The range's pillars once more, in no order: use(key - lo, index).  From the lists where all are in them, and nothing else is
  // to be written there.
  const bool listed = !full && (plain || T <= (uint32_t)kDirectShared);
  auto each = [&](auto use) {
    if (listed) {
      for (uint32_t e = lane; e < count; e += 64) use(mine[e] >> idx_bits, mine[e] & idx_mask);
      return;
    }
    for (int i0 = 0; i0 < n; i0 += ROUND) {
      Row r[ROWS];
      fetch(r, i0);
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        const int i = i0 + u * kDirectThreads + tid;
        const uint32_t code = direct_key<Z, FRAMES>(r[u].c, dk, last_frame) - lo;
        if (i < n && code < len) use(code, (uint32_t)i);
      }
    }
  };
  if (plain) {
    for (uint32_t w = w0; w < w0 + per && w < words; ++w) {
      first[w] = run;
      run += (uint32_t)__popc(bits[w]);
    }
    __syncthreads();
    each([&](uint32_t code, uint32_t i) {
      const uint32_t w = code >> 5;
      put(base + first[w] + (uint32_t)__popc(bits[w] & ((1u << (code & 31u)) - 1u)), lo + code, i);
    });
    return;
  }
  // Some share a cell.  Pillars of few cells that do not fit the lists, or of crowded words of the map, are counted by cell, in two
  // looks at the cloud of which wavefronts take consecutive pieces.
  int digit_bits = 0;
  auto in_order = [&](uint16_t* counts, auto digit, auto use) {  // digit: of a key value of the range, -1 if it is not counted
    const int piece = (n + kDirectThreads - 1) / kDirectThreads * 64, from = wave * piece, to = from + piece < n ? from + piece : n;
    Row r[2][ROWS];
    auto bring = [&](Row (&r)[ROWS], int i0) {
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        const int i = i0 + u * 64 + lane;
        r[u] = *reinterpret_cast<const Row*>(coords + (uint32_t)(i < n ? i : n - 1) * STRIDE);
      }
    };
    auto rank = [&](Row (&r)[ROWS], int i0) {
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        const int i = i0 + u * 64 + lane;
        const uint32_t code = direct_key<Z, FRAMES>(r[u].c, dk, last_frame) - lo;
        const int d = i < to && code < len ? digit(code) : -1;
        const uint32_t pos = rank_in_wave(counts, d < 0 ? 0u : (uint32_t)d, digit_bits, d >= 0);
        if (d >= 0) use(pos, code, (uint32_t)i);
      }
    };
    if (from < to) bring(r[0], from);
    for (int i0 = from; i0 < to; i0 += 2 * 64 * ROWS) {
      bring(r[1], i0 + 64 * ROWS);
      rank(r[0], i0);
      bring(r[0], i0 + 2 * 64 * ROWS);
      if (i0 + 64 * ROWS < to) rank(r[1], i0 + 64 * ROWS);
    }
  };
  // half: counts of a wavefront, two in a word.  start: where the first of words p's digits go, given how many there are
  auto count_and_put = [&](uint32_t half, auto digit, auto start) {
    uint16_t* const counts = reinterpret_cast<uint16_t*>(joined + wave * half);
    __syncthreads();
    for (uint32_t w = tid; w < kDirectWaves * half; w += kDirectThreads) joined[w] = 0u;
    __syncthreads();
    in_order(counts, digit, [](uint32_t, uint32_t, uint32_t) {});
    __syncthreads();
    for (uint32_t p0 = 0; p0 < half; p0 += kDirectThreads) {
      const uint32_t p = p0 + tid;
      const uint32_t total = p < half ? sum_over_waves<kDirectWaves>(joined, (int)half, (int)p) : 0u;
      const uint32_t at = start(p, (total & 0xffffu) + (total >> 16)), both = at | (at + (total & 0xffffu)) << 16;
      if (p < half)
#pragma unroll
        for (int w = 0; w < kDirectWaves; ++w) joined[w * half + p] += both;
    }
    __syncthreads();
    in_order(counts, digit, [&](uint32_t pos, uint32_t code, uint32_t i) { put(base + pos, lo + code, i); });
  };
  auto by_cell = [&] {
    for (uint32_t w = w0, at = run; w < w0 + per && w < words; ++w) {
      first[w] = at;
      at += (uint32_t)__popc(bits[w]);
    }
    while (1u << digit_bits < cells) ++digit_bits;
    uint32_t carry = 0;
    count_and_put((cells + 1u) / 2u, [&](uint32_t code) { return (int)(first[code >> 5] + __popc(bits[code >> 5] & ((1u << (code & 31u)) - 1u))); },
                  [&](uint32_t, uint32_t both) {
      uint32_t all;
      const uint32_t at = carry + block_exclusive_scan<kDirectThreads>(both, wave_totals, &all);
      carry += all;
      return at;
    });
  };
  const bool few = cells <= (uint32_t)kDirectDigits;
  if (few && !listed) {
    by_cell();
    return;
  }
  // Otherwise they are brought together by words.  first: counts, then where a word's next pillar goes, in the end where the word
  // ends; of a crowded word its end and number.
  const uint32_t cells_before = run;
  for (uint32_t w = tid; w < words; w += kDirectThreads) first[w] = 0u;
  __syncthreads();
  each([&](uint32_t code, uint32_t) { atomicAdd(&first[code >> 5], 1u); });
  __syncthreads();
  sum = 0;                                   // pillars, and << 16 crowded words
  for (uint32_t w = w0; w < w0 + per && w < words; ++w) sum += first[w] + (first[w] > (uint32_t)kDirectRanked ? 1u << 16 : 0u);
  uint32_t crowds;
  run = block_exclusive_scan<kDirectThreads>(sum, wave_totals, &crowds);
  crowds >>= 16;
  if (few && crowds && T > (uint32_t)kDirectThreads) {
    run = cells_before;
    by_cell();
    return;
  }
  const bool sorted = T <= (uint32_t)kDirectThreads;  // so few that crowds are no matter: the list's entries are put in order as they are
  for (uint32_t w = w0; w < w0 + per && w < words; ++w) {
    const uint32_t c = first[w];
    if (c > (uint32_t)kDirectRanked && !sorted) {
      crowd_start[run >> 16] = run & 0xffffu;
      first[w] = 1u << 31 | (run + c);
      run += c + (1u << 16);
    } else {
      first[w] = run & 0xffffu;
      run += c;
    }
  }
  __syncthreads();
  each([&](uint32_t code, uint32_t i) {
    if (first[code >> 5] >> 31) return;
    const uint32_t at = atomicAdd(&first[code >> 5], 1u);
    if (at < T) joined[at] = code << idx_bits | i;
  });
  __syncthreads();
  if (crowds && sorted) {
    direct_sort<kDirectThreads>(joined, T);
    for (uint32_t e = tid; e < T; e += kDirectThreads) put(base + e, lo + (joined[e] >> idx_bits), joined[e] & idx_mask);
    return;
  }
  auto rank = [&](uint32_t code, uint32_t i) {  // every pillar looks at all of its word
    const uint32_t w = code >> 5, end = first[w];
    if (!(end >> 31)) put(base + rank_in_run(joined, w ? first[w - 1u] & 0xffffu : 0u, end, code << idx_bits | i), lo + code, i);
  };
  if (crowds == 0u) {
    for (uint32_t e = tid; e < T; e += kDirectThreads) rank(joined[e] >> idx_bits, joined[e] & idx_mask);
    return;
  }
  each(rank);
  digit_bits = 5;                            // 32 key values of each crowded word
  while ((1u << (digit_bits - 5)) < crowds) ++digit_bits;
  count_and_put(crowds * 16u, [&](uint32_t code) {
    const uint32_t v = first[code >> 5];
    return v >> 31 ? (int)((v >> 16 & 0x7fffu) * 32u + (code & 31u)) : -1;
  }, [&](uint32_t p, uint32_t both) {        // sixteen threads for a word
    uint32_t inc = both;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const uint32_t t = __shfl_up(inc, d, 16);
      if ((tid & 15) >= d) inc += t;
    }
    return crowd_start[p < crowds * 16u ? p >> 4 : 0u] + inc - both;
  });
}

// ---- large clouds in two launches --------------------------------------------------------------------------------------
// The high bits of the key, frame and windows, number the buckets, of 1024 pillars or more on average.  k_split sorts each tile
// of the cloud by bucket, in a place of its own, and says in a table where the buckets begin in it.  k_buckets, a workgroup per
// bucket, finds the bucket's pieces of all tiles through a column of the table, whose sums also say how many pillars lie in
// front, and puts its pillars in order as k_direct does: a bit for each key value, positions by counting bits.  Where some share
// a cell, the key values are sorted in LDS, with the position in the bucket behind them, which is in order of the index; more
// pillars than the list holds are counted by cell, or sorted in two passes through memory where the cells are many.
//
// What bounds it: for a hundred thousand pillars its two launches, 4 us and a chain of six or seven round trips each; for
// millions the lines touched rather than the 16 bytes a pillar moved: the pieces of a bucket are a few entries long where the
// frames are mixed, a line each of entries and table (3.84 M pillars: k_split 28 us, k_buckets 30).  The radix path moves 8-byte
// words through three passes there.  From a graph, without fills, radix path / this, us: one sort, 30,000 pillars 19.4 / 8.9,
// 131,073 29.3 / 10.1, 240,000 31.7 / 11.4, 960,000 53 / 23, 2 M 72 / 38, 3.84 M 102 / 57.7; four sorts, 30,000 22.8 / 9.5, 240,000
// 45.7 / 19.8, 960,000 107 / 50.6.  With a fifth of the pillars sharing cells 240,000 31.7 / 16.1; on one, a hundred and ten thousand
// cells of a corner, 30,000 64, 100 and 31, 131,072 239, 406 and 128, 960,000 1909, 3100 and 652 (20 to 47 by the radix path).
constexpr int kSplitThreads = 512, kSplitWaves = kSplitThreads / 64;
constexpr int kSplitLeast = 2, kSplitFew = 4, kSplitMany = 16;  // pillars of a thread of k_split: few to fill the chip, many to
constexpr int64_t kSplitFewRows = 1 << 19, kSplitManyRows = 1 << 20;  // keep the pieces long; of all sorts, and of one
constexpr int kSplitLocalBits = 13;         // pillars of a tile: up to 8192
constexpr int kSplitCodeBits = 16;          // key values of a bucket
constexpr int kSplitMaxBuckets = 3800;      // the counters of k_split: 61 KB
constexpr int kSplitMinRows = 16385;        // pillars
constexpr int kSplitRows = 448, kSplitRowsMany = 1408, kSplitBuckets = 1024;  // of a bucket on average, at least; the more when
                                            // all sorts together have this many buckets
constexpr int kSplitMaxTiles = 512;
constexpr int kSplitList = 4096;            // pillars of a bucket in registers, and of its list in LDS
constexpr int kSplitOwn = kSplitList / kSplitThreads;
constexpr int kSplitDigits = 9;             // cells of a bucket, in bits, that one pass sorts: counters in place of the list
static_assert(kSplitWaves << kSplitDigits == kSplitList && 1 << kSplitDigits <= kSplitThreads && kSplitCodeBits <= 16, "");

// Bucket of key k: h - (h >> in_frame) * skip with h = k >> code_bits, which leaves out the numbers no window has.
struct SplitSort { DirectKeys k; int32_t code_bits, in_frame, skip, per_frame; };
struct SplitBatch { SplitSort s[kMaxSorts]; int32_t bins, bin_bits, tiles; };

// (What the first loads need comes first: it is in registers when a wavefront starts.)
template <bool Z, bool FRAMES, int OWN>
__global__ __launch_bounds__(kSplitThreads) void k_split(const int32_t* __restrict__ coords, int n, int S, int tiles, int bins,
                                                          int bin_bits, int frames, uint32_t* __restrict__ entries_all,
                                                          uint32_t* __restrict__ table_all, uint16_t* __restrict__ frame_table,
                                                          SplitBatch sb, PackJob pack) {
  constexpr int STRIDE = Z ? 4 : 3, TILE = kSplitThreads * OWN;
  extern __shared__ uint32_t words[];        // [kSplitWaves][bins / 2]: counts of two buckets; then the tile, sorted
  __shared__ uint32_t wave_totals[kSplitWaves];
  const int tid = threadIdx.x, lane = tid & 63, half = bins >> 1;
  if ((int)blockIdx.x >= S * tiles) {
    pack_tail(pack, ((int)blockIdx.x - S * tiles) * (kSplitThreads / 256) + (tid >> 8), tid & 255);
    return;
  }
  const int s = blockIdx.x % S, tile = blockIdx.x / S, tile0 = tile * TILE, local0 = (tid >> 6) * 64 * OWN + lane;
  struct Row { int32_t c[STRIDE]; };
  Row r[OWN];
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int i = tile0 + local0 + u * 64;
    r[u] = *reinterpret_cast<const Row*>(coords + (int64_t)(i < n ? i : n - 1) * STRIDE);
  }
  const DirectKeys dk = sb.s[s].k;
  const int code_bits = sb.s[s].code_bits, in_frame = sb.s[s].in_frame;
  const uint32_t skip = (uint32_t)sb.s[s].skip, none = (uint32_t)bins - 1u, last_frame = (uint32_t)frames - 1u;
  uint16_t* const mine = reinterpret_cast<uint16_t*>(words + (tid >> 6) * half);
  for (int w = tid; w < kSplitWaves * half; w += kSplitThreads) words[w] = 0u;
  uint32_t entry[OWN], at[OWN];              // at: bucket << 16 | rank, then the position
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int i = tile0 + local0 + u * 64;
    const uint32_t key = direct_key<Z, FRAMES>(r[u].c, dk, last_frame), h = key >> code_bits;
    at[u] = i < n ? h - __umul24(h >> in_frame, skip) : none;
    entry[u] = (key & ((1u << code_bits) - 1u)) << kSplitLocalBits | (uint32_t)(local0 + u * 64);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < OWN; ++u) at[u] = at[u] << 16 | rank_in_wave(mine, at[u], bin_bits, true);
  __syncthreads();
  constexpr int PER = (kSplitMaxBuckets + 2) / 2 / kSplitThreads + 1;  // words of a thread
  const int per = (half + kSplitThreads - 1) / kSplitThreads, w0 = tid * per;
  uint32_t total[PER], sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    total[q] = q < per && w0 + q < half ? sum_over_waves<kSplitWaves>(words, half, w0 + q) : 0u;
    sum += (total[q] & 0xffffu) + (total[q] >> 16);
  }
  uint32_t first = block_exclusive_scan<kSplitThreads>(sum, wave_totals, nullptr);
  uint32_t* const table = table_all + ((int64_t)s * tiles + tile) * half;
#pragma unroll
  for (int q = 0; q < PER; ++q)
    if (q < per && w0 + q < half) {
      const uint32_t both = first | (first + (total[q] & 0xffffu)) << 16;
      table[w0 + q] = both;
#pragma unroll
      for (int w = 0; w < kSplitWaves; ++w) words[w * half + w0 + q] += both;
      first += (total[q] & 0xffffu) + (total[q] >> 16);
    }
  __syncthreads();
  if (FRAMES && frame_table) {               // where the frames begin, once more: a frame's tiles side by side
    const int tiles8 = (tiles + 7) & ~7, per_frame = sb.s[s].per_frame;
    for (int b = tid; b < frames; b += kSplitThreads)
      frame_table[((int64_t)s * frames + b) * tiles8 + tile] = reinterpret_cast<const uint16_t*>(words)[b * per_frame];
  }
#pragma unroll
  for (int u = 0; u < OWN; ++u) at[u] = mine[at[u] >> 16] + (at[u] & 0xffffu);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < OWN; ++u) words[at[u]] = entry[u];
  __syncthreads();
  uint32_t* const entries = entries_all + (int64_t)s * n + tile0;
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int e = u * kSplitThreads + tid;
    if (tile0 + e < n) entries[e] = words[e];
  }
}

// The group list of a sort, by one workgroup, from where the frames' first buckets begin in the tiles: in a table of their own if
// there is room for it (frame_table, a frame's tiles side by side).  From the columns of the large one it was what k_buckets
// ended with: 128 frames in 469 tiles are 60,000 lines, 49 us where the buckets took 30.  starts, groups: [frames + 1]
__device__ __forceinline__ void split_groups(const uint16_t* __restrict__ table, const uint16_t* __restrict__ frame_table, int tiles,
                                             int bins, int per_frame, int n, int B, int G, int drop, int32_t* __restrict__ goff,
                                             int32_t* __restrict__ num_groups, uint32_t* starts, uint32_t* groups,
                                             uint32_t* wave_totals) {
  const int tid = threadIdx.x, l = tid & 15, tiles8 = (tiles + 7) & ~7;
  for (int b = tid >> 4; b < B; b += kSplitThreads / 16) {
    uint32_t sum = 0;
    if (b == 0) {                            // (the first frame begins with the cloud)
    } else if (frame_table) {
      typedef uint16_t eight __attribute__((ext_vector_type(8)));
      static_assert(kSplitMaxTiles <= 4 * 16 * 8, "four a lane");
      eight v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (8 * (l + 16 * k) < tiles) v[k] = *reinterpret_cast<const eight*>(frame_table + (int64_t)b * tiles8 + 8 * (l + 16 * k));
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (8 * (l + 16 * k) + j < tiles) sum += v[k][j];
    } else {
#pragma unroll 8
      for (int t = l; t < tiles; t += 16) sum += table[(int64_t)t * bins + b * per_frame];
    }
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 16);
    if (l == 0) starts[b] = sum;
  }
  if (tid == 0) starts[B] = (uint32_t)n;
  __syncthreads();
  uint32_t carry = 0;
  for (int b0 = 0; b0 < B; b0 += kSplitThreads) {
    const int b = b0 + tid;
    const uint32_t g = b < B ? groups_of(starts[b + 1] - starts[b], G, drop) : 0u;
    uint32_t all;
    const uint32_t ex = block_exclusive_scan<kSplitThreads>(g, wave_totals, &all);
    if (b < B) groups[b] = carry + ex;
    carry += all;
  }
  if (tid == 0) {
    groups[B] = carry;
    *num_groups = (int32_t)carry;
    goff[carry] = n;
  }
  __syncthreads();
  const int lanes = B >= 32 ? 16 : B >= 8 ? 64 : kSplitThreads;  // of a frame
  for (int b = tid / lanes; b < B; b += kSplitThreads / lanes)
    for (uint32_t k = tid % lanes; k < groups[b + 1] - groups[b]; k += lanes) goff[groups[b] + k] = (int32_t)(starts[b] + k * (uint32_t)G);
}

// end0 .. end3: buckets of the first sort, of the first two, ..
__global__ __launch_bounds__(kSplitThreads, 6) void k_buckets(const uint16_t* __restrict__ table_all, int n, int S, int tiles, int bins,
                                                            int tile_rows, int end0, int end1, int end2, int end3,
                                                            const uint32_t* __restrict__ entries_all, uint32_t* scratch,
                                                            const uint16_t* __restrict__ frame_table, int G, int drop, Batch bt,
                                                            SplitBatch sb) {
  extern __shared__ uint32_t list[];                       // [kSplitList] key value << 12 | position in the bucket; counters
  uint32_t* const cum = list + kSplitList;                 // [kSplitMaxTiles + 1] the bucket's pillars in the tiles before,
  uint32_t* const from = cum + kSplitMaxTiles + 1;         // [kSplitMaxTiles] and where those of a tile are, less that
  uint32_t* const bits = from + kSplitMaxTiles;            // [words]
  __shared__ uint32_t wave_totals[2 * kSplitWaves];
  __shared__ uint32_t crowded;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x < S) {
    const int s = blockIdx.x;
    split_groups(table_all + (int64_t)s * tiles * bins,
                 frame_table ? frame_table + (int64_t)s * bt.kp[s].B * ((tiles + 7) & ~7) : nullptr, tiles, bins, sb.s[s].per_frame, n, bt.kp[s].B, G, drop,
                 bt.group_offsets[s], bt.num_groups[s], list, list + kSplitMaxBuckets + 1, wave_totals);
    return;
  }
  // Neighbouring buckets go to the same die, whose cache then has the lines that they share.
  const int id = blockIdx.x - S, each = (end3 + 7) >> 3, nth = (id & 7) * each + (id >> 3);
  if (nth >= end3) return;
  const int s = (nth >= end0 ? 1 : 0) + (nth >= end1 ? 1 : 0) + (nth >= end2 ? 1 : 0);
  const int bucket = nth - (s == 0 ? 0 : s == 1 ? end0 : s == 2 ? end1 : end2);
  const uint16_t* __restrict__ const table = table_all + (int64_t)s * tiles * bins;
  uint32_t lo = 0, hi = 0, T, base;
  if (tid < tiles) {
    lo = table[(int64_t)tid * bins + bucket];
    hi = table[(int64_t)tid * bins + bucket + 1];
  }
  const KeyParams kp = bt.kp[s];
  const int code_bits = sb.s[s].code_bits, words = 1 << (code_bits - 5);
  uint32_t* const first = bits + words;                    // [words] position of a word's first pillar
  const uint32_t* __restrict__ const entries = entries_all + (int64_t)s * n;
  for (int w = tid; w < words; w += kSplitThreads) bits[w] = 0u;
  const uint32_t before = block_exclusive_scan_and_sum<kSplitThreads>(hi - lo, lo, wave_totals, &T, &base);
  if (T == 0u) return;
  cum[tid] = tid < tiles ? before : T;                     // (kSplitThreads == kSplitMaxTiles)
  from[tid] = (uint32_t)tid * (uint32_t)tile_rows + lo - before;
  if (tid == 0) cum[kSplitMaxTiles] = T;
  __syncthreads();
  const uint32_t frame = (uint32_t)bucket / (uint32_t)sb.s[s].per_frame;
  const uint32_t key0 = ((uint32_t)bucket + frame * (uint32_t)sb.s[s].skip) << code_bits;
  int32_t* __restrict__ const perm_s = bt.perm[s];
  int32_t* __restrict__ const inv_s = bt.inv_perm[s];
  uint64_t* __restrict__ const keys_s = bt.keys_sorted[s];
  auto put_beside = [&](uint32_t pos, uint32_t code, uint32_t i) {  // (all but perm)
    if (inv_s) inv_s[i] = (int32_t)pos;
    if (keys_s) {
      uint32_t b;
      keys_s[pos] = exported_key(key0 + code, kp, &b);
    }
  };
  auto put = [&](uint32_t pos, uint32_t code, uint32_t i) {
    perm_s[pos] = (int32_t)i;
    put_beside(pos, code, i);
  };
  // Pillars of the bucket, OWN of a thread: key value and index of e0 + tid, e0 + tid + kSplitThreads, ..  The tile of one is
  // the last that begins no later.
  auto nth_of = [&](uint32_t e0, int u) {
    const uint32_t e = e0 + u * kSplitThreads + tid;
    return e < T ? e : T - 1u;
  };
  // (N a thread of the workgroup at most: with a branch around each of eight the reads of the search waited for each other, clocks
  // of a workgroup's fetch, 30,000 pillars 5,500 -> 2,000, 3.84 M 8,600 -> 4,000; k_buckets for four sorts of 30,000, 80,000 and
  // 240,000 9.2 -> 6.4, 13.2 -> 10.2 and 17.9 -> 13.8 us)
  uint32_t top = 1;                          // the largest power of two below the number of tiles
  while (2u * top < (uint32_t)tiles) top *= 2u;
  auto fetch_n = [&](uint32_t (&code)[kSplitOwn], uint32_t (&index)[kSplitOwn], uint32_t e0, auto n_of) {
    constexpr int N = decltype(n_of)::value;
    uint32_t tile[N] = {};
#pragma unroll 1
    for (uint32_t step = top; step > 0; step >>= 1) {
      uint32_t begins[N];
#pragma unroll
      for (int u = 0; u < N; ++u) begins[u] = cum[tile[u] + step];
#pragma unroll
      for (int u = 0; u < N; ++u) tile[u] += begins[u] <= nth_of(e0, u) ? step : 0u;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) index[u] = from[tile[u]];
#pragma unroll
    for (int u = 0; u < N; ++u) index[u] = entries[index[u] + nth_of(e0, u)];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      code[u] = index[u] >> kSplitLocalBits;
      index[u] = __umul24(tile[u], (uint32_t)tile_rows) + (index[u] & ((1u << kSplitLocalBits) - 1u));
    }
  };
  auto fetch = [&](uint32_t (&code)[kSplitOwn], uint32_t (&index)[kSplitOwn], uint32_t e0) {
    const uint32_t left = T - e0;
    if (left <= (uint32_t)kSplitThreads) fetch_n(code, index, e0, std::integral_constant<int, 1>());
    else if (left <= 2u * kSplitThreads) fetch_n(code, index, e0, std::integral_constant<int, 2>());
    else if (left <= 4u * kSplitThreads) fetch_n(code, index, e0, std::integral_constant<int, 4>());
    else                                 fetch_n(code, index, e0, std::integral_constant<int, kSplitOwn>());
  };
  auto each_of = [&](uint32_t e0, auto use) {
#pragma unroll
    for (int u = 0; u < kSplitOwn; ++u) {
      if (e0 + u * kSplitThreads >= T) break;  // (all of the workgroup)
      if (e0 + u * kSplitThreads + tid < T) use(u, e0 + u * kSplitThreads + tid);
    }
  };
  uint32_t code[kSplitOwn], index[kSplitOwn];
  for (uint32_t e0 = 0; e0 < T; e0 += kSplitList) {
    fetch(code, index, e0);
    each_of(e0, [&](int u, uint32_t) {       // (of many on a cell, all but the first would wait for each other in vain)
      if (e0 == 0u || !(bits[code[u] >> 5] >> (code[u] & 31u) & 1u)) atomicOr(&bits[code[u] >> 5], 1u << (code[u] & 31u));
    });
  }
  __syncthreads();
  constexpr int PER = (1 << (kSplitCodeBits - 5)) / kSplitThreads;  // words of a thread
  const int per = (words + kSplitThreads - 1) / kSplitThreads, w0 = tid * per;
  uint32_t pop[PER], sum = 0, cells;
#pragma unroll
  for (int q = 0; q < PER; ++q) pop[q] = q < per && w0 + q < words ? bits[w0 + q] : 0u;
#pragma unroll
  for (int q = 0; q < PER; ++q) sum += pop[q] = (uint32_t)__popc(pop[q]);
  uint32_t run = block_exclusive_scan<kSplitThreads>(sum, wave_totals, &cells);
  cells = (uint32_t)__builtin_amdgcn_readfirstlane((int)cells);  // (one path or another, never both: without scratch memory)
  if (cells == T) {                          // no two pillars share a cell
    uint32_t at = base + run;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if (q < per && w0 + q < words) first[w0 + q] = at;
      at += pop[q];
    }
    __syncthreads();
    if (T <= (uint32_t)kSplitList) {         // perm through the list, so that it is written in order
      each_of(0, [&](int u, uint32_t) {
        const uint32_t c = code[u], w = c >> 5, pos = first[w] + (uint32_t)__popc(bits[w] & ((1u << (c & 31u)) - 1u));
        list[pos - base] = index[u];
        put_beside(pos, c, index[u]);
      });
      __syncthreads();
      for (uint32_t e = tid; e < T; e += kSplitThreads) perm_s[base + e] = (int32_t)list[e];
      return;
    }
    for (uint32_t e0 = 0; e0 < T; e0 += kSplitList) {
      fetch(code, index, e0);
      each_of(e0, [&](int u, uint32_t) {
        const uint32_t c = code[u], w = c >> 5;
        put(first[w] + (uint32_t)__popc(bits[w] & ((1u << (c & 31u)) - 1u)), c, index[u]);
      });
    }
    return;
  }
  if (T <= (uint32_t)kSplitList) {           // by words of the map, then ranked, as in k_direct
    __syncthreads();
    for (int w = tid; w < words; w += kSplitThreads) bits[w] = 0u;
    if (tid == 0) crowded = 0u;
    __syncthreads();
    each_of(0, [&](int u, uint32_t) { atomicAdd(&bits[code[u] >> 5], 1u); });
    __syncthreads();
    sum = 0;
    uint32_t largest = 0;
    for (int w = w0; w < w0 + per && w < words; ++w) {
      sum += bits[w];
      largest = bits[w] > largest ? bits[w] : largest;
    }
    if (largest > (uint32_t)kDirectRanked) crowded = 1u;
    run = block_exclusive_scan<kSplitThreads>(sum, wave_totals, nullptr);
    for (int w = w0; w < w0 + per && w < words; ++w) {
      const uint32_t c = bits[w];
      first[w] = bits[w] = run;              // bits: where the word's next pillar goes
      run += c;
    }
    __syncthreads();
    each_of(0, [&](int u, uint32_t e) { list[atomicAdd(&bits[code[u] >> 5], 1u)] = code[u] << 12 | e; });
    __syncthreads();
    if (crowded == 0u) {
      each_of(0, [&](int u, uint32_t e) {
        put(base + rank_in_run(list, first[code[u] >> 5], bits[code[u] >> 5], code[u] << 12 | e), code[u], index[u]);
      });
      return;
    }
    direct_sort<kSplitThreads>(list, T);
    // The positions in the bucket come back as places in the order; the indices are where they were.
    for (uint32_t e = tid; e < T; e += kSplitThreads) bits[list[e] & 0xfffu] = e;
    __syncthreads();
    each_of(0, [&](int u, uint32_t e) { put(base + bits[e], code[u], index[u]); });
    return;
  }
  // Stable passes, wavefronts with consecutive pieces: one by the cells' numbers where these are few, otherwise two by eight bits
  // of the key value with the pillars in memory in between.
  const uint32_t piece = (T + kSplitThreads - 1u) / kSplitThreads * 64u, begin = wave * piece;
  const uint32_t stop = begin + piece < T ? begin + piece : T;
  constexpr int STEPS = 6;                   // loads of a lane in flight
  // The wavefront's pillars as k_split left them, tile after tile: use(valid, key value, index), of up to 64 at a time
  auto from_tiles = [&](auto use) {
    int t = 0;
    for (int skip = kSplitMaxTiles / 2; skip > 0; skip >>= 1)
      if ((uint32_t)__builtin_amdgcn_readfirstlane((int)cum[t + skip]) <= begin) t += skip;
    uint32_t e = begin, tile_end = (uint32_t)__builtin_amdgcn_readfirstlane((int)cum[t + 1]);
    while (e < stop) {
      uint32_t v[STEPS], left[STEPS], tile_first[STEPS];
#pragma unroll
      for (int u = 0; u < STEPS; ++u) {
        left[u] = 0u;
        if (e < stop) {
          while (tile_end <= e) tile_end = (uint32_t)__builtin_amdgcn_readfirstlane((int)cum[++t + 1]);
          left[u] = (tile_end < stop ? tile_end : stop) - e;
          tile_first[u] = (uint32_t)t * (uint32_t)tile_rows;
          v[u] = entries[(uint32_t)__builtin_amdgcn_readfirstlane((int)from[t]) + e + ((uint32_t)lane < left[u] ? (uint32_t)lane : 0u)];
          e += left[u] < 64u ? left[u] : 64u;
        }
      }
#pragma unroll
      for (int u = 0; u < STEPS; ++u)
        if (left[u]) use((uint32_t)lane < left[u], v[u] >> kSplitLocalBits, tile_first[u] + (v[u] & ((1u << kSplitLocalBits) - 1u)));
    }
  };
  // read: as from_tiles.  use: where it goes, key value, index
  auto pass = [&](int bits_of, auto read, auto digit, auto use) {
    uint32_t* const counts = list + (wave << bits_of);     // [kSplitWaves][1 << bits_of]
    auto ranked = [&](bool valid, uint32_t c) -> uint32_t {  // place of the pillar, once more counted
      const uint32_t d = digit(c);
      const uint64_t same = same_number(d, bits_of) & __ballot(valid);
      const uint32_t before = counts[d], nth = lanes_below(same);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (valid && nth == 0u) counts[d] = before + (uint32_t)__popcll(same);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      return before + nth;
    };
    __syncthreads();
    for (int w = tid; w < kSplitWaves << bits_of; w += kSplitThreads) list[w] = 0u;
    __syncthreads();
    read([&](bool valid, uint32_t c, uint32_t) { ranked(valid, c); });
    __syncthreads();
    uint32_t total = 0;
    if (tid < 1 << bits_of)
      for (int w = 0; w < kSplitWaves; ++w) {
        const uint32_t v = list[(w << bits_of) + tid];
        list[(w << bits_of) + tid] = total;
        total += v;
      }
    const uint32_t start = block_exclusive_scan<kSplitThreads>(total, wave_totals, nullptr);
    if (tid < 1 << bits_of)
      for (int w = 0; w < kSplitWaves; ++w) list[(w << bits_of) + tid] += start;
    __syncthreads();
    read([&](bool valid, uint32_t c, uint32_t i) {
      const uint32_t pos = ranked(valid, c);
      if (valid) use(pos, c, i);
    });
  };
  auto put_in = [&](uint32_t pos, uint32_t c, uint32_t i) { put(base + pos, c, i); };
  if (cells <= 1u << kSplitDigits) {
    for (int w = w0; w < w0 + per && w < words; ++w) {
      first[w] = run;
      run += (uint32_t)__popc(bits[w]);
    }
    int bits_of = 0;
    while (1u << bits_of < cells) ++bits_of;
    pass(bits_of, from_tiles, [&](uint32_t c) { return first[c >> 5] + (uint32_t)__popc(bits[c >> 5] & ((1u << (c & 31u)) - 1u)); },
         put_in);
    return;
  }
  uint32_t* const codes = scratch + (int64_t)s * n + base;
  uint32_t* const indices = scratch + (int64_t)(S + s) * n + base;
  pass(8, from_tiles, [](uint32_t c) { return c & 255u; }, [&](uint32_t pos, uint32_t c, uint32_t i) {
    codes[pos] = c;
    indices[pos] = i;
  });
  auto from_memory = [&](auto use) {
    for (uint32_t e0 = begin; e0 < stop; e0 += 64 * STEPS) {
      uint32_t c[STEPS], i[STEPS];
#pragma unroll
      for (int u = 0; u < STEPS; ++u) {
        const uint32_t e = e0 + u * 64 + lane, at = e < stop ? e : stop - 1u;
        c[u] = codes[at];
        i[u] = indices[at];
      }
#pragma unroll
      for (int u = 0; u < STEPS; ++u)
        if (e0 + u * 64 < stop) use(e0 + u * 64 + lane < stop, c[u], i[u]);
    }
  };
  pass(8, from_memory, [](uint32_t c) { return c >> 8; }, put_in);
}

// Pass plan for keys of `key_bits` bits: digit width and number of passes.
struct PassPlan { bool small; int kpt, rb, passes; int64_t tiles; };
// (`sorts` decides between the paths only: digit width, passes and tiles, and with them the workspace, do not depend on it)
inline PassPlan pass_plan(int64_t n, int key_bits, int sorts) {
  PassPlan pp;
  pp.small = ceil_div(n > 0 ? n : 1, (int64_t)kSortThreads * kSmallKpt) * sorts <= kSmallMaxTiles;
  pp.kpt = pp.small ? kSmallKpt
         : ceil_div(n, (int64_t)kSortThreads * kMidKptA) <= kMidMaxTilesA ? kMidKptA
         : ceil_div(n, (int64_t)kSortThreads * kMidKptB) <= kMidMaxTilesB ? kMidKptB : kLargeKpt;
  pp.passes = (key_bits + 9) / 10;
  // the narrowest digit that still needs no extra pass: smaller tables, longer runs per digit
  pp.rb = 8 * pp.passes >= key_bits ? 8 : 9 * pp.passes >= key_bits ? 9 : 10;
  pp.tiles = ceil_div(n > 0 ? n : 1, (int64_t)kSortThreads * pp.kpt);
  return pp;
}

// How a sort makes its keys with 24-bit products; false if its grid is too large for them.
bool direct_keys(const ff_geom* g, const FlattenZ* z, const KeyParams& kp, DirectKeys* k) {
  const int at_l2 = kp.bits_l3, at_l1 = at_l2 + kp.bits_l2, at_w3 = at_l1 + kp.bits_l1, at_w2 = at_w3 + kp.bits_w3,
            at_w1 = at_w2 + kp.bits_w2;
  auto axis = [](DirectAxis& a, int64_t grid, int shift, int win, int at_w, int at_l) {
    a.shift = shift;
    a.max = (uint32_t)(grid + shift - 1);
    a.mul = ((1u << 20) + (uint32_t)win - 1u) / (uint32_t)win;
    a.unit_l = 1u << at_l;
    a.rest_w = (1u << at_w) - (uint32_t)win * a.unit_l;  // (the window's field begins where the local one's values end)
    return grid + shift <= kDirectMaxGrid;
  };
  if (!axis(k->x, g->grid_x, kp.sx, kp.win_x, kp.axis == 0 ? at_w1 : at_w2, kp.axis == 0 ? at_l1 : at_l2) ||
      !axis(k->y, g->grid_y, kp.sy, kp.win_y, kp.axis == 0 ? at_w2 : at_w1, kp.axis == 0 ? at_l2 : at_l1) ||
      !axis(k->z, z ? z->grid_z : 1, kp.sz, kp.win_z, at_w3, 0))
    return false;
  k->unit_b = 1u << (at_w1 + kp.bits_w1);
  return true;
}

// Whether this cloud is sorted in one launch (k_direct), and how.
bool direct_plan(int64_t n, const ff_geom* g, const FlattenZ* z, int sorts, const Batch& bt, int key_bits, DirectBatch* db) {
  if (n > kDirectMaxRows || g->num_frames > kDirectMaxFrames || key_bits > 24) return false;
  const int64_t codes = (int64_t)1 << key_bits;
  const int code_bits = 32 - bt.kp[0].idx_bits;
  const int64_t most = code_bits >= 17 ? kDirectMaxCodes : (int64_t)1 << code_bits;
  // As many workgroups as fill the chip with all sorts (an eighth of it left to the weight packing), fewer for few pillars.
  int64_t parts = sorts >= 4 ? 56 : 64;
  const int64_t enough = ceil_div(n, 128);
  if (parts > enough) parts = enough;
  if (parts * most < codes) parts = ceil_div(codes, most);
  // Beyond one workgroup a compute unit there is a second round: it pays for this few pillars (four sorts of eight frames, 512
  // workgroups, radix path / this one: 16,000 pillars 39 / 26 us, 60,000 52 / 57).
  if (parts * sorts > 512) return false;
  db->parts = (int32_t)parts;
  db->range = (uint32_t)(ceil_div(ceil_div(codes, parts), (int64_t)32) * 32);
  for (int s = 0; s < sorts; ++s)
    if (!direct_keys(g, z, bt.kp[s], &db->k[s])) return false;
  return true;
}

// Whether it is sorted by k_split and k_buckets, and how.
bool split_plan(int64_t n, const ff_geom* g, const FlattenZ* z, int sorts, const Batch& bt, int tile_rows, SplitBatch* sb) {
  if (n < kSplitMinRows || ceil_div(n, (int64_t)tile_rows) > kSplitMaxTiles) return false;
  sb->tiles = (int32_t)ceil_div(n, (int64_t)tile_rows);
  const int64_t fill = kSplitBuckets / sorts;
  int64_t most = n / kSplitRows < fill ? n / kSplitRows : fill;
  if (n / kSplitRowsMany > most) most = n / kSplitRowsMany;
  if (most > kSplitMaxBuckets) most = kSplitMaxBuckets;
  int64_t buckets = 0;
  for (int s = 0; s < sorts; ++s) {
    const KeyParams& kp = bt.kp[s];
    SplitSort& t = sb->s[s];
    const int at_frame = kp.key_bits - kp.bits_b, at_w1 = at_frame - kp.bits_w1;
    if (kp.key_bits > 32 || at_frame > 23 || !direct_keys(g, z, kp, &t.k)) return false;
    const int64_t nw1 = kp.axis == 0 ? ceil_div((int64_t)g->grid_x + kp.sx, kp.win_x) : ceil_div((int64_t)g->grid_y + kp.sy, kp.win_y);
    int64_t in_frame = 0;
    int c = 5;                               // the smallest buckets that are few enough
    for (;; ++c) {
      if (c > kSplitCodeBits || c > at_frame) return false;
      in_frame = c > at_w1 ? ceil_div(nw1, (int64_t)1 << (c - at_w1)) : nw1 << (at_w1 - c);
      if (in_frame * kp.B <= most) break;
    }
    t.code_bits = c;
    t.in_frame = at_frame - c;
    t.per_frame = (int32_t)in_frame;
    t.skip = (int32_t)(((int64_t)1 << t.in_frame) - in_frame);
    if (in_frame * kp.B > buckets) buckets = in_frame * kp.B;
  }
  sb->bins = (int32_t)((buckets + 2) & ~(int64_t)1);  // (one more for what lies behind the cloud in its last tile)
  sb->bin_bits = 1;
  while ((1 << sb->bin_bits) < sb->bins) ++sb->bin_bits;
  return (int64_t)sb->tiles * sb->bins * 2 <= n * 4;
}

struct Layout {
  size_t off_words0, off_words1, off_counts, off_totals, off_frames, total;
};

// Workspace for S sorts of n words whose keys have at most max_key_bits bits (a call may sort
// narrower keys than the workspace query assumed, and a narrower key can pick a wider digit).
void make_layout(int64_t n, int S, int num_frames, int max_key_bits, Layout* L) {
  size_t count_words = 0, total_words = 0;
  for (int kb = 0; kb <= max_key_bits; ++kb) {
    const PassPlan pp = pass_plan(n, kb, S);
    const size_t pc = pp.passes > 0 ? pp.passes : 1;  // key generation always fills one table
    const size_t cw = (size_t)S * pc * (size_t)pp.tiles * ((size_t)1 << pp.rb);
    const size_t tw = (size_t)S * pc * ((size_t)1 << pp.rb);
    if (cw > count_words) count_words = cw;
    if (tw > total_words) total_words = tw;
  }
  size_t off = 0;
  L->off_words0 = off; off += align_up((size_t)S * n * 8, 256);
  L->off_words1 = off; off += align_up((size_t)S * n * 8, 256);
  L->off_counts = off; off += align_up(count_words * 4 + 256, 256);
  L->off_totals = off; off += align_up(total_words * 4 + 256, 256);
  L->off_frames = off; off += align_up((size_t)S * 2 * ((size_t)num_frames + 1) * 4, 256);
  L->total = off;
}

}  // namespace

int make_flatten_plan(int64_t n, const ff_geom* g, int axis, int shift, FlattenPlan* plan) {
  return make_flatten_plan_z(n, g, nullptr, axis, shift, plan);
}

int make_flatten_plan_z(int64_t n, const ff_geom* g, const FlattenZ* z, int axis, int shift, FlattenPlan* plan) {
  if (!g || n < 0 || n > 0x7fffffffLL) return FF_ERR_ARG;
  if (z && (z->grid_z < 1 || z->win_z < 1 || z->win_z > 256)) return FF_ERR_ARG;
  if (g->num_frames < 1 || g->grid_x < 1 || g->grid_y < 1) return FF_ERR_ARG;
  if (g->win_x < 1 || g->win_x > 256 || g->win_y < 1 || g->win_y > 256) return FF_ERR_ARG;
  if (axis != 0 && axis != 1) return FF_ERR_ARG;
  if (g->num_frames > 65535) return FF_ERR_UNSUPPORTED;
  const int64_t sx = shift ? g->win_x / 2 : 0, sy = shift ? g->win_y / 2 : 0;
  const int64_t nwx = ceil_div((int64_t)g->grid_x + sx, g->win_x);
  const int64_t nwy = ceil_div((int64_t)g->grid_y + sy, g->win_y);
  if (nwx > 65535 || nwy > 65535) return FF_ERR_UNSUPPORTED;
  const int bwx = bit_width_u64((uint64_t)nwx - 1), bwy = bit_width_u64((uint64_t)nwy - 1);
  const int blx = bit_width_u64((uint64_t)g->win_x - 1), bly = bit_width_u64((uint64_t)g->win_y - 1);
  plan->bits_b = bit_width_u64((uint64_t)g->num_frames - 1);
  plan->bits_w1 = axis == 0 ? bwx : bwy;
  plan->bits_w2 = axis == 0 ? bwy : bwx;
  plan->bits_l1 = axis == 0 ? blx : bly;
  plan->bits_l2 = axis == 0 ? bly : blx;
  plan->bits_w3 = plan->bits_l3 = 0;
  if (z) {
    const int64_t nwz = ceil_div((int64_t)z->grid_z + (shift ? z->win_z / 2 : 0), z->win_z);
    if (nwz > 65535) return FF_ERR_UNSUPPORTED;
    plan->bits_w3 = bit_width_u64((uint64_t)nwz - 1);
    plan->bits_l3 = bit_width_u64((uint64_t)z->win_z - 1);
  }
  plan->key_bits = plan->bits_b + plan->bits_w1 + plan->bits_w2 + plan->bits_w3 + plan->bits_l1 + plan->bits_l2 +
                   plan->bits_l3;
  plan->idx_bits = n > 0 ? bit_width_u64((uint64_t)n - 1) : 0;
  if (plan->key_bits + plan->idx_bits > 64) return FF_ERR_UNSUPPORTED;
  plan->passes = (plan->key_bits + kRadixBits - 1) / kRadixBits;
  return FF_OK;
}

size_t flatten_workspace_bytes(int64_t n, const ff_geom* g, int num_sorts) {
  return flatten_workspace_bytes_z(n, g, nullptr, num_sorts);
}

size_t flatten_workspace_bytes_z(int64_t n, const ff_geom* g, const FlattenZ* z, int num_sorts) {
  // Independent of axis and shift: the shifted plan never has fewer key bits.
  FlattenPlan p;
  if (num_sorts < 1 || num_sorts > kMaxSorts) return 0;
  if (make_flatten_plan_z(n, g, z, 0, 1, &p) != FF_OK) return 0;
  Layout L;
  make_layout(n, num_sorts, g->num_frames, p.key_bits, &L);
  return L.total;
}

int flatten_launch(const int32_t* coords, int64_t n, const ff_geom* g, int num_sorts, const int* axis,
                   const int* shift, int G, int drop, int32_t* const* perm, int32_t* const* inv_perm,
                   int32_t* const* group_offsets, int32_t* const* num_groups, uint64_t* const* keys_sorted,
                   void* workspace, size_t workspace_bytes, const PackJob* pack, hipStream_t stream) {
  return flatten_launch_z(coords, n, g, nullptr, num_sorts, axis, shift, G, drop, perm, inv_perm, group_offsets,
                          num_groups, keys_sorted, workspace, workspace_bytes, pack, stream);
}

static int flatten_launch_impl(const int32_t* coords, const PointCells* pts, int64_t n, const ff_geom* g,
                               const FlattenZ* z, int num_sorts, const int* axis, const int* shift, int G, int drop,
                               int32_t* const* perm, int32_t* const* inv_perm, int32_t* const* group_offsets,
                               int32_t* const* num_groups, uint64_t* const* keys_sorted, void* workspace,
                               size_t workspace_bytes, const PackJob* pack, hipStream_t stream);

int flatten_launch_z(const int32_t* coords, int64_t n, const ff_geom* g, const FlattenZ* z, int num_sorts,
                     const int* axis, const int* shift, int G, int drop, int32_t* const* perm,
                     int32_t* const* inv_perm, int32_t* const* group_offsets, int32_t* const* num_groups,
                     uint64_t* const* keys_sorted, void* workspace, size_t workspace_bytes, const PackJob* pack,
                     hipStream_t stream) {
  return flatten_launch_impl(coords, nullptr, n, g, z, num_sorts, axis, shift, G, drop, perm, inv_perm, group_offsets,
                             num_groups, keys_sorted, workspace, workspace_bytes, pack, stream);
}

int flatten_launch_points(const PointCells* pts, int64_t n, const ff_geom* g, int32_t* perm, int32_t* group_offsets,
                          int32_t* num_groups, uint64_t* keys_sorted, void* workspace, size_t workspace_bytes,
                          hipStream_t stream) {
  if (!pts || (n > 0 && !pts->xy)) return FF_ERR_ARG;
  const int axis = 0, shift = 0;
  return flatten_launch_impl(nullptr, pts, n, g, nullptr, 1, &axis, &shift, 0x40000000, 0, &perm, nullptr,
                             &group_offsets, &num_groups, &keys_sorted, workspace, workspace_bytes, nullptr, stream);
}

static int flatten_launch_impl(const int32_t* coords, const PointCells* pts, int64_t n, const ff_geom* g,
                               const FlattenZ* z, int num_sorts, const int* axis, const int* shift, int G, int drop,
                               int32_t* const* perm, int32_t* const* inv_perm, int32_t* const* group_offsets,
                               int32_t* const* num_groups, uint64_t* const* keys_sorted, void* workspace,
                               size_t workspace_bytes, const PackJob* pack, hipStream_t stream) {
  if (num_sorts < 1 || num_sorts > kMaxSorts || G < 1) return FF_ERR_ARG;
  if (z && keys_sorted) return FF_ERR_ARG;  // the exported key format has no room for the z fields
  Batch bt;
  int max_key_bits = 0;
  for (int s = 0; s < num_sorts; ++s) {
    FlattenPlan plan;
    const int st = make_flatten_plan_z(n, g, z, axis[s], shift[s], &plan);
    if (st != FF_OK) return st;
    if (!group_offsets[s] || !num_groups[s] || (n > 0 && !perm[s])) return FF_ERR_ARG;
    KeyParams& kp = bt.kp[s];
    kp.B = g->num_frames; kp.win_x = g->win_x; kp.win_y = g->win_y; kp.win_z = z ? z->win_z : 1;
    kp.sx = shift[s] ? g->win_x / 2 : 0; kp.sy = shift[s] ? g->win_y / 2 : 0;
    kp.sz = z && shift[s] ? z->win_z / 2 : 0;
    kp.axis = axis[s]; kp.stride = z ? 4 : 3;
    kp.bits_b = plan.bits_b; kp.bits_w1 = plan.bits_w1; kp.bits_w2 = plan.bits_w2; kp.bits_w3 = plan.bits_w3;
    kp.bits_l1 = plan.bits_l1; kp.bits_l2 = plan.bits_l2; kp.bits_l3 = plan.bits_l3;
    kp.key_bits = plan.key_bits; kp.idx_bits = plan.idx_bits;
    bt.perm[s] = perm[s]; bt.group_offsets[s] = group_offsets[s]; bt.num_groups[s] = num_groups[s];
    bt.keys_sorted[s] = keys_sorted ? keys_sorted[s] : nullptr;
    bt.inv_perm[s] = inv_perm ? inv_perm[s] : nullptr;
    if (plan.key_bits > max_key_bits) max_key_bits = plan.key_bits;
  }
  for (int s = num_sorts; s < kMaxSorts; ++s) {
    bt.kp[s] = bt.kp[0]; bt.perm[s] = nullptr; bt.group_offsets[s] = nullptr; bt.num_groups[s] = nullptr;
    bt.keys_sorted[s] = nullptr;
    bt.inv_perm[s] = nullptr;
  }
  if (n > 0 && !coords && !pts) return FF_ERR_ARG;
  const PointCells point_src = pts ? *pts : PointCells();  // xy == nullptr: integer coordinates
  Layout L;
  make_layout(n, num_sorts, g->num_frames, max_key_bits, &L);
  if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < L.total) return FF_ERR_WORKSPACE;

  char* ws = (char*)workspace;
  uint64_t* buf[2] = {(uint64_t*)(ws + L.off_words0), (uint64_t*)(ws + L.off_words1)};
  uint32_t* counts = (uint32_t*)(ws + L.off_counts);
  uint32_t* totals = (uint32_t*)(ws + L.off_totals);
  int32_t* frame_tab = (int32_t*)(ws + L.off_frames);

  DirectBatch db;
  if (n > 0 && !pts && direct_plan(n, g, z, num_sorts, bt, max_key_bits, &db)) {
    PackJob job = PackJob();
    job.layers = 0; job.blocks = 1;
    if (pack) job = *pack;
    const unsigned blocks = (unsigned)(num_sorts * (db.parts + 1) + ceil_div((int64_t)job.layers * job.blocks, kDirectThreads / 256));
    const size_t lds = (size_t)(kDirectList + kDirectShared) * 4 + db.range / 32 * 8;
    static std::atomic<uint64_t> allowed[4] = {{0}, {0}, {0}, {0}};  // bit d: the largest dynamic LDS size is allowed on device d
    auto go = [&](auto kern, int which) -> int {
      int dev = 0;
      if (hipGetDevice(&dev) != hipSuccess) return FF_ERR_LAUNCH;
      const uint64_t bit = 1ull << (dev & 63);
      if (!(allowed[which].load(std::memory_order_acquire) & bit)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (kDirectList + kDirectShared) * 4 + kDirectMaxCodes / 32 * 8) != hipSuccess)
          return FF_ERR_LAUNCH;
        allowed[which].fetch_or(bit, std::memory_order_release);
      }
      hipLaunchKernelGGL(kern, dim3(blocks), dim3(kDirectThreads), lds, stream, coords, (int)n, num_sorts, db.parts, db.range, G,
                         drop, bt, db, job);
      return launch_status();
    };
    if (g->num_frames > 1) return z ? go(k_direct<true, true>, 3) : go(k_direct<false, true>, 2);
    return z ? go(k_direct<true, false>, 1) : go(k_direct<false, false>, 0);
  }

  const int own = n >= kSplitManyRows ? kSplitMany : n * num_sorts > kSplitFewRows ? kSplitFew : kSplitLeast;
  const int tile_rows = kSplitThreads * own;
  SplitBatch sb;
  if (!pts && split_plan(n, g, z, num_sorts, bt, tile_rows, &sb)) {
    PackJob job = PackJob();
    job.layers = 0; job.blocks = 1;
    if (pack) job = *pack;
    uint32_t* entries = (uint32_t*)buf[0];
    uint32_t* table = entries + (int64_t)num_sorts * n;
    // (what is left of the first buffer of words; a 16-byte boundary)
    const size_t table_end = align_up((size_t)num_sorts * (n * 4 + (int64_t)sb.tiles * sb.bins * 2), 16);
    const size_t frame_bytes = (size_t)num_sorts * g->num_frames * ((sb.tiles + 7) & ~7) * 2;
    uint16_t* frame_table = g->num_frames > 1 && table_end + frame_bytes <= (size_t)num_sorts * n * 8
                                ? (uint16_t*)((char*)buf[0] + table_end) : nullptr;
    const unsigned blocks = (unsigned)(num_sorts * sb.tiles + ceil_div((int64_t)job.layers * job.blocks, kSplitThreads / 256));
    const size_t counters = (size_t)kSplitWaves * sb.bins * 2, stage = (size_t)tile_rows * 4;
    int64_t buckets = 0, ends[kMaxSorts];
    int words = 0;
    for (int s = 0; s < kMaxSorts; ++s) {
      if (s < num_sorts) buckets += (int64_t)sb.s[s].per_frame * bt.kp[s].B;
      ends[s] = buckets;
    }
    for (int s = 0; s < num_sorts; ++s) {
      if (1 << (sb.s[s].code_bits - 5) > words) words = 1 << (sb.s[s].code_bits - 5);
    }
    // (bits and first of a bucket; the places of a list's entries, which take the same memory; the group list's tables)
    size_t lds = (size_t)(kSplitList + 2 * kSplitMaxTiles + 1) * 4 + (size_t)(2 * words > kSplitList ? 2 * words : kSplitList) * 4;
    auto go = [&](auto split) {
      hipLaunchKernelGGL(split, dim3(blocks), dim3(kSplitThreads), counters > stage ? counters : stage, stream, coords, (int)n,
                         num_sorts, sb.tiles, sb.bins, sb.bin_bits, (int)g->num_frames, entries, table, frame_table,
                         sb, job);
      hipLaunchKernelGGL(k_buckets, dim3((unsigned)(num_sorts + 8 * ceil_div(buckets, 8))), dim3(kSplitThreads), lds, stream,
                         (const uint16_t*)table, (int)n, num_sorts, sb.tiles, sb.bins, tile_rows, (int)ends[0], (int)ends[1],
                         (int)ends[2], (int)ends[3], entries, (uint32_t*)buf[1], frame_table, G, drop, bt, sb);
      return launch_status();
    };
    auto go_z = [&](auto Z, auto frames) {
      constexpr bool z_ = decltype(Z)::value, f_ = decltype(frames)::value;
      return own == kSplitMany ? go(k_split<z_, f_, kSplitMany>)
           : own == kSplitFew ? go(k_split<z_, f_, kSplitFew>) : go(k_split<z_, f_, kSplitLeast>);
    };
    if (g->num_frames > 1) return z ? go_z(std::true_type(), std::true_type()) : go_z(std::false_type(), std::true_type());
    return z ? go_z(std::true_type(), std::false_type()) : go_z(std::false_type(), std::false_type());
  }

  int cur = 0;
  bool outputs_done = false;
  if (n > 0) {
    const bool in_block = inv_perm && inv_perm[0];  // only a block asks for the inverse permutations
    const PassPlan pp = pass_plan(n, max_key_bits, in_block ? num_sorts : 1);
    const int P = pp.passes > 0 ? pp.passes : 1;  // zero key bits: the words are generated in order
    // The last pass can write the outputs itself when its digit contains the whole frame field.
    bool fuse = pp.passes > 0;
    for (int s = 0; s < num_sorts; ++s)
      fuse = fuse && bt.kp[s].key_bits - (pp.passes - 1) * pp.rb >= bt.kp[s].bits_b;
    const dim3 grid((unsigned)pp.tiles, (unsigned)num_sorts), block(kSortThreads);
    // The first radix pass takes the weight-packing workgroups along (key generation when there is no
    // pass): that launch is bound by the latency of a few sort workgroups and leaves most of the chip idle.
    PackJob no_job = PackJob();
    no_job.layers = 0; no_job.blocks = 1;
    const PackJob job = pack ? *pack : no_job;
    // With radix passes to run, the layers are shared out between key generation and the first pass (both
    // launches are short and leave most compute units idle; one of them alone would be stretched by the packing).
    PackJob job_a = job, job_b = no_job;   // job_a: key generation (everything when there is no pass), job_b: first pass
    if (pp.passes > 0 && job.layers > 0) {
      job_a.layers = job.layers / 2;
      job_b = job;
      job_b.first = job_a.layers;
      job_b.layers = job.layers - job_a.layers;
      if (job_a.layers == 0) job_a = no_job;
    }
    const dim3 grid_a((unsigned)(pp.tiles + ceil_div((int64_t)job_a.layers * job_a.blocks, num_sorts)), (unsigned)num_sorts);
    const dim3 grid_pack((unsigned)(pp.tiles + ceil_div((int64_t)job_b.layers * job_b.blocks, num_sorts)), (unsigned)num_sorts);
#define FF_PASSES(RB, KPT, SCANNED)                                                                                  \
    do {                                                                                                             \
      hipLaunchKernelGGL((k_keygen<RB, KPT>), grid_a, block, 0, stream, coords, n, bt, P, pp.tiles, buf[0], counts,  \
                         job_a, point_src);                                                                          \
      for (int pass = 0; pass < pp.passes; ++pass) {                                                                 \
        if (SCANNED) {                                                                                               \
          if (pass > 0)                                                                                              \
            hipLaunchKernelGGL((k_tile_counts<RB, KPT>), grid, block, 0, stream, buf[cur], n, bt, pass, P, pp.tiles, \
                               counts);                                                                              \
          auto scan = [&](auto kern, int digits) {                                                                   \
            hipLaunchKernelGGL(kern, dim3((1u << RB) / digits, (unsigned)num_sorts), dim3(kScanThreads), 0, stream,  \
                               counts, totals, pass, P, pp.tiles);                                                   \
          };                                                                                                         \
          if (pp.tiles <= kScanWideTiles) scan(k_scan_cols<RB, kScanWide, kScanFewRows>, kScanWide);                 \
          else if (pp.tiles <= kScanFewRowsTiles) scan(k_scan_cols<RB, kScanNarrow, kScanFewRows>, kScanNarrow);     \
          else scan(k_scan_cols<RB, kScanNarrow, kScanManyRows>, kScanNarrow);                                       \
        }                                                                                                            \
        if (fuse && pass == pp.passes - 1)                                                                           \
          hipLaunchKernelGGL((k_pass<RB, KPT, true, SCANNED>), pass == 0 ? grid_pack : grid, block, 0, stream,      \
                             buf[cur], buf[cur ^ 1], n, bt, pass, P, pp.tiles, G, drop, counts, totals,              \
                             pass == 0 ? job_b : no_job);                                                              \
        else                                                                                                         \
          hipLaunchKernelGGL((k_pass<RB, KPT, false, SCANNED>), pass == 0 ? grid_pack : grid, block, 0, stream,     \
                             buf[cur], buf[cur ^ 1], n, bt, pass, P, pp.tiles, G, drop, counts, totals,              \
                             pass == 0 ? job_b : no_job);                                                              \
        cur ^= 1;                                                                                                    \
      }                                                                                                              \
    } while (0)
    if (!pp.small && pp.kpt == kMidKptA && pp.rb == 8) FF_PASSES(8, kMidKptA, true);
    else if (!pp.small && pp.kpt == kMidKptA && pp.rb == 9) FF_PASSES(9, kMidKptA, true);
    else if (!pp.small && pp.kpt == kMidKptA) FF_PASSES(10, kMidKptA, true);
    else if (pp.kpt == kMidKptB && pp.rb == 8) FF_PASSES(8, kMidKptB, true);
    else if (pp.kpt == kMidKptB && pp.rb == 9) FF_PASSES(9, kMidKptB, true);
    else if (pp.kpt == kMidKptB) FF_PASSES(10, kMidKptB, true);
    else if (!pp.small && pp.rb == 8) FF_PASSES(8, kLargeKpt, true);
    else if (!pp.small && pp.rb == 9) FF_PASSES(9, kLargeKpt, true);
    else if (!pp.small) FF_PASSES(10, kLargeKpt, true);
    else if (pp.rb == 8) FF_PASSES(8, kSmallKpt, false);
    else if (pp.rb == 9) FF_PASSES(9, kSmallKpt, false);
    else FF_PASSES(10, kSmallKpt, false);
#undef FF_PASSES
    outputs_done = fuse;
  }
  if (!outputs_done) {
    if (g->num_frames > 256 || (g->num_frames > 1 && n > 65536))  // else every output block derives it itself
      hipLaunchKernelGGL(k_frames, dim3((unsigned)num_sorts), dim3(256), 0, stream, buf[cur], n, bt, G, drop, frame_tab);
    hipLaunchKernelGGL(k_finalize, dim3((unsigned)(n > 0 ? ceil_div(n, 256) : 1), (unsigned)num_sorts), dim3(256), 0,
                       stream, buf[cur], n, bt, G, drop, frame_tab);
  }
  return launch_status();
}

}  // namespace ff
