// Group attention layer (paper Sec. 4.2.2, Eq. (2)) in 16-bit storage as ONE fused kernel whose wavefronts cut the FEATURES:
//
//   gather -> LN1 -> packed QKV projection -> per-head softmax(Q K^T / sqrt(d)) V -> out-proj
//   + residual -> LN2 -> Linear + GELU -> Linear + residual -> scatter
//
// Mapping.  A workgroup owns one group (or GPW small ones) as blocks of 32 rows.  Its C / 32 wavefronts each compute 32
// features of Q, K and V (whole heads: scores, softmax and P V stay inside a wavefront), of the output projection and of
// the second FFN product, and their share of the hidden units, for all rows.  A weight fragment goes from L2 straight to
// the registers of the one wavefront that needs it and multiplies every row block; the activations (LN1 output, attention
// output, LN2 output, hidden units) go round through LDS in operand order, six barriers a layer.
//
// All products are v_mfma_f32_32x32x16, computed transposed: D[output feature][row], lane (h, n) = 32 h + n of a tile
// holds row n and features (r & 3) + 8 (r >> 2) + 4 h in registers r = 0..15 (V: operand roles swapped, D[row][feature]).
// Registers 4 k .. 4 k + 3 and 8 + 4 k .. 8 + 4 k + 3, rounded to 16 bits, are the operand of step k of a later product
// over these 32 features: that is the order of inputs the packed weights (pack_weights.h) come in, whose 16 x 32 fragments
// are read as halves of 32 x 16 ones.  Heads of 16: registers 8 a .. 8 a + 7 of Q and K are one step of head a, and in P V
// the 16 rows of the A operand that belong to the other head are ones, so that the row sums of P come with the product.
//
// What bounds it.  One group on a compute unit (C = 128, G = 64): the chain of one wavefront, 9 us, of which 2 are the trip to
// its rows; a lone wavefront issues an instruction every five to seven cycles.  Two groups: 14 us.  Many: instruction issue
// (1,657 vector instructions a wavefront, a fifth of them exponentials and their 16-bit roundings, beside 161 products of 32
// cycles) and weight delivery (256 KB a group from L2, a quarter of the time in a build without it); the matrix pipe is
// busy 43 % of the time.  Before (wavefronts that cut the rows, every one reading all weights from LDS) / now, us a
// launch: C = 128, G = 64, 12,345 rows 14.5 / 10.3, 480,000 rows 208 / 190; G = 100, 30,000 rows 32.8 / 27; G = 128,
// 80,000 rows 46.5 / 42.5; C = 256, G = 64, 2,000 rows 40 / 16, 60,000 rows 85 / 79; G = 96, 240,000 rows 364 / 311.
#include "elem16.h"
#include "pack_weights.h"
#include <atomic>
#include <type_traits>

namespace ff {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c) {
#ifdef FF_LAYER_F16
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(el8, a), __builtin_bit_cast(el8, b), c, 0, 0, 0);
#else
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(el8, a), __builtin_bit_cast(el8, b), c, 0, 0, 0);
#endif
}
// Products of the last sixteen rows: the sums come out the same bit for bit as from two products of 32 rows and half the inputs
// (measured on 51,200 sums of 128 terms, bfloat16 and half; with the inputs in another order 20 to 45 % of them differ).
__device__ __forceinline__ f32x4 mma16(u32x4 a, u32x4 b, f32x4 c) {
#ifdef FF_LAYER_F16
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(el8, a), __builtin_bit_cast(el8, b), c, 0, 0, 0);
#else
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(el8, a), __builtin_bit_cast(el8, b), c, 0, 0, 0);
#endif
}
// Of the four rows of 16 lanes: a = a0 a1 a2 a3, b likewise -> a0 b0 a2 b2, a1 b1 a3 b3
__device__ __forceinline__ void swap_rows(uint32_t& a, uint32_t& b) {
  auto t = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = t[0]; b = t[1];
}
// -> a0 a1 b0 b1, a2 a3 b2 b3
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b) {
  auto t = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = t[0]; b = t[1];
}
// v of lane n and of lane n + 32 combined, in every lane
__device__ __forceinline__ float half_sum(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}
__device__ __forceinline__ float half_max(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
// Sum over LPR (8, 16, 32) neighbouring lanes.
template <int LPR> __device__ __forceinline__ float lane_sum(float v) {
  v += dpp<0xB1>(v);                            // quad_perm 1,0,3,2
  v += dpp<0x4E>(v);                            // quad_perm 2,3,0,1
  v += dpp<0x141>(v);                           // row_half_mirror
  if constexpr (LPR >= 16) v += dpp<0x140>(v);  // row_mirror
  if constexpr (LPR >= 32) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  }
  return v;
}
// Nothing is moved across by the instruction scheduler: it would sink loads issued ahead to where they are used.
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }
// Workgroup barrier that waits for this wavefront's LDS operations only: weight fragments requested ahead stay in
// flight across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Groups of 65 to 80: the last sixteen rows run through the linear layers, LayerNorm 2 and GELU as such, on 16 x 16 x 32 products
// (a sixth less of all that than as half of a block of 32), and in the layout of a block only through the attention.  The weights
// of two steps become two tiles of 16 features by eight lane swaps, which ride beside the products of the other rows.  240,000
// rows, C = 256, G = 69, us a layer: 408 -> 386; 32,117 rows, C = 128, embedding: 24, the same; registers 256 -> 204.  (Groups of
// 33 to 48 and 97 to 112 stay with half a block: four blocks so, and two with 16-bit results, need scratch memory, at C = 128 and, 36 to
// 232 bytes, at 256.  There, 500 groups with 16-bit and float32 results, us: G = 48 39.1 and 41.8, so 58.1 and 39.4; G = 112 76.2
// and 83.5, so 82.3 and 82.7.)
constexpr bool tail_of_16(int PT, bool HALF) { return HALF && PT == 3; }
constexpr int kLdsBytes = 160 * 1024;  // LDS of one compute unit

template <int C, int F, int RB, bool TAIL>
struct Plan {
  static constexpr int NS = C / 32, NT = 64 * NS, R = 32 * RB - (TAIL ? 16 : 0);
  static constexpr int A = R * C * 2;          // one set of operands: LN1 output, LN2 output, second half of the hidden units;
  static constexpr int B = A;                  // another: attention output, first half of the hidden units, rows on their way out
  static constexpr int STATS = R * NS * 8;
  static constexpr int PAR = (5 * C + F) * 4;  // query bias, output bias, LN2 scale and shift, FFN biases
  static constexpr int TAB = RB * 64;          // which rows are members, as operand masks
  static constexpr int SRC = R * (RB % 2 == 0 ? 8 : 4);  // where the rows came from, and (four blocks) their pillars
  static constexpr int TOTAL = A + B + STATS + PAR + TAB + SRC;
  static_assert(F == 2 * C, "half of the hidden units are one set of operands");
};

// SPLIT: the workgroup takes half of a group's queries (half_of: which), and the keys and values of all of it.
template <int C, int DH, int F, int PT, int GPW, bool HALF, int MINW, bool OUT_F32, bool PE, bool SPLIT>
__device__ __forceinline__ void slice_layer(
    const uint16_t* __restrict__ feats, const int32_t* __restrict__ perm, const u32x4* __restrict__ packed, int n, int G,
    int in_sorted, int max_groups, const int32_t* __restrict__ goff, const int32_t* __restrict__ num_groups,
    const int32_t* __restrict__ out_index, void* __restrict__ out, const uint16_t* __restrict__ pos_embed, int drop, float eps,
    const int workgroup, const int half_of) {
  constexpr int RB = PT * GPW;             // row blocks of the workgroup
  constexpr bool TAIL = tail_of_16(PT, HALF);
  constexpr int NF = TAIL ? RB - 1 : RB;   // row blocks of 32
  constexpr int NQ = SPLIT ? NF / 2 : NF;  // of them, those of its queries,
  const int qb = half_of * NQ;             // from this one on
  static_assert(!SPLIT || (!TAIL && GPW == 1 && RB % 2 == 0), "half of the blocks");
  using PL = Plan<C, F, RB, TAIL>;
  constexpr int NS = PL::NS;
  constexpr int KB = C / 32, NB = C / 16;  // 32-wide input blocks, 16-wide output blocks
  constexpr int KS = C / 16;               // steps along C
  constexpr int FH = 6 * KB + NB, FF = 2 * KB + NB;  // fragments of a head-dim unit and of a hidden unit of the packed stream
  constexpr int WD = RB <= 3 && MINW <= 2 ? 4 : 3;  // weight operands in flight
  constexpr int NH = 32 / DH;              // heads of a wavefront
  constexpr int LPR = C / 8, RPI = 64 / LPR;  // lanes per row (16 bytes each), rows per load instruction
  constexpr int NL = PL::R / 16;           // load instructions of a wavefront
  static_assert(DH == 16 || DH == 32, "head dim");
  constexpr int RPW = NL * RPI;            // rows a wavefront loads and normalises: of one group
  constexpr int NLQ = SPLIT ? NL / 2 : NL, RPWQ = NLQ * RPI;  // and stores
  static_assert(RPW * NS == PL::R && (GPW == 1 || 32 * PT % RPW == 0), "of one group");

  extern __shared__ u32x4 lds[];
  u32x4* const Ab = lds;
  u32x4* const Bb = lds + PL::A / 16;
  char* const ldsc = reinterpret_cast<char*>(lds) + PL::A + PL::B;
  f32x2* const stats = reinterpret_cast<f32x2*>(ldsc);
  float* const par = reinterpret_cast<float*>(ldsc + PL::STATS);
  uint32_t* const tab = reinterpret_cast<uint32_t*>(ldsc + PL::STATS + PL::PAR);
  int32_t* const src = reinterpret_cast<int32_t*>(ldsc + PL::STATS + PL::PAR + PL::TAB);
  // Four whole row blocks (of the widest form three and a half) leave no registers beside the attention: the pillars wait in LDS,
  // the weights that come after it are requested behind it, and all that follows from the lane's number is worked out again (beside
  // the split groups' form it took two or three registers more than there are: 128 groups of 128 rows 13.09 / 12.98 us).  12,000
  // and 30,000 rows with 6 to 25 registers in scratch memory / so, us: 128 features, G = 128, float32 results 21.8 / 20.9 and 25.7
  // / 24.4; 256 features, G = 120 33.0 / 32.3 and 46.1 / 44.3.  At 128 features with 16-bit results it is even, G = 120 19.9 / 19.5 and
  // 21.6 / 21.9, G = 128 19.2 / 19.5 and 21.1 / 21.4; where there are registers it costs 1 to 4 %.
  constexpr bool FULL = SPLIT || RB > 3 && (!HALF || (C > 128 && PE));
  int32_t* const pillar = src + PL::R;
  constexpr int P_BQ = 0, P_BO = C, P_G2 = 2 * C, P_B2N = 3 * C, P_B2 = 4 * C, P_B1 = 5 * C;

  const int tid = threadIdx.x;
  int lane = tid & 63, nrow = lane & 31, h = lane >> 5;
  const int trow = lane & 15, tq = lane >> 4;    // of the last sixteen rows: the row, and features 4 tq .. + 3 of each tile of 16
  const int s = __builtin_amdgcn_readfirstlane(tid >> 6);  // slice

  // ---- weights: a 32 x 16 operand is one 16-byte piece per lane of two 16 x 32 fragments -----------------------------
  // (buffer loads: the lane's part of the address is one register, the rest a scalar)
  const auto wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4*>(packed), 0, (KB * FH + (F / 32) * FF) * 1024, 0x00020000);
  auto w_load = [&](uint32_t lane_off, int frag, int bytes) -> u32x4 {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, (int)lane_off + bytes, frag * 1024, 0));
  };
  const uint32_t second = (lane >> 4) & 1;       // row of the tile: 0..15 or 16..31
  uint32_t lane_rows, lane_cols;
  auto offsets = [&]() {
    const uint32_t piece = (uint32_t)((16 * (lane >> 5) + (lane & 15)) * 16), row16 = (lane >> 4) & 1;
    lane_rows = piece + row16 * (KB * 1024u);    // Q, K, V, W1: the second 16 rows come KB fragments later
    lane_cols = piece + row16 * 1024u;           // W_o, W2: next to each other
  };
  offsets();
  auto rows_at = [&](int frag, int ks) { return w_load(lane_rows, frag + ks / 8 * 4, ks % 8 * 512); };  // of a row tile
  auto wk_at = [&](int ks) { return rows_at(s * FH, ks); };
  auto wv_at = [&](int ks) { return rows_at(s * FH + 2 * KB, ks); };
  auto wq_at = [&](int ks) { return rows_at(s * FH + 4 * KB, ks); };
  auto wo_at = [&](int ks) { return w_load(lane_cols, (ks / 2) * FH + 6 * KB + 2 * s, ks % 2 * 512); };
  auto w1_at = [&](int t, int ks) { return rows_at(KB * FH + (t * NS + s) * FF, ks); };
  auto w2_at = [&](int ks) { return w_load(lane_cols, KB * FH + (ks / 2) * FF + 2 * KB + 2 * s, ks % 2 * 512); };

  // ---- which rows ----------------------------------------------------------------------------------------------------
  // Slot sl of the wavefront's group -> sorted position.  Rows beyond the group's members repeat its last member: their
  // scores then never exceed the real ones, and they are cut out of the sums (below).
  const int gl_s = GPW == 1 ? 0 : s * RPW / (32 * PT);  // the group whose rows this wavefront loads and stores
  const int g_s = workgroup * GPW + gl_s;
  const int slot0 = s * RPW - gl_s * 32 * PT;
  const int lr = lane / LPR, lc = lane % LPR;
  int first = 0;                           // sorted position of the wavefront's first row
  int off[NL];                             // and how far from it mine are
  auto place = [&](int start_at, int last) {
    first = __builtin_amdgcn_readfirstlane(start_at + (slot0 < last ? slot0 : last));
#pragma unroll
    for (int t = 0; t < NL; ++t) {
      const int sl = slot0 + t * RPI + lr;
      off[t] = (sl < last ? sl : last) - (slot0 < last ? slot0 : last);
    }
  };
  int pil[NL];
  auto fetch_pillars = [&]() {
#pragma unroll
    for (int t = 0; t < NL; ++t) pil[t] = (perm + first)[(uint32_t)off[t]];
  };
  u32x4 raw[NL];
  auto fetch_rows = [&]() {
    if (in_sorted) {                       // side by side
#pragma unroll
      for (int t = 0; t < NL; ++t)
        raw[t] = *reinterpret_cast<const u32x4*>(feats + (int64_t)first * C + (uint32_t)(off[t] * C + 8 * lc));
    } else {
#pragma unroll
      for (int t = 0; t < NL; ++t) raw[t] = *reinterpret_cast<const u32x4*>(feats + (int64_t)pil[t] * C + 8 * lc);
    }
  };
  // Groups of the first (or only) frame start at g * G: what is loaded from there does not wait for the group list.
  {
    const uint32_t g0 = (uint32_t)g_s * (uint32_t)G, end = (uint32_t)n - 1u;
    const uint32_t from = g0 < end ? g0 : end, left = end - from;
    place((int)from, (int)(left < (uint32_t)G - 1u ? left : (uint32_t)G - 1u));
  }
  if (in_sorted == 2) fetch_rows();        // before anything that waits
  fetch_pillars();
  uint32_t touched[RB > 3 ? 1 : 2];
  touch_lines<PL::NT, (KB * FH + (F / 32) * FF) * 1024>(packed, (max_groups + GPW - 1) / GPW, tid, touched);
  f32x4 gam[2], bet[2];                    // LayerNorm 1 scale and shift of my features
  const float* const params = reinterpret_cast<const float*>(packed + (size_t)(KB * FH + (F / 32) * FF) * 64);
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    gam[e] = *reinterpret_cast<const f32x4*>(params + 8 * lc + 4 * e);
    bet[e] = *reinterpret_cast<const f32x4*>(params + C + 8 * lc + 4 * e);
  }
  static_assert((5 * C + F) / 4 <= PL::NT, "one piece a thread");
  f32x4 par_piece;
  if (tid < (5 * C + F) / 4) par_piece = *reinterpret_cast<const f32x4*>(params + 2 * C + 4 * tid);

  const int ngroups = *num_groups;
  int start = 0, m = 0, end1 = 0;          // of that group
  bool whole = true;                       // every row of the workgroup is a member of its group
#pragma unroll
  for (int gl = 0; gl < GPW; ++gl) {
    const int g = workgroup * GPW + gl;
    const int gc = g < max_groups ? g : max_groups - 1;
    const int o0 = goff[gc], o1 = goff[gc + 1];
    // A list of full groups only ('Drop Residual') has the next start beyond this group's end.
    const int mg = g < ngroups ? (o1 - o0 < G ? o1 - o0 : G) : 0;
    if (gl == gl_s) { start = g < ngroups ? o0 : 0; m = mg; end1 = o1; }
    whole = whole && (mg == 32 * PT || mg == 0);
    if (tid < PT * 16) {                   // operand masks: entry (block, step, half, pair of rows)
      const int key = 32 * (tid >> 4) + 16 * ((tid >> 3) & 1) + 8 * ((tid >> 1) & 1) + 4 * ((tid >> 2) & 1) + 2 * (tid & 1);
      const int mm = mg > 0 ? mg : 32 * PT;
      tab[gl * PT * 16 + tid] = (key < mm ? 0xffffu : 0u) | (key + 1 < mm ? 0xffff0000u : 0u);
    }
  }
  const bool guessed = (int64_t)g_s * G == start && (m == G || start + m == n);  // wave-uniform, as is m
  if (!guessed) {
    place(start, m > 0 ? m - 1 : 0);
    if (m > 0) {
      fetch_pillars();
    } else {                               // no such group: its slots hold row 0, whatever is in perm
#pragma unroll
      for (int t = 0; t < NL; ++t) pil[t] = 0;
    }
  }
  if (in_sorted != 2 || !guessed) fetch_rows();
  u32x4 pe[PE ? NL : 1];
  if constexpr (PE) {
#pragma unroll
    for (int t = 0; t < NL; ++t) pe[t] = *reinterpret_cast<const u32x4*>(pos_embed + (int64_t)pil[t] * C + 8 * lc);
  }

  // ---- LN1 -> A ------------------------------------------------------------------------------------------------------
#pragma unroll
  for (int t = 0; t < NL; ++t) {
    const int row = s * RPW + t * RPI + lr;
    if (lc == 0) {
      src[row] = in_sorted ? first + off[t] : pil[t];
      if constexpr (FULL) pillar[row] = pil[t];
    }
    float y[8], su = 0.f, ss = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) { y[2 * j] = el_lo(raw[t][j]); y[2 * j + 1] = el_hi(raw[t][j]); }
#pragma unroll
    for (int j = 0; j < 8; ++j) su += y[j];
    const float mu = lane_sum<LPR>(su) * (1.0f / C);
#pragma unroll
    for (int j = 0; j < 8; ++j) ss = fmaf(y[j], y[j], ss);
    const float var = fmaxf(lane_sum<LPR>(ss) * (1.0f / C) - mu * mu, 0.f);
    const float sc = rsqrtf(var + eps), sh = -mu * sc;
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = fmaf(fmaf(y[j], sc, sh), gam[j / 4][j % 4], bet[j / 4][j % 4]);
    // features 8 lc .. + 7: eight bytes for each half of step lc & 1 of input block lc / 4
    auto put = [&](u32x4* dst) {
      if (TAIL && row >= 32 * NF) {        // of the last sixteen: eight bytes each of two runs of four features
        char* const p = reinterpret_cast<char*>(dst + (NF * KS + (lc >> 2)) * 64 + 32 * (lc & 1) + (row & 15)) + 8 * ((lc >> 1) & 1);
        *reinterpret_cast<u32x2*>(p) = u32x2{pack2(y[0], y[1]), pack2(y[2], y[3])};
        *reinterpret_cast<u32x2*>(p + 256) = u32x2{pack2(y[4], y[5]), pack2(y[6], y[7])};
        return;
      }
      char* const p = reinterpret_cast<char*>(dst + ((row >> 5) * KS + 2 * (lc >> 2) + (lc & 1)) * 64 + (row & 31)) + 8 * ((lc >> 1) & 1);
      *reinterpret_cast<u32x2*>(p) = u32x2{pack2(y[0], y[1]), pack2(y[2], y[3])};
      *reinterpret_cast<u32x2*>(p + 512) = u32x2{pack2(y[4], y[5]), pack2(y[6], y[7])};
    };
    put(Ab);
    if constexpr (PE) {
#pragma unroll
      for (int j = 0; j < 4; ++j) { y[2 * j] += el_lo(pe[t][j]); y[2 * j + 1] += el_hi(pe[t][j]); }
      put(Bb);
    }
  }
  if (tid < (5 * C + F) / 4) reinterpret_cast<f32x4*>(par)[tid] = par_piece;
  touch_done(touched);
  // ---- rows of no group ('Drop Residual'): copied, unless there is no list -----------------------------------------
  if (drop && ngroups >= 0 && half_of == 0) {
    auto copy_rows = [&](int lo, int hi, int w0, int nw) {  // by wavefronts w0 .. w0 + nw - 1
      hi = hi < n ? hi : n;
      for (int p = lo + (s - w0) * RPI + lr; p < hi; p += nw * RPI) {
        const int pillar = perm[p];
        const u32x4 v = *reinterpret_cast<const u32x4*>(feats + (int64_t)(in_sorted ? p : pillar) * C + 8 * lc);
        const int64_t to = (int64_t)(out_index ? out_index[pillar] : pillar) * C + 8 * lc;
        if constexpr (OUT_F32) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            *reinterpret_cast<f32x2*>(reinterpret_cast<float*>(out) + to + 2 * e) = f32x2{el_lo(v[e]), el_hi(v[e])};
        } else {
          *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(out) + to) = v;
        }
      }
    };
    constexpr int WPG = NS / GPW;  // wavefronts of a group
    if (g_s == 0) copy_rows(0, ngroups > 0 ? start : n, gl_s * WPG, WPG);
    if (g_s < ngroups) copy_rows(start + m, end1, gl_s * WPG, WPG);
  }

  const f32x16 kZero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto vec16 = [&](int off) -> f32x16 {    // 16 entries of a per-feature vector in accumulator order
    f32x16 v;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const f32x4 t = *reinterpret_cast<const f32x4*>(par + off + 8 * b + 4 * h);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[4 * b + j] = t[j];
    }
    return v;
  };
  auto vec4 = [&](f32x4 (&v)[2], int off) {  // the same for the last sixteen rows
#pragma unroll
    for (int t = 0; t < 2; ++t) v[t] = *reinterpret_cast<const f32x4*>(par + off + 16 * t + 4 * tq);
  };
  // Operand of a product over the 32 features of a slice, of the last sixteen rows
  auto operand16 = [&](const f32x4 (&v)[2]) -> u32x4 {
    return u32x4{pack2(v[0][0], v[0][1]), pack2(v[0][2], v[0][3]), pack2(v[1][0], v[1][1]), pack2(v[1][2], v[1][3])};
  };
  // Operand of step k of a product over the 32 features of an accumulator
  auto operand = [&](const f32x16& v, int k) -> u32x4 {
    return u32x4{pack2(v[4 * k], v[4 * k + 1]), pack2(v[4 * k + 2], v[4 * k + 3]),
                 pack2(v[8 + 4 * k], v[8 + 4 * k + 1]), pack2(v[8 + 4 * k + 2], v[8 + 4 * k + 3])};
  };

  // A bias as the start of a sum: one product, of the bias in the first input and ones (16-bit numbers both, so exact), and
  // zeros in all other inputs of both (an infinite bias times zero would be no number).
  u32x4 first_one = {h == 0 ? kOnePair & 0xffffu : 0u, 0u, 0u, 0u};
  auto bias = [&](int off) -> u32x4 { return u32x4{h == 0 ? pack2(par[off + nrow], 0.f) : 0u, 0u, 0u, 0u}; };

  // Steps of a product: N weight operands and NF activation operands (of `rows`) a step, handed to `mm`; every second step the
  // weights of two as tiles of sixteen features, with the operand of the last sixteen rows, to `mt`.  Weights are requested D - 1 steps
  // ahead, the first of them by `ahead`, before the caller's barrier; step k of this product is step `at` + k of whatever
  // `w` and `wf` stand for.  `beside`: work of the vector units for each step.
  auto ahead = [&](auto& w, auto wf) {
    constexpr int D = sizeof(w) / sizeof(w[0]);
#pragma unroll
    for (int d = 0; d < D - 1; ++d) wf(w[d], d);
  };
  auto nothing = [](int) {};
  auto product_of = [&](auto blocks, auto& w, auto wf, int at, const u32x4* rows, auto mm, auto mt, auto beside) {
    constexpr int D = sizeof(w) / sizeof(w[0]), N = sizeof(w[0]) / 16, MINE = decltype(blocks)::value;
    const u32x4* const p = rows + lane;
    const u32x4* const tail = p + NF * KS * 64;
    constexpr int DA = N == 1 && MINE <= 3 ? 3 : 2;
    u32x4 a[DA][MINE], a16[2];
#pragma unroll
    for (int d = 0; d < DA - 1; ++d)
#pragma unroll
      for (int b = 0; b < MINE; ++b) a[d][b] = p[(b * KS + d) * 64];
    if constexpr (TAIL) a16[0] = tail[0];
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      fence();
      u32x4 before[N];
      if constexpr (TAIL) {
        if (k % 2) {
#pragma unroll
          for (int i = 0; i < N; ++i) before[i] = w[(at + k - 1) % D][i];
          if (k + 1 < KS) a16[(k + 1) / 2 % 2] = tail[(k + 1) / 2 * 64];
        }
      }
      wf(w[(at + k + D - 1) % D], at + k + D - 1);
      if (k + DA - 1 < KS) {
#pragma unroll
        for (int b = 0; b < MINE; ++b) a[(k + DA - 1) % DA][b] = p[(b * KS + k + DA - 1) * 64];
      }
      mm(w[(at + k) % D], a[k % DA]);
      if constexpr (TAIL) {
        if (k % 2) {                       // two steps' weights as two tiles of 16 features x 32 inputs
          u32x4 t[N][2];
#pragma unroll
          for (int i = 0; i < N; ++i) {
            t[i][0] = before[i];
            t[i][1] = w[(at + k) % D][i];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              uint32_t lo = t[i][0][j], hi = t[i][1][j];
              swap_halves(lo, hi);
              swap_rows(lo, hi);
              t[i][0][j] = lo; t[i][1][j] = hi;
            }
          }
          mt(t, a16[k / 2 % 2]);
        }
      }
      beside(k);
    }
    fence();
  };

  auto product = [&](auto& w, auto wf, int at, const u32x4* rows, auto mm, auto mt, auto beside) {  // of the queries' rows
    product_of(std::integral_constant<int, NQ>(), w, wf, at, rows, mm, mt, beside);
  };
  auto product_all = [&](auto& w, auto wf, int at, const u32x4* rows, auto mm, auto mt, auto beside) {
    product_of(std::integral_constant<int, NF>(), w, wf, at, rows, mm, mt, beside);
  };

  // ---- Q, K, V of this slice -----------------------------------------------------------------------------------------
  u32x4 Q[RB][2], K[RB][2], V[RB][2];      // rounded: registers 8 a .. 8 a + 7 of the accumulators
  auto halves = [&](u32x4 (&d)[2], const f32x16& v) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int j = 0; j < 4; ++j) d[a][j] = pack2(v[8 * a + 2 * j], v[8 * a + 2 * j + 1]);
  };
  constexpr float qscale = (DH == 16 ? 0.25f : 0.17677669529663687f) * 1.44269504088896340736f;  // log2(e) / sqrt(d)
  {
    constexpr bool JOINT = RB <= 2 && !PE && !SPLIT;  // all three at once; otherwise the values first,
    constexpr bool PAIR = RB <= 3 && !SPLIT;  // and then keys and queries together (four row blocks: one after the other)
    u32x4 w1[WD][1], w2[4][2], w3[2][3];
    auto vf = [&](u32x4 (&d)[1], int k) { if (k < KS) d[0] = wv_at(k); };
    auto kf = [&](u32x4 (&d)[1], int k) { if (k < KS) d[0] = wk_at(k); };
    auto qf = [&](u32x4 (&d)[1], int k) { if (k < KS) d[0] = wq_at(k); };
    auto kqf = [&](u32x4 (&d)[2], int k) { if (k < KS) { d[0] = wk_at(k); d[1] = wq_at(k); } };
    auto kqvf = [&](u32x4 (&d)[3], int k) { if (k < KS) { d[0] = wk_at(k); d[1] = wq_at(k); d[2] = wv_at(k); } };
    if constexpr (JOINT) ahead(w3, kqvf);
    else ahead(w1, vf);
    lds_barrier();
    f32x16 aq[NQ], ak[NF], av[NF];
    f32x4 tq4[2], tk4[2], tv4[2];          // of the last sixteen rows: two tiles of 16 features
    auto start_at = [&](f32x16 (&v)[NF], f32x4 (&t)[2]) {
#pragma unroll
      for (int b = 0; b < NF; ++b) v[b] = kZero;
      t[0] = t[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto done = [&](u32x4 (&d)[RB][2], auto& v) {
#pragma unroll
      for (int b = 0; b < (int)(sizeof(v) / sizeof(v[0])); ++b) halves(d[b], v[b]);
    };
    // Sixteen rows in the layout of 32: rows 16 .. 31 repeat them (queries, keys) or stay unused (values)
    auto done16 = [&](u32x4 (&d)[RB][2], const f32x4 (&t)[2], bool values) {
      if constexpr (TAIL) {
        uint32_t lo[4], hi[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) lo[j] = pack2(t[j / 2][2 * (j % 2)], t[j / 2][2 * (j % 2) + 1]);
        if (values) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            hi[j] = lo[2 + j];
            swap_rows(lo[j], hi[j]);
            swap_halves(lo[j], hi[j]);
          }
          d[RB - 1][0] = u32x4{lo[0], lo[1], hi[0], hi[1]};
          d[RB - 1][1] = u32x4{0u, 0u, 0u, 0u};
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            hi[j] = lo[j];
            swap_rows(lo[j], hi[j]);
            swap_halves(lo[j], hi[j]);
          }
#pragma unroll
          for (int a = 0; a < 2; ++a) d[RB - 1][a] = u32x4{lo[2 * a], lo[2 * a + 1], hi[2 * a], hi[2 * a + 1]};
        }
      }
    };
    const u32x4* const qk = PE ? Bb : Ab;
    start_at(av, tv4);
    if constexpr (!JOINT) {
      product_all(w1, vf, 0, Ab, [&](const u32x4 (&w)[1], const u32x4 (&a)[NF]) {
#pragma unroll
        for (int b = 0; b < NF; ++b) av[b] = mma(a[b], w[0], av[b]);
      }, [&](const u32x4 (&w)[1][2], u32x4 a) {
#pragma unroll
        for (int t = 0; t < 2; ++t) tv4[t] = mma16(a, w[0][t], tv4[t]);
      }, nothing);
      if constexpr (PAIR) ahead(w2, kqf);
      else ahead(w1, kf);
      done(V, av);
      done16(V, tv4, true);
    }
    start_at(ak, tk4);
    {
      const u32x4 bq = bias(P_BQ + 32 * s);
#pragma unroll
      for (int b = 0; b < NQ; ++b) aq[b] = mma(bq, first_one, kZero);
      if constexpr (TAIL) vec4(tq4, P_BQ + 32 * s);
    }
    if constexpr (JOINT) {
      product_all(w3, kqvf, 0, Ab, [&](const u32x4 (&w)[3], const u32x4 (&a)[NF]) {
#pragma unroll
        for (int b = 0; b < NF; ++b) {
          ak[b] = mma(w[0], a[b], ak[b]);
          aq[b] = mma(w[1], a[b], aq[b]);
          av[b] = mma(a[b], w[2], av[b]);
        }
      }, [&](const u32x4 (&w)[3][2], u32x4 a) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          tk4[t] = mma16(w[0][t], a, tk4[t]);
          tq4[t] = mma16(w[1][t], a, tq4[t]);
          tv4[t] = mma16(a, w[2][t], tv4[t]);
        }
      }, nothing);
      done(V, av);
      done16(V, tv4, true);
    } else if constexpr (PAIR) {
      product_all(w2, kqf, 0, qk, [&](const u32x4 (&w)[2], const u32x4 (&a)[NF]) {
#pragma unroll
        for (int b = 0; b < NF; ++b) {
          ak[b] = mma(w[0], a[b], ak[b]);
          aq[b] = mma(w[1], a[b], aq[b]);
        }
      }, [&](const u32x4 (&w)[2][2], u32x4 a) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          tk4[t] = mma16(w[0][t], a, tk4[t]);
          tq4[t] = mma16(w[1][t], a, tq4[t]);
        }
      }, nothing);
    } else {
      auto onto = [&](f32x4 (&v)[2]) {
        return [&](const u32x4 (&w)[1][2], u32x4 a) {
#pragma unroll
          for (int t = 0; t < 2; ++t) v[t] = mma16(w[0][t], a, v[t]);
        };
      };
      product_all(w1, kf, 0, qk, [&](const u32x4 (&w)[1], const u32x4 (&a)[NF]) {
#pragma unroll
        for (int b = 0; b < NF; ++b) ak[b] = mma(w[0], a[b], ak[b]);
      }, onto(tk4), nothing);
      ahead(w1, qf);
      done(K, ak);
      done16(K, tk4, false);
      product(w1, qf, 0, qk + qb * KS * 64, [&](const u32x4 (&w)[1], const u32x4 (&a)[NQ]) {
#pragma unroll
        for (int b = 0; b < NQ; ++b) aq[b] = mma(w[0], a[b], aq[b]);
      }, onto(tq4), nothing);
    }
    done(Q, aq);
    done16(Q, tq4, false);
    if constexpr (JOINT || PAIR) {
      done(K, ak);
      done16(K, tk4, false);
    }
    if constexpr (PE) lds_barrier();       // the attention output goes where the embedded rows were
  }

  // ---- attention -----------------------------------------------------------------------------------------------------
  // The weights of everything after it are one stream: W_o, two tiles of W_1, W_2.
  u32x4 w[WD][1];
  auto wf = [&](u32x4 (&d)[1], int k) {
    if (k < KS) d[0] = wo_at(k);
    else if (k < 3 * KS) d[0] = w1_at(k / KS - 1, k % KS);
    else if (k < 5 * KS) d[0] = w2_at(k - 3 * KS);
  };
  // SHORT: some rows of the workgroup are no members.  HALF: no group has members in the second half of its last block.
  auto attention = [&](auto shortc) {
    constexpr bool SHORT = decltype(shortc)::value;
    auto member = [&](int b, int t) -> u32x4 {  // mask of the rows of operand (b, t)
      return reinterpret_cast<const u32x4*>(tab)[(b * 2 + t) * 2 + h];
    };
    auto ones = [&](int b, int t) -> u32x4 {
      u32x4 one = {kOnePair, kOnePair, kOnePair, kOnePair};
      if constexpr (SHORT) one &= member(b, t);
      return one;
    };
    if constexpr (SHORT) {
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int t = 0; t < 2; ++t) V[b][t] &= member(b, t);
    }
#pragma unroll
    for (int gl = 0; gl < GPW; ++gl) {
#pragma unroll
      for (int hd = 0; hd < NH; ++hd) {
        // A operand of P V: the head's value rows, and (heads of 16) ones in the other head's rows
        u32x4 va[PT][2];
#pragma unroll
        for (int kt = 0; kt < PT; ++kt)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const int b = gl * PT + kt;
            if constexpr (DH == 32) {
              va[kt][t] = V[b][t];
            } else {
              const u32x4 one = ones(b, t);
#pragma unroll
              for (int j = 0; j < 4; ++j) va[kt][t][j] = (int)second == hd ? V[b][t][j] : one[j];
            }
          }
#pragma unroll
        for (int q0 = 0; q0 < (SPLIT ? NQ : PT); ++q0) {
          const int qt = gl * PT + q0;
          f32x16 O, rs;
          auto used = [](int kt) { return HALF && kt == PT - 1 ? 8 : 16; };  // registers of a block that stand for members
          auto scores = [&](int kt) -> f32x16 {
            f32x16 S = mma(K[gl * PT + kt][DH == 16 ? hd : 0], Q[qt][DH == 16 ? hd : 0], kZero);
            if constexpr (DH == 32) S = mma(K[gl * PT + kt][1], Q[qt][1], S);
            return S;
          };
          auto accumulate = [&](int kt, const f32x16& P) {
            u32x4 p[2];
            halves(p, P);
#pragma unroll
            for (int t = 0; t < (HALF && kt == PT - 1 ? 1 : 2); ++t) {
              O = mma(va[kt][t], p[t], kt == 0 && t == 0 ? kZero : O);
              if constexpr (DH == 32) rs = mma(ones(gl * PT + kt, t), p[t], kt == 0 && t == 0 ? kZero : rs);
            }
          };
          auto sum = [&]() { return DH == 32 ? rs[0] : hd == 0 ? O[8] : O[0]; };
          f32x16 S[PT];
#pragma unroll
          for (int kt = 0; kt < PT; ++kt) S[kt] = scores(kt);
          float mx = S[0][0];
#pragma unroll
          for (int kt = 0; kt < PT; ++kt)
#pragma unroll
            for (int r = 0; r < used(kt); ++r) mx = fmaxf(mx, S[kt][r]);
          mx = -half_max(mx) * qscale;
          // p = 2^((s - max) * log2(e) / sqrt(d)): the score scale lives in the exponent argument
#pragma unroll
          for (int kt = 0; kt < PT; ++kt) {
#pragma unroll
            for (int r = 0; r < used(kt); ++r) S[kt][r] = __builtin_amdgcn_exp2f(fmaf(S[kt][r], qscale, mx));
            accumulate(kt, S[kt]);
          }
          const float inv = __builtin_amdgcn_rcpf(sum());
          const bool last16 = TAIL && qt == NF;
          u32x4* const dst = Bb + (last16 ? (NF * KS + s) * 64 + 16 * h + trow : (qt * KS + 2 * s) * 64 + lane);
          const int step = last16 ? 32 : 64;
          if (last16 && nrow > 15) continue;  // (they repeat the other sixteen)
          if constexpr (DH == 16) {        // the head's eight features: half of the operands of both steps
            float o[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) o[r] = O[8 * hd + r] * inv;
#pragma unroll
            for (int k = 0; k < 2; ++k)
              *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(dst + k * step) + 8 * hd) =
                  u32x2{pack2(o[4 * k], o[4 * k + 1]), pack2(o[4 * k + 2], o[4 * k + 3])};
          } else {
            O *= inv;
#pragma unroll
            for (int k = 0; k < 2; ++k) dst[k * step] = operand(O, k);
          }
        }
      }
    }
  };
  if constexpr (!FULL) ahead(w, wf);
  if (!HALF && whole) attention(std::false_type());
  else attention(std::true_type());
  if constexpr (FULL) {
    asm volatile("" : "+v"(lane));
    nrow = lane & 31;
    h = lane >> 5;
    first_one[0] = h == 0 ? kOnePair & 0xffffu : 0u;
    offsets();
    ahead(w, wf);
  }
  const int lr_out = lane / LPR, lc_out = lane % LPR;

  // ---- output projection + residual ----------------------------------------------------------------------------------
  // The rows again, 16 bytes a lane: lane h holds features 16 h + 8 u .. + 7 of the slice, the operand of a product whose other
  // operand is one where the feature is the output's own.  It adds the numbers as they are (1 x), and leaves the vector units
  // out of it.
  u32x4 again[NQ][2], unit[2], again16, unit16[2];
#pragma unroll
  for (int b = 0; b < NQ; ++b)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      again[b][u] = *reinterpret_cast<const u32x4*>(feats + (int64_t)src[32 * (qb + b) + nrow] * C + 32 * s + 16 * h + 8 * u);
  {
    const int mine = nrow - 16 * h;
    const uint32_t one = (kOnePair & 0xffffu) << (16 * (mine & 1));
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) unit[u][j] = (mine >> 1) == 4 * u + j ? one : 0u;
  }
  if constexpr (TAIL) {                    // (all 32 features of the slice are one step: lane tq holds 8 tq .. + 7)
    again16 = *reinterpret_cast<const u32x4*>(feats + (int64_t)src[32 * NF + trow] * C + 32 * s + 8 * tq);
    const uint32_t one = (kOnePair & 0xffffu) << (16 * (trow & 1));
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) unit16[t][j] = 2 * t + (trow >> 3) == tq && ((trow & 7) >> 1) == j ? one : 0u;
  }
  f32x16 x1[NQ];                           // residual stream of (my 32 features, all rows)
  f32x4 x16[2];
  {
    const f32x16 bo = vec16(P_BO + 32 * s);
#pragma unroll
    for (int b = 0; b < NQ; ++b) x1[b] = bo;
    if constexpr (TAIL) vec4(x16, P_BO + 32 * s);
  }
  auto onto_x1 = [&](const u32x4 (&w)[1], const u32x4 (&a)[NQ]) {
#pragma unroll
    for (int b = 0; b < NQ; ++b) x1[b] = mma(w[0], a[b], x1[b]);
  };
  auto onto_x16 = [&](const u32x4 (&w)[1][2], u32x4 a) {
#pragma unroll
    for (int t = 0; t < 2; ++t) x16[t] = mma16(w[0][t], a, x16[t]);
  };
  lds_barrier();
  product(w, wf, 0, Bb, onto_x1, onto_x16, nothing);
#pragma unroll
  for (int b = 0; b < NQ; ++b)
#pragma unroll
    for (int u = 0; u < 2; ++u) x1[b] = mma(unit[u], again[b][u], x1[b]);
  if constexpr (TAIL) {
#pragma unroll
    for (int t = 0; t < 2; ++t) x16[t] = mma16(unit16[t], again16, x16[t]);
  }
  int orow[NLQ];                           // rows of `out` of my rows
#pragma unroll
  for (int t = 0; t < NLQ; ++t) {
    const int p = FULL ? pillar[32 * qb + s * RPWQ + t * RPI + lr_out] : pil[t];
    orow[t] = out_index ? out_index[p] : p;
  }

  // ---- LN2 -> A ------------------------------------------------------------------------------------------------------
  // Sum and sum of squares of a row: every wavefront's 32 features, combined through LDS.
  auto sums = [&](const f32x16& x) -> f32x2 {  // of this lane's features
    float su4[4], ss4[4];                  // (short chains)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      su4[j] = x[j];
      ss4[j] = x[j] * x[j];
#pragma unroll
      for (int e = 1; e < 4; ++e) { su4[j] += x[4 * e + j]; ss4[j] = fmaf(x[4 * e + j], x[4 * e + j], ss4[j]); }
    }
    return f32x2{(su4[0] + su4[1]) + (su4[2] + su4[3]), (ss4[0] + ss4[1]) + (ss4[2] + ss4[3])};
  };
#pragma unroll
  for (int b = 0; b < NQ; ++b) {
    const f32x2 v = sums(x1[b]);
    const float su = half_sum(v[0]), ss = half_sum(v[1]);
    if (h == 0) stats[(b * 32 + nrow) * NS + s] = f32x2{su, ss};
  }
  if constexpr (TAIL) {                    // (lanes n and n + 32 hold what one lane holds of a whole block: the same sums)
    f32x16 x;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      uint32_t lo = __float_as_uint(x16[r / 4][r % 4]), hi = lo;
      swap_halves(lo, hi);
      x[8 * (r / 4) + r % 4] = __uint_as_float(lo);
      x[8 * (r / 4) + 4 + r % 4] = __uint_as_float(hi);
    }
    const f32x2 v = sums(x);
    uint32_t s0 = __float_as_uint(v[0]), s1 = s0, q0 = __float_as_uint(v[1]), q1 = q0;
    swap_rows(s0, s1);
    swap_rows(q0, q1);
    if (tq == 0)
      stats[(NF * 32 + trow) * NS + s] = f32x2{__uint_as_float(s0) + __uint_as_float(s1), __uint_as_float(q0) + __uint_as_float(q1)};
  }
  lds_barrier();
  {
    const f32x16 gm = vec16(P_G2 + 32 * s), bt = vec16(P_B2N + 32 * s);
    const u32x4 b2 = bias(P_B2 + 32 * s);
    auto scale_shift = [&](int row) -> f32x2 {
      float su = 0.f, ss = 0.f;
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const f32x2 st = stats[row * NS + k];
        su += st[0];
        ss += st[1];
      }
      const float mu = su * (1.0f / C), var = fmaxf(ss * (1.0f / C) - mu * mu, 0.f);
      const float sc = rsqrtf(var + eps);
      return f32x2{sc, -mu * sc};
    };
    if constexpr (TAIL) {
      const f32x2 ssh = scale_shift(NF * 32 + trow);
      f32x4 z[2], g4[2], b4[2];
      vec4(g4, P_G2 + 32 * s);
      vec4(b4, P_B2N + 32 * s);
#pragma unroll
      for (int r = 0; r < 8; ++r) z[r / 4][r % 4] = fmaf(fmaf(x16[r / 4][r % 4], ssh[0], ssh[1]), g4[r / 4][r % 4], b4[r / 4][r % 4]);
      Ab[(NF * KS + s) * 64 + lane] = operand16(z);
#pragma unroll
      for (int t = 0; t < 2; ++t)
        x16[t] = mma16(u32x4{tq == 0 ? pack2(par[P_B2 + 32 * s + 16 * t + trow], 0.f) : 0u, 0u, 0u, 0u},
                       u32x4{tq == 0 ? kOnePair & 0xffffu : 0u, 0u, 0u, 0u}, x16[t]);
    }
#pragma unroll
    for (int b = 0; b < NQ; ++b) {
      const f32x2 ssh = scale_shift(b * 32 + nrow);
      const float sc = ssh[0], sh = ssh[1];
      f32x16 z;
#pragma unroll
      for (int r = 0; r < 16; ++r) z[r] = fmaf(fmaf(x1[b][r], sc, sh), gm[r], bt[r]);
#pragma unroll
      for (int k = 0; k < 2; ++k) Ab[(b * KS + 2 * s + k) * 64 + lane] = operand(z, k);
      x1[b] = mma(b2, first_one, x1[b]);
    }
  }
  lds_barrier();

  // ---- FFN -------------------------------------------------------------------------------------------------------
  // Two hidden tiles a wavefront: tile t of slice s is unit t NS + s.  GELU of a tile runs beside the products that come
  // after it: those of the second tile, and the first half of the second FFN product.
  {
    f32x16 acc[2][NQ];
    f32x4 acc16[2][2];
    auto gelu_part = [&](int t, int k) {   // of step k
      constexpr int ALL = 16 * NQ + (TAIL ? 8 : 0);
#pragma unroll
      for (int i = k * ALL / KS; i < (k + 1) * ALL / KS; ++i) {
        if (i < 16 * NQ) acc[t][i / 16][i % 16] = gelu2_fast(acc[t][i / 16][i % 16]);
        else acc16[t][(i - 16 * NQ) / 4][i % 4] = gelu2_fast(acc16[t][(i - 16 * NQ) / 4][i % 4]);
      }
    };
    auto put_hidden = [&](int t, u32x4* to) {
#pragma unroll
      for (int b = 0; b < NQ; ++b)
#pragma unroll
        for (int k = 0; k < 2; ++k) to[(b * KS + 2 * s + k) * 64 + lane] = operand(acc[t][b], k);
      if constexpr (TAIL) to[(NF * KS + s) * 64 + lane] = operand16(acc16[t]);
    };
    auto first = [&](int t) {
      const u32x4 b1 = bias(P_B1 + 32 * (t * NS + s));
#pragma unroll
      for (int b = 0; b < NQ; ++b) acc[t][b] = mma(b1, first_one, kZero);
      if constexpr (TAIL) vec4(acc16[t], P_B1 + 32 * (t * NS + s));
      return [&, t](const u32x4 (&w)[1], const u32x4 (&a)[NQ]) {
#pragma unroll
        for (int b = 0; b < NQ; ++b) acc[t][b] = mma(w[0], a[b], acc[t][b]);
      };
    };
    auto first16 = [&](int t) {
      return [&, t](const u32x4 (&w)[1][2], u32x4 a) {
#pragma unroll
        for (int e = 0; e < 2; ++e) acc16[t][e] = mma16(w[0][e], a, acc16[t][e]);
      };
    };
    product(w, wf, KS, Ab, first(0), first16(0), nothing);
    if constexpr (NQ <= 3) {
      product(w, wf, 2 * KS, Ab, first(1), first16(1), [&](int k) { gelu_part(0, k); });
      put_hidden(0, Bb);
    } else {                               // (no registers for two tiles)
#pragma unroll
      for (int k = 0; k < KS; ++k) gelu_part(0, k);
      put_hidden(0, Bb);
      product(w, wf, 2 * KS, Ab, first(1), first16(1), nothing);
    }
    lds_barrier();
    product(w, wf, 3 * KS, Bb, onto_x1, onto_x16, [&](int k) { gelu_part(1, k); });
    put_hidden(1, Ab);
    lds_barrier();
    product(w, wf, 4 * KS, Ab, onto_x1, onto_x16, nothing);
  }

  // ---- scatter -------------------------------------------------------------------------------------------------------
  u32x4* const Out = Bb;
  const int mine = SPLIT ? 32 * qb + s * RPWQ : slot0;  // slot of the first row I store
  if constexpr (!OUT_F32) {                // whole rows through LDS
    if constexpr (TAIL) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
        *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(Out + (32 * NF + trow) * LPR + ((4 * s + 2 * t + (tq >> 1)) ^ trow)) + 8 * (tq & 1)) =
            u32x2{pack2(x16[t][0], x16[t][1]), pack2(x16[t][2], x16[t][3])};
    }
#pragma unroll
    for (int b = 0; b < NQ; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(Out + (32 * b + nrow) * LPR + ((4 * s + e) ^ (nrow & 15))) + 8 * h) =
            u32x2{pack2(x1[b][4 * e], x1[b][4 * e + 1]), pack2(x1[b][4 * e + 2], x1[b][4 * e + 3])};
    lds_barrier();
#pragma unroll
    for (int t = 0; t < NLQ; ++t) {
      const int row = s * RPWQ + t * RPI + lr_out;
      const u32x4 v = Out[row * LPR + (lc_out ^ (row & 15))];
      if (mine + t * RPI + lr_out < m)  // non-temporal: the next reader is another XCD, and the kernel's end has less to write back
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(out) + (size_t)orow[t] * C + 8 * lc_out));
    }
  } else {                                 // output rows of all row blocks, through LDS; then 16 bytes a lane and piece
    int32_t* const rowof = reinterpret_cast<int32_t*>(Out);
    if (lc_out == 0) {
#pragma unroll
      for (int t = 0; t < NLQ; ++t) rowof[s * RPWQ + t * RPI + lr_out] = mine + t * RPI + lr_out < m ? orow[t] : -1;
    }
    lds_barrier();
    if constexpr (TAIL) {
      const int o = rowof[32 * NF + trow];
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (o >= 0) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out) + (size_t)o * C + 32 * s + 16 * t + 4 * tq) = x16[t];
    }
#pragma unroll
    for (int b = 0; b < NQ; ++b) {
      const int o = rowof[32 * b + nrow];
      if (o >= 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out) + (size_t)o * C + 32 * s + 8 * e + 4 * h) =
              f32x4{x1[b][4 * e], x1[b][4 * e + 1], x1[b][4 * e + 2], x1[b][4 * e + 3]};
      }
    }
  }
}

// Two and four row blocks, 128 features: two workgroups share a compute unit, 512 the chip, and a few groups more than that, or
// a few groups in all, have a compute unit each and leave the others idle.  Up to 128 of them are therefore taken by two workgroups
// each, half of the queries to each, which both make the keys and values of all: the same operations on every row.  Whole / so, us from
// a graph: G = 128, 64 groups 17.9 / 12.6, 128 18.0 / 13.0, 520 42.2 / 36.5, 626 43.0 / 38.2, 1100 68.6 / 64.1; G = 100 128 groups 17.9 / 13.0,
// 626 40.8 / 36.2; G = 64, 64 groups 9.6 / 7.7, 128 9.6 / 8.0; G = 40 9.3 / 7.7 and 9.4 / 8.2; with an embedding G = 128, 128 groups 19.0 /
// 14.3, G = 64 10.0 / 8.4; with float32 results 20.0 / 14.6 and 10.7 / 8.9.  (160 groups by halves 20.1 and, G = 64, 11.3, whole 19.8 and
// 11.0; 188 beyond a round 51 and 46: more than fit beside each other.)
constexpr bool can_split(int C, int PT, int MINW) { return C == 128 && (PT == 4 || (PT == 2 && MINW == 2)); }
constexpr int kSplitGroups = 128, kGroupsAtOnce = 512;

// SPLITS: of the launches in which some groups are split (the others are 0.5 us a launch faster without the code).
template <int C, int DH, int F, int PT, int GPW, bool HALF, int MINW, bool OUT_F32, bool PE, bool SPLITS>
__global__ __launch_bounds__(2 * C, MINW) void k_layer_slice(
    const uint16_t* __restrict__ feats, const int32_t* __restrict__ perm, const u32x4* __restrict__ packed, int n, int G,
    int in_sorted, int max_groups, const int32_t* __restrict__ goff, const int32_t* __restrict__ num_groups,
    const int32_t* __restrict__ out_index, void* __restrict__ out, const uint16_t* __restrict__ pos_embed, int drop, float eps) {
  if constexpr (SPLITS) {                  // (a group a workgroup: from the number of groups, which is in a register from the start)
    static_assert((kGroupsAtOnce & (kGroupsAtOnce - 1)) == 0, "whole rounds");
    const int unsplit = max_groups & ~(kGroupsAtOnce - 1), beyond = (int)blockIdx.x - unsplit;
    if (beyond >= 0) {
      slice_layer<C, DH, F, PT, GPW, HALF, MINW, OUT_F32, PE, true>(feats, perm, packed, n, G, in_sorted, max_groups, goff, num_groups,
                                                                    out_index, out, pos_embed, drop, eps, unsplit + beyond / 2, beyond & 1);
      return;
    }
  }
  slice_layer<C, DH, F, PT, GPW, HALF, MINW, OUT_F32, PE, false>(feats, perm, packed, n, G, in_sorted, max_groups, goff, num_groups,
                                                                 out_index, out, pos_embed, drop, eps, blockIdx.x, 0);
}

template <int C, int DH, int F, int PT, int GPW, bool HALF, int MINW>
int launch_cfg(const LayerSlice& c, hipStream_t stream) {
  constexpr int lds_bytes = Plan<C, F, PT * GPW, tail_of_16(PT, HALF)>::TOTAL;
  static_assert(lds_bytes <= kLdsBytes, "LDS");
  const ff_layer_weights* w = c.w;
  const int workgroups = (c.max_groups + GPW - 1) / GPW, left = workgroups % kGroupsAtOnce;
  // (An embedding that the results overwrite is read and written group by group, each by one workgroup.)
  const int split = can_split(C, PT, MINW) && left <= kSplitGroups && w->pos_embed != c.out ? left : 0;
  // The dynamic LDS size has to be allowed once per kernel and device.
  static std::atomic<uint64_t> allowed[8] = {};  // bit d: done on device d
  auto go = [&](auto kern, int which) -> int {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return FF_ERR_LAUNCH;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(allowed[which].load(std::memory_order_acquire) & bit)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                              lds_bytes) != hipSuccess)
        return FF_ERR_LAUNCH;
      allowed[which].fetch_or(bit, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(workgroups + split)), dim3(2 * C), lds_bytes, stream,
                       (const uint16_t*)c.feats, c.perm, (const u32x4*)c.packed, c.n, c.G, c.in_sorted, (int)c.max_groups,
                       c.group_offsets, c.num_groups, c.out_index, c.out, (const uint16_t*)w->pos_embed, c.drop ? 1 : 0,
                       w->ln_eps);
    return launch_status();
  };
  auto form = [&](auto splits) -> int {
    constexpr bool S = decltype(splits)::value;
    if (w->pos_embed)
      return c.out_f32 ? go(k_layer_slice<C, DH, F, PT, GPW, HALF, MINW, true, true, S>, 3 + 4 * S)
                       : go(k_layer_slice<C, DH, F, PT, GPW, HALF, MINW, false, true, S>, 2 + 4 * S);
    return c.out_f32 ? go(k_layer_slice<C, DH, F, PT, GPW, HALF, MINW, true, false, S>, 1 + 4 * S)
                     : go(k_layer_slice<C, DH, F, PT, GPW, HALF, MINW, false, false, S>, 0 + 4 * S);
  };
  if constexpr (can_split(C, PT, MINW))
    if (split > 0) return form(std::true_type());
  return form(std::false_type());
}

}  // namespace

int FF_LAYER_SYM(layer_slice_launch)(const LayerSlice& c, hipStream_t stream) {
  if (c.max_groups == 0 || c.n == 0) return FF_OK;
  const int G = c.G, blocks = c.blocks ? c.blocks : (G + 31) / 32;
  if (G > 32 * blocks) return FF_ERR_UNSUPPORTED;
#define FF_GO(C, DH, F, PT, GPW, MINW)                                                        \
  return G <= 32 * PT - 16 && !c.whole ? launch_cfg<C, DH, F, PT, GPW, true, MINW>(c, stream) \
                                       : launch_cfg<C, DH, F, PT, GPW, false, MINW>(c, stream)
  // Up to two workgroups a compute unit: as many registers as two wavefronts on a SIMD have; beyond, three share it (30,000
  // rows, G = 64: 13.9 / 14.2 us, 240,000 rows: 103 / 98).
  const bool few = c.waves ? c.waves == 2 : ceil_div(c.max_groups, G <= 32 ? 2 : 1) <= 512;
  switch (c.w->C * 8 + blocks) {
    case 128 * 8 + 1:
      if (few) FF_GO(128, 16, 256, 1, 2, 2);
      FF_GO(128, 16, 256, 1, 2, 3);
    case 128 * 8 + 2:
      if (few) FF_GO(128, 16, 256, 2, 1, 2);
      FF_GO(128, 16, 256, 2, 1, 3);
    case 128 * 8 + 3: FF_GO(128, 16, 256, 3, 1, 2);
    case 128 * 8 + 4: FF_GO(128, 16, 256, 4, 1, 2);
    case 256 * 8 + 1: FF_GO(256, 32, 512, 1, 2, 2);
    case 256 * 8 + 2: FF_GO(256, 32, 512, 2, 1, 2);
    case 256 * 8 + 3: FF_GO(256, 32, 512, 3, 1, 2);
    case 256 * 8 + 4: FF_GO(256, 32, 512, 4, 1, 2);
  }
#undef FF_GO
  return FF_ERR_UNSUPPORTED;
}

}  // namespace ff
