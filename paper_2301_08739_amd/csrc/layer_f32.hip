// Group attention layer (paper Sec. 4.2.2, Eq. (2)) in float32 as ONE fused kernel on the matrix cores of gfx950:
//
//   gather -> LN1 -> packed QKV projection -> per-head softmax(Q K^T / sqrt(d)) V -> out-proj
//   + residual -> LN2 -> Linear + GELU (erf) -> Linear + residual -> scatter
//
// Arithmetic.  The linear layers run on bfloat16 products without giving up float32: every operand is written as the
// sum of three bfloat16 numbers, x = hi + mid + lo, which is exact (3 x 8 significant bits), products of two such
// numbers are exact in float32, and the six products hi hi, hi mid, mid hi, mid mid, hi lo, lo hi are accumulated in
// float32.  What is left out (mid lo, lo mid, lo lo) is below 2^-23 of a product, the size of one float32 rounding.
// Six v_mfma_f32_32x32x16_bf16 take 192 cycles where eight v_mfma_f32_32x32x2_f32 take 512.  Scores and P V, a sixth of
// the products, use the float32 instructions as they are: splitting Q, K, V and P would cost more than it saves.
//
// Mapping.  A workgroup owns one group (two of at most 32 members when there are many): PT blocks of 32 rows.  Its C / 32
// wavefronts cut the FEATURES: wavefront s computes features 32 s .. 32 s + 31 of Q, K and V (whole heads: scores, softmax
// and P V stay inside a wavefront), of the output projection and of the second FFN product, and its share of the hidden
// units, for all rows.  A weight fragment is read by exactly one wavefront, straight from L2 into registers, and
// multiplies every row block; what goes round between the wavefronts are the activations (LN1 output, attention output,
// LN2 output, hidden units), split once by their producer and passed through LDS in operand order.
//
// A "fragment" is 32 rows x 16 inputs of one of the three parts, 1 KB, 16 bytes per lane (lane = 32 h + row).  Products
// are computed transposed, D[output feature][row]: lane (h, n) of a tile holds row n and features
// (r & 3) + 8 (r >> 2) + 4 h in registers r = 0..15.  Registers 8 f .. 8 f + 7, split, are an operand of a later product
// whose inputs are numbered in that order (the weights that meet them are permuted to match when they are packed), and
// register r as it stands is one k-step of a 32x32x2 product: K and Q feed S^T = K Q^T, V (operand roles swapped) and
// P = exp2(S^T) feed P V, nothing is shuffled between lanes.  So it is with heads of 32.  With heads of 16 half of a 32x32x2
// product of P V would be for rows that no one wants; there the products are 16x16x4, for which registers change lanes in
// pairs, once for K, Q and V and once for every output (permlane swaps, 2 for 128 numbers).  Row sums of P are added beside the
// products.  Against 32x32x2 products with the sums as rows of ones, us a layer: 30,000 rows at C = 128, G = 64 61.4 -> 59.6,
// 100,000 192 -> 183, 20,000 at C = 64, G = 64 40.4 -> 38.4; C = 256 (sums only) 172 -> 165; errors against float64 1 to 6 %
// smaller.  Four row blocks keep 144 to 340 bytes a lane in scratch with them and are the faster for it all the same: 30,000
// rows at C = 64, G = 128 76 -> 73, C = 128, G = 128 110 -> 109, with an embedding 133 -> 118, 120,000 rows 430 -> 421 and
// 489 -> 459; only C = 128, G = 120 without an embedding is behind, 112 -> 116 and 439 -> 448.  32x32x2 products with zeros
// for the other head's rows and the sums beside them need no scratch there and were slower (78, 111, 124, 434, 478, 115, 448).
//
// What bounds it: the matrix pipe, about 33k cycles per wavefront at C = 128, G = 64, two wavefronts per SIMD (30k rows:
// two groups on most compute units), and nearly as many issue cycles of GELU, exponentials, splits and LayerNorm beside
// it.  Measured, 30,000 rows at C = 128, G = 64: 60 us a layer = 148 TFLOP/s (the plain kernels: 455 us); 2,000 rows at
// C = 64, G = 32: 13 us (31 us).
#include "common.h"
#include "pack_weights.h"
#include <atomic>
#include <type_traits>

namespace ff {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

struct Split {  // one lane's share of a fragment: hi, mid, lo (direct form: the eight floats in p[0] and p[1])
  u32x4 p[3];
};

__device__ __forceinline__ uint32_t pack2(float a, float b) {  // round to nearest even
  const f32x2 f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf2));
}
// v[0..7] = hi + mid + lo, each eight bfloat16
__device__ __forceinline__ Split split8(const float* v) {
  Split s;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float a = v[2 * j], b = v[2 * j + 1];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const uint32_t u = pack2(a, b);
      s.p[k][j] = u;
      if (k < 2) { a -= __uint_as_float(u << 16); b -= __uint_as_float(u & 0xffff0000u); }
    }
  }
  return s;
}
// The same eight numbers as they are (direct form), and back.
__device__ __forceinline__ Split raw8(const float* v) {
  Split s;
#pragma unroll
  for (int j = 0; j < 8; ++j) s.p[j / 4][j % 4] = __float_as_uint(v[j]);
  s.p[2] = u32x4{0u, 0u, 0u, 0u};
  return s;
}
__device__ __forceinline__ float raw_at(const Split& s, int j) { return __uint_as_float(s.p[j / 4][j % 4]); }
// Number j of a split operand: the sum of its parts is exact, and infinite parts stand alone (split_part).
__device__ __forceinline__ float sum_at(const Split& s, int j) {
  auto part = [&](int k) {
    const uint32_t u = s.p[k][j / 2];
    return __uint_as_float(j % 2 ? u & 0xffff0000u : u << 16);
  };
  return part(0) + (part(1) + part(2));
}
__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}
// big += hi hi, small += the other five.  The products round towards zero at the size of what they add to: apart, only
// one in six of them meets the large sum.  For the same reason a sum starts from its bias and the residual is added to
// the finished sum.  Error of a layer against float64, 9,001 rows, C = 128, G = 64: mean 0.99e-7, largest 1.1e-6; with the
// residual as the first term 1.7e-7 and 3.7e-6; plain kernels 2.1e-7 and 3.1e-6.
__device__ __forceinline__ void mma(const Split& a, const Split& b, f32x16& big, f32x16& small) {
  small = mfma_bf16(a.p[2], b.p[0], small);
  small = mfma_bf16(a.p[0], b.p[2], small);
  small = mfma_bf16(a.p[1], b.p[1], small);
  big = mfma_bf16(a.p[0], b.p[0], big);
  small = mfma_bf16(a.p[1], b.p[0], small);
  small = mfma_bf16(a.p[0], b.p[1], small);
}
__device__ __forceinline__ f32x16 mma2(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ f32x4 mma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// Of the four rows of 16 lanes: a = a0 a1 a2 a3, b likewise -> a0 b0 a2 b2, a1 b1 a3 b3
__device__ __forceinline__ void swap_rows(float& a, float& b) {
  auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(t[0]); b = __uint_as_float(t[1]);
}
// -> a0 a1 b0 b1, a2 a3 b2 b3
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(t[0]); b = __uint_as_float(t[1]);
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
// Sum over LPR (4, 8, 16) neighbouring lanes.
template <int LPR> __device__ __forceinline__ float lane_sum(float v) {
  v += dpp<0xB1>(v);                            // quad_perm 1,0,3,2
  v += dpp<0x4E>(v);                            // quad_perm 2,3,0,1
  if constexpr (LPR >= 8) v += dpp<0x141>(v);   // row_half_mirror
  if constexpr (LPR >= 16) v += dpp<0x140>(v);  // row_mirror
  return v;
}

// GELU(v) = v Phi(v) = max(v, 0) - t Phi(-t), t = |v|, with Phi(-t) = 2^P(t) and P a polynomial fitted to the base-2
// logarithm of the Gaussian tail on [0, 6].  Beyond, it keeps falling to 2^-50 at t = 8.5, where t stops: what is left
// of the tail is below 1e-14 whatever v.  max(v, 0) is written (v + |v|) / 2, which keeps a NaN and has, like
// 0.5 v (1 + erf), no value at minus infinity.  Without branches: 13 vector operations and one exponential (erff: a
// branch and some 35).  Largest error 2.4e-7 over [-9, 9] and 2.2e-10 on [-9, -6]; 0.5 v (1 + erf) in float32 with erf
// rounded correctly: 4.5e-7 and 5.9e-9.
__device__ __forceinline__ float gelu(float v) {
  const float t = fminf(fabsf(v), 8.5f);
  float p = 4.41011849e-07f;
  p = fmaf(p, t, -8.55969938e-06f);
  p = fmaf(p, t, 6.93239272e-05f);
  p = fmaf(p, t, -2.67630414e-04f);
  p = fmaf(p, t, -1.29715954e-05f);
  p = fmaf(p, t, 6.95772702e-03f);
  p = fmaf(p, t, -5.24485335e-02f);
  p = fmaf(p, t, -4.59217966e-01f);
  p = fmaf(p, t, -1.15110457f);
  p = fmaf(p, t, -1.0f);
  return fmaf(-t, __builtin_amdgcn_exp2f(p), fmaf(0.5f, fabsf(v), 0.5f * v));
}

// Nothing is moved across by the instruction scheduler: it would sink loads issued ahead to where they are used.
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }
// Keeps products on their side of a fence: they have no side effects, and the compiler places such instructions freely
// before it comes to scheduling.
__device__ __forceinline__ void pin(f32x16& v) { asm volatile("" : "+v"(v)); }
// Workgroup barrier that waits for this wavefront's LDS operations only: weight fragments requested ahead stay in
// flight across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

struct Weights {
  const u32x4* packed;  // the four matrices, split and in fragment order (pack_weights.h)
  const float *ln1_g, *ln1_b, *b_qkv, *b_o, *ln2_g, *ln2_b, *b1, *b2;
};

constexpr int kLdsBytes = 160 * 1024;  // LDS of one compute unit

template <int C, int F, int PT>
struct Plan {
  static constexpr int NS = C / 32, NT = 64 * NS, R = 32 * PT;
  static constexpr int A = R * C * 6;          // LN1 output, then attention output, then LN2 output
  static constexpr int H = R * 16 * NS * 6;    // 16 hidden units of every wavefront
  static constexpr int STATS = R * NS * 8;
  static constexpr int PAR = (5 * C + F) * 4;  // query bias, output bias, LN2 scale and shift, FFN biases
  static constexpr int TOTAL = A + H + STATS + PAR;
};

// Returns, the same for every thread of the workgroup, whether some result is infinite or no number; nothing has been
// stored then.  DIRECT: the linear layers on float32 products of the numbers themselves, and the results are stored
// whatever they are.
//
// Why two forms: three parts cannot stand for an infinity (inf - inf is no number), for a number that rounds to one in
// bfloat16, or for what becomes infinite on the way (a hidden unit), and inf * hi + inf * mid is no number where inf * x
// is infinite.  Whatever of that happens in a row reaches all its results, as the products are dense and nothing on the
// way turns it into a number again, so one look at the results finds it.  The workgroup then starts over in the direct
// form, which gives infinities and NaNs where float32 arithmetic gives them.  The look takes half an instruction per result.
template <int C, int DH, int F, int PT, int GPW, bool PE, bool DIRECT>
__device__ __forceinline__ bool layer_f32_rows(
    const float* __restrict__ feats, float* __restrict__ out, const float* __restrict__ pos_embed,
    const int32_t* __restrict__ perm, const int32_t* __restrict__ goff, const int32_t* __restrict__ num_groups,
    int max_groups, int n, int G, const int32_t* __restrict__ out_index, int in_sorted, int drop, float eps,
    const Weights& wt, const int tid) {
  using PL = Plan<C, F, PT>;
  constexpr int NS = PL::NS, NT = PL::NT;
  constexpr int KS = C / 16;               // fragments along C
  constexpr int HT = F / 32 / NS;          // hidden tiles of a wavefront
  constexpr int PTG = PT / GPW;            // row blocks of a group
  constexpr int NH = 32 / DH;              // heads of a wavefront
  constexpr int PARTS = DIRECT ? 2 : 3;    // of an operand in LDS
  constexpr int LPR = C / 16, RPS = 64 / LPR;  // LN1: lanes per row (two runs of 8 features each), rows per step
  static_assert(DH == 16 || DH == 32, "head dim");
  static_assert(PT % GPW == 0 && HT == 2, "whole blocks, two hidden tiles per wavefront");

  extern __shared__ u32x4 lds[];
  u32x4* const Ab = lds;
  u32x4* const Hb = lds + PL::A / 16;
  char* const ldsc = reinterpret_cast<char*>(lds);
  f32x2* const stats = reinterpret_cast<f32x2*>(ldsc + PL::A + PL::H);
  float* const par = reinterpret_cast<float*>(ldsc + PL::A + PL::H + PL::STATS);
  constexpr int P_BQ = 0, P_BO = C, P_G2 = 2 * C, P_B2N = 3 * C, P_B2 = 4 * C, P_B1 = 5 * C;

  const int lane = tid & 63, nrow = lane & 31, h = lane >> 5;
  const int s = __builtin_amdgcn_readfirstlane(tid >> 6);  // slice

  // ---- weight stream of the slice: wave-uniform base, the lane's part of the address is a 32-bit offset -----------
  constexpr int SLICE_FR = 4 * KS + HT * KS + F / 16;
  const char* const wbase = reinterpret_cast<const char*>(wt.packed) + (size_t)s * SLICE_FR * 3072;
  const uint32_t lane16 = lane * 16;
  auto w_at = [&](int frag) -> Split {
    Split r;
#pragma unroll
    for (int k = 0; k < 3; ++k) r.p[k] = *reinterpret_cast<const u32x4*>(wbase + (frag * 3 + k) * 1024 + lane16);
    return r;
  };
  auto pack8 = [](const float* v) { return DIRECT ? raw8(v) : split8(v); };
  auto wq_at = [&](int which, int ks) { return w_at(which * KS + ks); };
  auto wo_at = [&](int ks) { return w_at(3 * KS + ks); };
  auto w1_at = [&](int t, int ks) { return w_at((4 + t) * KS + ks); };
  auto w2_at = [&](int u, int k) { return w_at((4 + HT) * KS + 2 * (k * HT + u / 2) + u % 2); };  // unit u of slice k

  // ---- which rows ----------------------------------------------------------------------------------------------------
  int start[GPW], m[GPW], end1[GPW];
  // Row `r` of the workgroup -> sorted position.  Rows beyond the group's members repeat its last member: their scores
  // then never exceed the real ones, and they are cut out of the sums below.
  auto position = [&](int r) -> int {
    const int gl = GPW == 1 ? 0 : r >> 5;
    const int sl = GPW == 1 ? r : r & 31;
    const int mm = GPW == 1 || gl == 0 ? m[0] : m[GPW - 1];
    const int st = GPW == 1 || gl == 0 ? start[0] : start[GPW - 1];
    const int last = mm > 0 ? mm - 1 : 0;
    return st + (sl < last ? sl : last);
  };
  // The same without the group list, right for groups that start at multiples of G (the first or only frame): what is
  // loaded with it does not wait for the list.
  auto guess = [&](int r) -> int {
    const int gl = GPW == 1 ? 0 : r >> 5;
    const int sl = GPW == 1 ? r : r & 31;
    const uint32_t g0 = (uint32_t)(blockIdx.x * GPW + gl) * (uint32_t)G;
    const uint32_t at = g0 + (uint32_t)(sl < G ? sl : G - 1);
    return (int)(at < (uint32_t)n ? at : (uint32_t)n - 1u);
  };
  // LN1 layout: LPR lanes share a row, wavefront s takes rows (s PT + t) RPS + lane / LPR, t < PT.
  const int lr = lane / LPR, lc = lane % LPR;
  int pil[PT];                             // pillar of my LN1 / store rows
  int xrow[PT];                            // row of feats of (row block, n): the residual
  f32x4 raw[PT][2][2];                     // features 8 (lc + LPR k) .. + 7 of my rows
  // Slots without a member, and all of them before the group list is there, meet entries of perm that need not name a row.
  auto pillar_at = [&](int p) -> int {
    const uint32_t i = (uint32_t)perm[p], last = (uint32_t)n - 1u;
    return (int)(i < last ? i : last);
  };
  auto fetch = [&](auto pos) {
#pragma unroll
    for (int t = 0; t < PT; ++t) pil[t] = pillar_at(pos((s * PT + t) * RPS + lr));
#pragma unroll
    for (int t = 0; t < PT; ++t) xrow[t] = in_sorted ? pos(32 * t + nrow) : pillar_at(pos(32 * t + nrow));
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int64_t row = in_sorted ? pos((s * PT + t) * RPS + lr) : pil[t];
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 2; ++e)
          raw[t][k][e] = *reinterpret_cast<const f32x4*>(feats + row * C + 8 * (lc + LPR * k) + 4 * e);
    }
  };
  fetch(guess);                            // before anything that waits
  // (Up to a workgroup a compute unit: two layers of 2,000 rows, C = 64, 31.0 -> 29.3 us.  Beyond, 768 KB of weights beside
  // the rows of all workgroups only delay these: four layers of 30,000 rows, C = 128, 235 us without and 239 with it.)
  uint32_t touched[2] = {0, 0};
  const int workgroups = (max_groups + GPW - 1) / GPW;
  if (workgroups <= 256) touch_lines<NT, NS * SLICE_FR * 3072>(wt.packed, workgroups, tid, touched);
  const int ngroups = *num_groups;
  bool all_guessed = true;
#pragma unroll
  for (int gl = 0; gl < GPW; ++gl) {
    const int g = blockIdx.x * GPW + gl;
    const int gc = g < max_groups ? g : max_groups - 1;
    const int o0 = goff[gc], o1 = goff[gc + 1];
    const bool valid = g < ngroups;
    start[gl] = valid ? o0 : 0;
    end1[gl] = o1;
    // A list of full groups only ('Drop Residual') has the next start beyond this group's end.
    m[gl] = valid ? (o1 - o0 < G ? o1 - o0 : G) : 0;
    all_guessed = all_guessed && (!valid || ((int64_t)g * G == o0 && (m[gl] == G || o0 + m[gl] == n)));
  }
  f32x4 gam[2][2], bet[2][2];              // LayerNorm 1 scale and shift of my features
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      gam[k][e] = *reinterpret_cast<const f32x4*>(wt.ln1_g + 8 * (lc + LPR * k) + 4 * e);
      bet[k][e] = *reinterpret_cast<const f32x4*>(wt.ln1_b + 8 * (lc + LPR * k) + 4 * e);
    }
  // The other vectors in the order of `par`, a column of it each thread (asked for together, written when the rows are there).
  static_assert(NT == 2 * C && F == NT && P_BO == C && P_G2 == NT && P_B2N == 3 * C && P_B2 == 2 * NT, "columns of 2 C");
  const bool low = tid < C;
  const int col = low ? tid : tid - C;
  const float par_at[4] = {(low ? wt.b_qkv : wt.b_o)[col], (low ? wt.ln2_g : wt.ln2_b)[col], wt.b2[col], wt.b1[tid]};
  const float bv = wt.b_qkv[2 * C + 32 * s + nrow];
  // The key bias shifts all scores of a query alike and drops out of the softmax, unless it is no finite number.
  const float bk = wt.b_qkv[C + 32 * s + nrow] * 0.f;
  if (!all_guessed) fetch(position);       // wave-uniform

  // ---- LN1 -> A (natural input order) ------------------------------------------------------------------------------
  Split wq0 = wq_at(PE ? 2 : 0, 0);        // first fragment of the first projection
  auto a_at = [&](int pt, int ks, int part) -> u32x4& { return Ab[((pt * KS + ks) * 3 + part) * 64 + lane]; };
  f32x4 pe[PE ? PT : 1][2][2];
  if constexpr (PE) {
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 2; ++e)
          pe[t][k][e] = *reinterpret_cast<const f32x4*>(pos_embed + (int64_t)pil[t] * C + 8 * (lc + LPR * k) + 4 * e);
  }
  // scale and shift the rows, and write them (plus the embedding) to A
  float y[PT][16];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    float su = 0.f, ss = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) { y[t][i] = raw[t][i / 8][i / 4 % 2][i % 4]; su += y[t][i]; }
    const float mu = lane_sum<LPR>(su) * (1.0f / C);
#pragma unroll
    for (int i = 0; i < 16; ++i) { const float d = y[t][i] - mu; ss = fmaf(d, d, ss); }
    const float rstd = 1.0f / sqrtf(lane_sum<LPR>(ss) * (1.0f / C) + eps);
#pragma unroll
    for (int i = 0; i < 16; ++i) y[t][i] = fmaf((y[t][i] - mu) * rstd, gam[i / 8][i / 4 % 2][i % 4], bet[i / 8][i / 4 % 2][i % 4]);
  }
  auto put_rows = [&](bool embed) {
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int row = (s * PT + t) * RPS + lr;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int p = lc + LPR * k;        // run of 8 features: fragment p / 2, half p & 1
        float z[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) z[i] = y[t][8 * k + i] + (PE && embed ? pe[PE ? t : 0][k][i / 4][i % 4] : 0.f);
        const Split sp = pack8(PE && embed ? z : &y[t][8 * k]);
#pragma unroll
        for (int part = 0; part < PARTS; ++part)
          Ab[(((row >> 5) * KS + (p >> 1)) * 3 + part) * 64 + (p & 1) * 32 + (row & 31)] = sp.p[part];
      }
    }
  };
  put_rows(false);
  par[tid] = par_at[0];
  par[P_G2 + tid] = par_at[1];
  if (low) par[P_B2 + tid] = par_at[2];
  par[P_B1 + tid] = par_at[3];
  touch_done(touched);

  // ---- rows of no group ('Drop Residual'): copied, unless there is no list -----------------------------------------
  if (drop && ngroups >= 0) {
    auto copy_rows = [&](int lo, int hi) {
      constexpr int PR = C / 4;            // 16-byte pieces per row
      hi = hi < n ? hi : n;
      for (int p = lo + tid / PR; p < hi; p += NT / PR) {
        const int pillar = perm[p];
        const f32x4 v = *reinterpret_cast<const f32x4*>(feats + (int64_t)(in_sorted ? p : pillar) * C + (tid % PR) * 4);
        *reinterpret_cast<f32x4*>(out + (int64_t)(out_index ? out_index[pillar] : pillar) * C + (tid % PR) * 4) = v;
      }
    };
#pragma unroll
    for (int gl = 0; gl < GPW; ++gl) {
      const int g = blockIdx.x * GPW + gl;
      if (g == 0) copy_rows(0, ngroups > 0 ? start[gl] : n);
      if (g < ngroups) copy_rows(start[gl] + m[gl], end1[gl]);
    }
  }

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
  const f32x16 kZero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto row_frags = [&](int pt, int ks) -> Split {
    Split a;
#pragma unroll
    for (int part = 0; part < PARTS; ++part) a.p[part] = a_at(pt, ks, part);
    return a;
  };

  // acc[pt] += W times the rows in A or H (swap: rows times W^T): DW sets of weights in flight (as many as cover a trip
  // to L2), the first one from the
  // caller; a block's rows are replaced as soon as its products are issued; `beside`: work of the vector units for every
  // step
  auto product_on = [&](f32x16 (&acc)[PT], f32x16 (&lo)[PT], Split w0, auto weight, auto rows, int steps, bool swap, auto beside) {
    if constexpr (DIRECT) {
#pragma unroll 1
      for (int k = 0; k < steps; ++k) {
        const Split w = weight(k);
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) {
          const Split a = rows(pt, k);
#pragma unroll
          for (int j = 0; j < 8; ++j)
            acc[pt] = swap ? mma2(raw_at(a, j), sum_at(w, j), acc[pt]) : mma2(sum_at(w, j), raw_at(a, j), acc[pt]);
        }
      }
#pragma unroll
      for (int k = 0; k < steps; ++k) beside(k);
      return;
    }
    constexpr int DW = PT == 1 ? 5 : 3;
    Split w[DW], a[PT];
    w[0] = w0;
#pragma unroll
    for (int d = 1; d < DW - 1; ++d)
      if (d < steps) w[d] = weight(d);
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) a[pt] = rows(pt, 0);
#pragma unroll
    for (int k = 0; k < steps; ++k) {
      fence();
      if (k + DW - 1 < steps) w[(k + DW - 1) % DW] = weight(k + DW - 1);
#pragma unroll
      for (int pt = 0; pt < PT; ++pt) {
        if (swap) mma(a[pt], w[k % DW], acc[pt], lo[pt]);
        else mma(w[k % DW], a[pt], acc[pt], lo[pt]);
        pin(acc[pt]);
        pin(lo[pt]);
        fence();
        if (k + 1 < steps) a[pt] = rows(pt, k + 1);
      }
      beside(k);
    }
    fence();
  };
  auto product = [&](f32x16 (&acc)[PT], Split w0, auto weight, auto rows, int steps, bool swap, auto beside) {
    f32x16 lo[PT];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) lo[pt] = kZero;
    product_on(acc, lo, w0, weight, rows, steps, swap, beside);
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) acc[pt] += lo[pt];
  };
  auto nothing = [](int) {};

  // ---- Q, K, V of this slice -----------------------------------------------------------------------------------------
  f32x16 Q[PT], K[PT], V[PT];
  lds_barrier();
  {
    const f32x16 bq = vec16(P_BQ + 32 * s);
    const float k0 = __builtin_amdgcn_ballot_w64(bk != 0.f) ? __builtin_nanf("") : 0.f;
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) { Q[pt] = bq; K[pt] = kZero + k0; V[pt] = kZero; }
    // One after the other (both sums of all three would not fit the registers).
    if constexpr (PE) {  // values from LN(F), queries and keys from LN(F) + PE
      product(V, wq0, [&](int ks) { return wq_at(2, ks); }, row_frags, KS, true, nothing);
      wq0 = wq_at(0, 0);
      lds_barrier();
      put_rows(true);
      lds_barrier();
    }
    product(Q, wq0, [&](int ks) { return wq_at(0, ks); }, row_frags, KS, false, nothing);
    asm volatile("" ::: "memory");         // (operands are read again instead of kept in registers)
    product(K, wq_at(1, 0), [&](int ks) { return wq_at(1, ks); }, row_frags, KS, false, nothing);
    if constexpr (!PE) {
      asm volatile("" ::: "memory");
      product(V, wq_at(2, 0), [&](int ks) { return wq_at(2, ks); }, row_frags, KS, true, nothing);
    }
    lds_barrier();                         // A has been read: the attention output goes there
  }
  constexpr float qscale = (DH == 16 ? 0.25f : 0.17677669529663687f) * 1.44269504088896340736f;  // log2(e) / sqrt(d)
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) {
    Q[pt] *= qscale;
    V[pt] += bv;
  }

  // ---- attention -----------------------------------------------------------------------------------------------------
  // SHORT: some group of the workgroup has fewer members than its blocks hold; the rows beyond them are cut out of P V
  // by clearing them in the A operand, and out of the row sums.
  Split wo0 = wo_at(0);
  auto attention = [&](auto shortc) {
    constexpr bool SHORT = decltype(shortc)::value;
    // Whether row `key` of group gl is one of its members
    auto in = [&](int gl, int key) { return !SHORT || key < m[gl]; };
    // o: the lane's share of a fragment of A
    auto put_head = [&](int qt, int frag, const float* o) {
      const Split sp = pack8(o);
#pragma unroll
      for (int part = 0; part < PARTS; ++part) a_at(qt, frag, part) = sp.p[part];
    };
    if constexpr (NH == 2) {
      // Heads of 16: products of 16 x 16, lane (g, i) = 16 g + i.  Two registers of K and Q, features f and f + 1 of rows
      // (h, n), become the operands of rows 0 .. 15 and 16 .. 31; two of V, rows r and r + 8 of both heads, those of the
      // heads, with row 16 b + 4 g + r in lane group g as the scores have it.
#pragma unroll
      for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          float a = Q[pt][2 * r], b = Q[pt][2 * r + 1];
          swap_rows(a, b);
          Q[pt][2 * r] = a; Q[pt][2 * r + 1] = b;
          a = K[pt][2 * r]; b = K[pt][2 * r + 1];
          swap_rows(a, b);
          K[pt][2 * r] = a; K[pt][2 * r + 1] = b;
          const int v = 8 * (r / 4) + r % 4;
          a = V[pt][v]; b = V[pt][v + 4];
          swap_halves(a, b);
          swap_rows(a, b);
          const bool real = in(pt / PTG, 32 * (pt % PTG) + 16 * (r / 4) + 4 * (lane >> 4) + r % 4);
          V[pt][v] = real ? a : 0.f; V[pt][v + 4] = real ? b : 0.f;
        }
#pragma unroll
      for (int gl = 0; gl < GPW; ++gl)
#pragma unroll
        for (int hd = 0; hd < 2; ++hd)
#pragma unroll
          for (int q0 = 0; q0 < PTG; ++q0) {
            const int qt = gl * PTG + q0;
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            f32x4 S[PTG][2][2], O[2] = {zero, zero};
#pragma unroll
            for (int kt = 0; kt < PTG; ++kt) {
#pragma unroll
              for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                  for (int q = 0; q < 2; ++q)
                    S[kt][b][q] = mma4(K[gl * PTG + kt][8 * hd + 2 * r + b], Q[qt][8 * hd + 2 * r + q], r ? S[kt][b][q] : zero);
            }
            float mx[2] = {S[0][0][0][0], S[0][0][1][0]}, sum[2] = {0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < PTG; ++kt)
#pragma unroll
              for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int q = 0; q < 2; ++q) mx[q] = fmaxf(mx[q], S[kt][i / 4][q][i % 4]);
            swap_rows(mx[0], mx[1]);
            mx[0] = mx[1] = half_max(fmaxf(mx[0], mx[1]));
            swap_rows(mx[0], mx[1]);
#pragma unroll
            for (int kt = 0; kt < PTG; ++kt)
#pragma unroll
              for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                  const float p = __builtin_amdgcn_exp2f(S[kt][i / 4][q][i % 4] - mx[q]);
                  O[q] = mma4(V[gl * PTG + kt][8 * (i / 4) + 4 * hd + i % 4], p, O[q]);
                  sum[q] += in(gl, 32 * kt + 16 * (i / 4) + 4 * (lane >> 4) + i % 4) ? p : 0.f;
                }
            // back to lanes (h, n)
            swap_rows(sum[0], sum[1]);
            const float inv = 1.0f / half_sum(sum[0] + sum[1]);
            float o[8];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float a = O[0][r], b = O[1][r];
              swap_rows(a, b);
              swap_halves(a, b);
              o[r] = a * inv;
              o[4 + r] = b * inv;
            }
            put_head(qt, 2 * s + hd, o);
          }
    } else {
#pragma unroll
      for (int gl = 0; gl < GPW; ++gl) {
        f32x16 va[PTG];
#pragma unroll
        for (int kt = 0; kt < PTG; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            va[kt][r] = in(gl, 32 * kt + (r & 3) + 8 * (r >> 2) + 4 * h) ? V[gl * PTG + kt][r] : 0.f;
#pragma unroll
        for (int q0 = 0; q0 < PTG; ++q0) {
          const int qt = gl * PTG + q0;
          f32x16 S[PTG], O = kZero;
#pragma unroll
          for (int kt = 0; kt < PTG; ++kt) {
            S[kt] = kZero;
#pragma unroll
            for (int r = 0; r < 16; ++r) S[kt] = mma2(K[gl * PTG + kt][r], Q[qt][r], S[kt]);
          }
          float mx = S[0][0], sum[2] = {0.f, 0.f};
#pragma unroll
          for (int kt = 0; kt < PTG; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S[kt][r]);
          mx = half_max(mx);
#pragma unroll
          for (int kt = 0; kt < PTG; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const float p = __builtin_amdgcn_exp2f(S[kt][r] - mx);
              O = mma2(va[kt][r], p, O);
              sum[r % 2] += in(gl, 32 * kt + (r & 3) + 8 * (r >> 2) + 4 * h) ? p : 0.f;
            }
          const float inv = 1.0f / half_sum(sum[0] + sum[1]);
#pragma unroll
          for (int f = 0; f < 2; ++f) {
            float o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = O[8 * f + j] * inv;
            put_head(qt, 2 * s + f, o);
          }
        }
      }
    }
  };
  {
    bool whole = true;
#pragma unroll
    for (int gl = 0; gl < GPW; ++gl) whole = whole && m[gl] == 32 * PTG;
    if (!DIRECT && whole) attention(std::false_type());
    else attention(std::true_type());
  }

  // ---- output projection + residual ----------------------------------------------------------------------------------
  f32x16 x1[PT];                           // residual stream of (my 32 features, all rows)
#pragma unroll
  for (int pt = 0; pt < PT; ++pt)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(feats + (int64_t)xrow[pt] * C + 32 * s + 8 * b + 4 * h);
#pragma unroll
      for (int j = 0; j < 4; ++j) x1[pt][4 * b + j] = v[j];
    }
  lds_barrier();
  {
    const f32x16 bo = vec16(P_BO + 32 * s);
    f32x16 o[PT];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) o[pt] = bo;
    product(o, wo0, wo_at, row_frags, KS, false, nothing);
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) x1[pt] += o[pt];
  }
  int orow[PT];                            // rows of `out` of my LN1 / store rows
#pragma unroll
  for (int t = 0; t < PT; ++t) orow[t] = out_index ? out_index[pil[t]] : pil[t];

  // ---- LN2 -> A (accumulator order) ------------------------------------------------------------------------------
  // Statistics of a row: every wavefront's 32 features (sum, and sum of squares about the slice's own mean), combined
  // through LDS.
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) {
    float su = 0.f, ss = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) su += x1[pt][r];
    su = half_sum(su);
    const float mu = su * (1.0f / 32);
#pragma unroll
    for (int r = 0; r < 16; ++r) { const float d = x1[pt][r] - mu; ss = fmaf(d, d, ss); }
    ss = half_sum(ss);
    if (h == 0) stats[(pt * 32 + nrow) * NS + s] = f32x2{su, ss};
  }
  Split w10 = w1_at(0, 0);
  lds_barrier();
  {
    const f32x16 gm = vec16(P_G2 + 32 * s), bt = vec16(P_B2N + 32 * s);
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
      f32x2 st[NS];
      float su = 0.f, ss = 0.f;
#pragma unroll
      for (int k = 0; k < NS; ++k) { st[k] = stats[(pt * 32 + nrow) * NS + k]; su += st[k][0]; ss += st[k][1]; }
      const float mu = su * (1.0f / C);
#pragma unroll
      for (int k = 0; k < NS; ++k) { const float d = st[k][0] * (1.0f / 32) - mu; ss = fmaf(32.f * d, d, ss); }
      const float rstd = 1.0f / sqrtf(ss * (1.0f / C) + eps);
      float z[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) z[r] = fmaf((x1[pt][r] - mu) * rstd, gm[r], bt[r]);
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const Split sp = pack8(z + 8 * f);
#pragma unroll
        for (int part = 0; part < PARTS; ++part) a_at(pt, 2 * s + f, part) = sp.p[part];
      }
    }
  }
  lds_barrier();

  // ---- FFN -------------------------------------------------------------------------------------------------------
  // The hidden units go round 16 per wavefront at a time (unit u: half u % 2 of hidden tile u / 2).  GELU of what comes
  // next runs beside products where there are some.
  auto gelu_part = [&](f32x16 (&acc)[PT], int i0, int i1) {
#pragma unroll
    for (int i = i0; i < i1; ++i) acc[i / 16][i % 16] = gelu(acc[i / 16][i % 16]);
  };
  auto put_unit = [&](f32x16 (&acc)[PT], int f) {
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = acc[pt][8 * f + j];
      const Split sp = pack8(v);
#pragma unroll
      for (int part = 0; part < PARTS; ++part) Hb[((pt * NS + s) * 3 + part) * 64 + lane] = sp.p[part];
    }
  };
  auto h_frags = [&](int pt, int k) -> Split {
    Split b;
#pragma unroll
    for (int part = 0; part < PARTS; ++part) b.p[part] = Hb[((pt * NS + k) * 3 + part) * 64 + lane];
    return b;
  };
  {
    f32x16 acc[2][PT];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f32x16 b1 = vec16(P_B1 + 32 * (s * HT + t));
#pragma unroll
      for (int pt = 0; pt < PT; ++pt) acc[t][pt] = b1;
    }
    product(acc[0], w10, [&](int ks) { return w1_at(0, ks); }, row_frags, KS, false, nothing);
    asm volatile("" ::: "memory");         // (the second tile reads its operands again instead of keeping them in registers)
    product(acc[1], w1_at(1, 0), [&](int ks) { return w1_at(1, ks); }, row_frags, KS, false,
            [&](int k) { gelu_part(acc[0], k * PT * 16 / KS, (k + 1) * PT * 16 / KS); });
    f32x16 y2[PT], y2lo[PT];               // both sums go on over the four units
    const f32x16 b2 = vec16(P_B2 + 32 * s);
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) { y2[pt] = b2; y2lo[pt] = kZero; }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const Split w20 = w2_at(u, 0);
      if (u > 0) lds_barrier();            // the unit before has been read
      put_unit(acc[u / 2], u % 2);
      lds_barrier();
      product_on(y2, y2lo, w20, [&](int k) { return w2_at(u, k); }, h_frags, NS, false, [&](int k) {
        if (u < 2) gelu_part(acc[1], (u * NS + k) * PT * 8 / NS, (u * NS + k + 1) * PT * 8 / NS);
      });
    }
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) x1[pt] += y2[pt] + y2lo[pt];
  }

  uint32_t* const unfit = reinterpret_cast<uint32_t*>(stats);  // per wavefront: some result is no finite number
  if constexpr (!DIRECT) {
    float z[2] = {0.f, 0.f};               // largest magnitude, NaN where there is one
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
      if (m[pt / PTG] > 0) {               // (a group past the last one divides by its empty row sums)
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r / 2 % 2] = __builtin_elementwise_maximum(z[r / 2 % 2], fabsf(x1[pt][r]));
      }
    const uint64_t any = __builtin_amdgcn_ballot_w64(!(__builtin_elementwise_maximum(z[0], z[1]) < __builtin_inff()));
    if (lane == 0) unfit[s] = any != 0;
  }

  // ---- scatter: whole rows through LDS (16-byte pieces swizzled by row), over A, which is free --------------------
#pragma unroll
  for (int pt = 0; pt < PT; ++pt)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int row = 32 * pt + nrow, p = 8 * s + 2 * b + h;
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = x1[pt][4 * b + j];
      *reinterpret_cast<f32x4*>(ldsc + row * (C * 4) + ((p ^ (row & 15)) * 16)) = v;
    }
  lds_barrier();
  const uint32_t over = DIRECT ? 0 : unfit[lane % NS];
  f32x4 v[PT][4];                          // read beside the flags
#pragma unroll
  for (int t = 0; t < PT; ++t)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int row = (s * PT + t) * RPS + lr, p = lc + LPR * k;
      v[t][k] = *reinterpret_cast<const f32x4*>(ldsc + row * (C * 4) + ((p ^ (row & 15)) * 16));
    }
  fence();
  if (!DIRECT && __builtin_amdgcn_ballot_w64(over != 0)) return true;
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int row = (s * PT + t) * RPS + lr;
    const int gl = GPW == 1 ? 0 : row >> 5, sl = GPW == 1 ? row : row & 31;
    if (sl < (GPW == 1 || gl == 0 ? m[0] : m[GPW - 1])) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int p = lc + LPR * k;
        // non-temporal: the next reader is another XCD, and the kernel's end has less to write back
        __builtin_nontemporal_store(v[t][k], reinterpret_cast<f32x4*>(out + (size_t)orow[t] * C + p * 4));
      }
    }
  }
  return false;
}

// What the second form uses of the first form's inputs is read again: kept, it would take registers from the first.
template <typename T> __device__ __forceinline__ T* again(T* p) {
  asm volatile("" : "+s"(p));
  return p;
}

template <int C, int DH, int F, int PT, int GPW, int MINW, bool PE>
__global__ __launch_bounds__(2 * C, MINW) void k_layer_f32(
    const float* __restrict__ feats, const int32_t* __restrict__ perm, int n, int G, int in_sorted, int max_groups,
    const int32_t* __restrict__ goff, const int32_t* __restrict__ num_groups, const int32_t* __restrict__ out_index,
    float* __restrict__ out, const float* __restrict__ pos_embed, int drop, float eps, Weights wt) {
  if (!layer_f32_rows<C, DH, F, PT, GPW, PE, false>(feats, out, pos_embed, perm, goff, num_groups, max_groups, n, G,
                                                    out_index, in_sorted, drop, eps, wt, threadIdx.x))
    return;
  lds_barrier();                           // every wavefront has read what made it start over
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const Weights w2{again(wt.packed), again(wt.ln1_g), again(wt.ln1_b), again(wt.b_qkv), again(wt.b_o),
                   again(wt.ln2_g), again(wt.ln2_b), again(wt.b1), again(wt.b2)};
  layer_f32_rows<C, DH, F, PT, GPW, PE, true>(again(feats), again(out), again(pos_embed), again(perm), again(goff),
                                              again(num_groups), max_groups, n, G, again(out_index), in_sorted, 0, eps,
                                              w2, tid);
}

template <int C, int DH, int F, int PT, int GPW, int MINW>
int launch_cfg(const LayerF32& c, hipStream_t stream) {
  constexpr int lds_bytes = Plan<C, F, PT>::TOTAL;
  static_assert(lds_bytes <= kLdsBytes, "LDS");
  static_assert(Plan<C, F, PT>::R * C * 4 <= Plan<C, F, PT>::A, "rows on their way out");
  const ff_layer_weights* w = c.w;
  const Weights wt{static_cast<const u32x4*>(c.packed), (const float*)w->ln1_g, (const float*)w->ln1_b,
                   (const float*)w->b_qkv, (const float*)w->b_o, (const float*)w->ln2_g, (const float*)w->ln2_b,
                   (const float*)w->b1, (const float*)w->b2};
  // The dynamic LDS size has to be allowed once per kernel and device.
  static std::atomic<uint64_t> allowed[2] = {{0}, {0}};  // bit d: done on device d
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
    hipLaunchKernelGGL(kern, dim3((unsigned)((c.max_groups + GPW - 1) / GPW)), dim3(2 * C), lds_bytes, stream,
                       (const float*)c.feats, c.perm, c.n, c.G, c.in_sorted, (int)c.max_groups, c.group_offsets, c.num_groups,
                       c.out_index, (float*)c.out, (const float*)w->pos_embed, c.drop ? 1 : 0, w->ln_eps, wt);
    return launch_status();
  };
  if (w->pos_embed) return go(k_layer_f32<C, DH, F, PT, GPW, MINW, true>, 1);
  return go(k_layer_f32<C, DH, F, PT, GPW, MINW, false>, 0);
}

__global__ __launch_bounds__(256) void k_pack_f32(PackBatch pb, int C, int F, int total_frags) {
  pack_weights_f32_thread(pb, blockIdx.y, (int)(blockIdx.x * 256 + threadIdx.x), C, F, total_frags);
}

}  // namespace

// (C, head dim, F) = (64, 16, 128), (128, 16, 256) and (256, 32, 512), whose rows fit the LDS: G <= 128, at C = 256
// G <= 64.
bool layer_f32_supported(const ff_layer_weights* w, int G) {
  const int C = w->C, F = w->F, d = C / w->heads;
  if (C == 256) return d == 32 && F == 512 && G <= 64;
  return ((C == 128 && F == 256) || (C == 64 && F == 128)) && d == 16 && G <= 128;
}

// Groups beyond 64 members take three or four row blocks and with them a wavefront per SIMD: a launch lasts as long as one
// such workgroup however few there are (C = 64: 53 and 77 us, C = 128: 77 and 108 us), while the plain kernels' time grows
// with the rows.  Below the lines here they are ahead.  Measured, us a call of fused / plain, G = 69 and 96, 100 and 128:
//   C = 64   3,000 rows 54 / 45   53 / 54   77 / 55    77 / 63      C = 128   1,000 rows 77 / 53   77 / 62   109 / 63   109 / 71
//            4,500      54 / 53   53 / 60   78 / 63    77 / 71                2,000      78 / 65   77 / 73   109 / 75   108 / 83
//            6,000      54 / 56   53 / 64   78 / 67    77 / 74                3,000      77 / 80   77 / 87   109 / 89   108 / 97
//            8,300      54 / 83   54 / 89   78 / 93    77 / 101               4,500      77 / 111  77 / 116  110 / 119  109 / 128
// Blocks of four layers (the weights split beside the sort) turn at about nine tenths of these rows.
bool layer_f32_pays(const ff_layer_weights* w, int G, int64_t n) {
  if (G <= 64) return true;
  const bool three = G <= 96;
  const int beyond = G - (three ? 65 : 97);
  return w->C == 64 ? n >= (three ? 5120 : 8448) - 70 * beyond : n >= (three ? 2944 : 4096) - 18 * beyond;
}

size_t layer_f32_packed_bytes(const ff_layer_weights* w) { return (size_t)pack_frag_count_f32(w->C, w->F) * 3072; }

int layer_f32_pack(const ff_layer_weights* w, void* packed, hipStream_t stream) {
  PackJob job;
  make_pack_job(w, 1, packed, 0, kPackF32, &job);
  hipLaunchKernelGGL(k_pack_f32, dim3((unsigned)job.blocks), dim3(256), 0, stream, job.pb, job.C, job.F, job.total_frags);
  return launch_status();
}

int layer_f32_launch(const LayerF32& c, hipStream_t stream) {
  if (c.max_groups == 0 || c.n == 0) return FF_OK;
  const int G = c.G;
  // G <= 32: a workgroup per group while all of them run at once (three wavefronts per SIMD on 256 compute units); two
  // groups share the weight stream otherwise (it would be what bounds a launch of many: 3 KB per 192 cycles of products
  // and wavefront).  Measured, G = 32, us a call with one group / two groups per workgroup:
  //   C = 64    512 groups 22 / 25   768 23 / 34   1,024 24 / 34   1,536 32 / 37   2,048 46 / 51   6,000 117 / 111
  //   C = 128   400 groups 33 / 34   600 45 / 52     768 51 / 52     850 61 / 53   1,536 93 / 84   6,000 339 / 307
  // C = 256 has the form with two groups only.
  const bool few = c.max_groups <= 256 * 12 * 32 / c.w->C;
  // (Three wavefronts per SIMD have to be asked for: the direct form alone would take two registers too many.)
  switch (c.w->C) {
    case 64:
      if (G <= 32 && few) return launch_cfg<64, 16, 128, 1, 1, 3>(c, stream);
      if (G <= 32) return launch_cfg<64, 16, 128, 2, 2, 2>(c, stream);
      if (G <= 64) return launch_cfg<64, 16, 128, 2, 1, 2>(c, stream);
      if (G <= 96) return launch_cfg<64, 16, 128, 3, 1, 1>(c, stream);
      return launch_cfg<64, 16, 128, 4, 1, 1>(c, stream);
    case 128:
      if (G <= 32 && few) return launch_cfg<128, 16, 256, 1, 1, 3>(c, stream);
      if (G <= 32) return launch_cfg<128, 16, 256, 2, 2, 2>(c, stream);
      if (G <= 64) return launch_cfg<128, 16, 256, 2, 1, 2>(c, stream);
      if (G <= 96) return launch_cfg<128, 16, 256, 3, 1, 1>(c, stream);
      return launch_cfg<128, 16, 256, 4, 1, 1>(c, stream);
    case 256:
      if (G <= 32) return launch_cfg<256, 32, 512, 2, 2, 2>(c, stream);
      return launch_cfg<256, 32, 512, 2, 1, 2>(c, stream);
  }
  return FF_ERR_UNSUPPORTED;
}

}  // namespace ff
