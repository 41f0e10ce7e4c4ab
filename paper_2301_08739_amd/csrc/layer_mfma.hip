// Group attention layer (paper Sec. 4.2.2, Eq. (2); Sec. 4.3 'Efficient MHSA' / 'Efficient FFN') in 16-bit storage at 64
// features as ONE fused kernel on the matrix cores of gfx950 (128 and 256 features: layer_slice.hip; this file chooses):
//
//   gather -> LN1 -> packed QKV projection -> per-head softmax(Q K^T / sqrt(d)) V -> out-proj
//   + residual -> LN2 -> Linear + GELU -> Linear + residual -> scatter
//
// Scores, probabilities, Q/K/V and the FFN hidden activations never leave the chip.
//
// Mapping.  A wavefront owns 16 pillars of one group ("its" pillars); WPG wavefronts
// share a group, NW wavefronts form a workgroup.  Everything is computed transposed, features x
// pillars, with v_mfma_f32_16x16x32_bf16: the weight tile is the A operand (16 output features x
// 32 inputs), the activations of 16 pillars are the B operand, and the accumulator holds
// D[feature 4q+j][pillar i] in lane (i = lane & 15, q = lane >> 4).  That accumulator layout is,
// after conversion to bf16, directly a B operand of the next product whose 8 k-slots in lane q
// are inputs {4q..4q+3} of two consecutive 16-blocks; weights are pre-permuted along k to match
// (pack kernel below), so activations chain from product to product in registers without any
// LDS round trip.  V is produced with the operand roles swapped (pillars x features), which is
// exactly the A operand P*V needs.  LayerNorm statistics and the softmax need only a reduction
// over the four lanes that share a pillar.
//
// Weights reach the matrix cores through LDS.  The packed stream is cut into 8 KB chunks that the
// workgroup copies asynchronously (global memory -> LDS, no registers) into a ring of as many slots
// as the LDS holds; slots are refilled only at workgroup barriers (one per head-dim unit, where the
// group's K and V are exchanged anyway, and a few in the FFN).  Every wavefront reads the fragments
// in stream order through a window of 8 fragments in registers, requested 8 products ahead of
// their use, so that LDS latency is hidden behind the matrix cores.
#include "common.h"
#include "elem16.h"
#include "pack_weights.h"
#include <atomic>

namespace ff {
namespace {

// Reductions over the 4 lanes that share a pillar (lane, lane^16, lane^32, lane^48), on the
// vector ALU: v_permlane16_swap / v_permlane32_swap with both operands equal to v return the
// pair (v from the even half, v from the odd half) in every lane.
__device__ __forceinline__ float quad_sum(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float quad_max(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ f32x4 mfma32(const Frag8& a, const Frag8& b, f32x4 c) {
#ifdef FF_LAYER_F16
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a.v, b.v, c, 0, 0, 0);
#else
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
#endif
}
// The k = 16 product takes no accumulator: it can only START a chain, from zero.  A k = 16 product issued right
// behind a k = 32 product that writes the accumulator it reads has been seen to read the old value on this chip,
// so every product that continues a chain goes through mfma32 (an odd 16-wide block multiplies zeros in its
// upper half), and this signature keeps a chained k = 16 call from compiling.
__device__ __forceinline__ f32x4 mfma16_from_zero(const Frag4& a, const Frag4& b) {
  const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#ifdef FF_LAYER_F16
  return __builtin_amdgcn_mfma_f32_16x16x16f16(a.v, b.v, z, 0, 0, 0);
#else
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.v, b.v, z, 0, 0, 0);
#endif
}
// Number of 1 KB fragments of the packed weight stream of one layer.
__host__ __device__ constexpr int frags_per_hp(int C) { return 6 * (C / 32) + C / 16; }
__host__ __device__ constexpr int frags_per_fc(int C) { return 2 * (C / 32) + C / 16; }

// ---- weight packing (pack_weights.h) as a kernel of its own: grid (blocks per layer, layers) -----------
#ifdef FF_LAYER_F16
constexpr bool kHalf = true;
#else
constexpr bool kHalf = false;
#endif
__global__ __launch_bounds__(256) void k_pack_weights(PackBatch pb, int C, int F, int total_frags) {
  pack_weights_thread<kHalf>(pb, blockIdx.y, (int)(blockIdx.x * 256 + threadIdx.x), C, F, total_frags);
}

// ---- the fused layer ------------------------------------------------------------------------------
constexpr int C = 64, F = 128, DH = 16;  // features, hidden units, head dimension
// LDS map (bytes): [weight ring RING x 16 KB][small parameters as fp32: (7C + F) x 4][K/V exchange, 2 buffers].
struct ParamOff {  // float offsets inside the small-parameter area
  static constexpr int LN1G = 0, LN1B = C, BQ = 2 * C, BO = 3 * C, LN2G = 4 * C, LN2B = 5 * C, B2 = 6 * C,
                       B1 = 7 * C, TOTAL = 7 * C + F;
};

// Fragments per staged chunk: a hidden unit is 8 fragments (units are whole chunks).
constexpr int kChunkFrags = 8;
constexpr int kLdsBytes = 160 * 1024;  // LDS of one compute unit
constexpr int kComputeUnits = 256;      // of an MI355X
constexpr int kWindow = 8;             // weight fragments a wavefront keeps in flight (LDS -> registers)

template <int WPG, int NW, int MINW>
struct LdsPlan {
  static constexpr int GPW = NW / WPG;
  static constexpr int WGS = (MINW * 4 / NW) > 1 ? (MINW * 4 / NW) : 1;  // workgroups meant to share a compute unit
  static constexpr int PARAMS = pack_param_bytes(C, F);   // padded to whole 1 KB pieces
  static constexpr int KVX_ONE = 2 * 2 * WPG * 64 * 8;    // K and V of one group, one unit
  static constexpr int KVX = 2 * GPW * KVX_ONE;           // double buffered
  static constexpr int NCHUNK = ((C / 32) * (6 * (C / 32) + C / 16) + (F / 32) * (2 * (C / 32) + C / 16)) / kChunkFrags;
  static constexpr int FIT = (kLdsBytes / WGS - PARAMS - KVX) / (kChunkFrags * 1024);
  static constexpr int RING = FIT < NCHUNK ? FIT : NCHUNK;
  static constexpr int TOTAL = RING * kChunkFrags * 1024 + PARAMS + KVX;
  static_assert(RING >= 2, "weight ring");
};

template <int WPG, int NW, int MINW, bool OUT_F32, bool PE>
__global__ __launch_bounds__(NW * 64, MINW) void k_layer_mfma(
    const uint16_t* __restrict__ feats, const int32_t* __restrict__ perm, const u32x4* __restrict__ packed, int n, int G,
    int in_sorted, int max_groups, const int32_t* __restrict__ goff, const int32_t* __restrict__ num_groups,
    const int32_t* __restrict__ out_index, void* __restrict__ out, const uint16_t* __restrict__ pos_embed, int drop, float eps) {
  constexpr int KB = C / 32;          // 32-wide blocks of the input features
  constexpr int NB = C / 16;          // 16-wide blocks of the output features
  constexpr int HP = C / 32;          // 32-wide head-dim units
  constexpr int FC = F / 32;          // 32-wide hidden units
  constexpr int NKB = WPG;            // key blocks of a group
  constexpr int NT = NW * 64;
  constexpr int GPW = NW / WPG;       // groups per workgroup
  constexpr int CF = kChunkFrags;
  constexpr int FH = 6 * KB + NB;     // fragments of one head-dim unit: Q, K, V rows, W_o slice
  constexpr int FF = 2 * KB + NB;     // fragments of one hidden unit: W1 rows, W2 slice
  constexpr int CPH = FH / CF, CPF = FF / CF;
  // The unit loops are unrolled completely, which turns the ring bookkeeping into constants, except the two head-dim
  // units of mappings with many key blocks and few registers (no scratch).
  constexpr int FFN_UNROLL = 16;
  constexpr int ATT_UNROLL = NKB > 4 && MINW >= 4 ? 1 : 2;
  constexpr bool LEAN = MINW >= 4;    // four wavefronts on a SIMD: 128 registers each
  constexpr int PF = LEAN ? 4 : kWindow;
  using LP = LdsPlan<WPG, NW, MINW>;
  constexpr int NCHUNK = LP::NCHUNK, RING = LP::RING;
  using PO = ParamOff;
  static_assert(FH % CF == 0 && FF % CF == 0 && CF % PF == 0, "units are whole chunks");

  extern __shared__ u32x4 lds[];
  u32x4* ring = lds;                                            // [RING][CF * 64]
  // These areas lie beyond the 64 KB an LDS instruction reaches from a base register: their offset
  // is hidden from constant folding so that each gets a base register of its own.
  uint32_t par_units = RING * CF * 64;
  asm volatile("" : "+v"(par_units));
  float* par = reinterpret_cast<float*>(lds + par_units);       // [PO::TOTAL]
  u32x2* kvx = reinterpret_cast<u32x2*>(reinterpret_cast<char*>(par) + LP::PARAMS);  // K/V exchange

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, q = lane >> 4;
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int gl = wu / WPG, part = wu % WPG;
  const int g = blockIdx.x * GPW + gl;
  // group_offsets has at least max_groups + 1 entries: read this group's bounds without waiting
  // for num_groups, so that the loads travel together.
  const int gc = g < max_groups ? g : max_groups - 1;
  const int off0 = goff[gc], off1 = goff[gc + 1];
  const int ngroups = *num_groups;
  // Groups of the first (or only) frame start at g * G: fetch the pillar indices from there
  // without waiting for the offsets, and use them if the guess turns out right.
  // (unsigned 32-bit: g * G stays below n + num_frames * G, and one minimum clamps it)
  const uint32_t at = (uint32_t)g * (uint32_t)G + (uint32_t)(part * 16 + i);
  const int32_t guess = perm[at < (uint32_t)n ? at : (uint32_t)n - 1u];
  // in_sorted: row p of feats is the pillar at sorted position p (the previous layer of a block wrote
  // its result in this layer's order), so the rows of a group are contiguous and need no index.
  // in_sorted == 2 (one frame): they are fetched from the guessed start without waiting for anything.
  uint2 early[NB];
  if (in_sorted == 2) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      early[nb] = *reinterpret_cast<const uint2*>(feats + (size_t)(at < (uint32_t)n ? at : (uint32_t)n - 1u) * C + 16 * nb + 4 * q);
  }
  int start = 0, m = 0;
  // A list of full groups only ('Drop Residual') has the next start beyond this group's end.
  if (g < ngroups) { start = off0; m = off1 - off0 < G ? off1 - off0 : G; }

  // ---- weight stream: global memory -> LDS ring -> registers -----------------------------------------
  // Chunk c of the packed stream lives in ring slot c % RING.  `issued` chunks have been requested,
  // chunks below `visible` are known to have landed for every wavefront.  Both advance only at
  // workgroup barriers that every wavefront reaches with the same values.
  int issued = 0, visible = 0;
  auto issue = [&](int chunk) {  // asynchronous copy, 1 KB per instruction, no registers in between
#pragma unroll
    for (int t = 0; t < (CF + NW - 1) / NW; ++t) {
      const int f = wu + t * NW;
      if ((t + 1) * NW <= CF || f < CF) {  // wave-uniform
        if constexpr (LEAN) {  // per-lane address form of the copy below: the scalar operands of the other form
                               // cost registers
          const u32x4* srcv = packed + ((size_t)chunk * CF + f) * 64 + lane;
          const uint32_t dst = (uint32_t)reinterpret_cast<uintptr_t>(
              (__attribute__((address_space(3))) void*)(ring + ((chunk % RING) * CF + f) * 64));
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                       :
                       : "s"(dst), "v"(srcv)
                       : "memory", "m0");
        } else {
          // The copy is written in assembly so that the compiler does not know of it: while it sees an
          // LDS-writing load in flight it waits for every counter to drain at each use of an LDS value
          // (lgkmcnt(0) after every refill of the register window, one exposed LDS latency each time).
          // The protocol above already orders these copies against the reads of the ring (vmcnt(0) and a
          // barrier before a chunk is read), and a vmcnt the compiler computes for its own loads only
          // waits longer with copies in flight that it does not count.
          const uint64_t src = reinterpret_cast<uint64_t>(packed + ((size_t)chunk * CF + f) * 64);  // wave-uniform
          const uint32_t dst = (uint32_t)reinterpret_cast<uintptr_t>(
              (__attribute__((address_space(3))) void*)(ring + ((chunk % RING) * CF + f) * 64));     // LDS byte address
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                       :
                       : "s"(dst), "v"(lane * 16), "s"(src)
                       : "memory", "m0");
        }
      }
    }
  };
  // Barrier.  Every wavefront has finished with all chunks below `consumed` when it arrives.
  auto sync = [&](int consumed) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // my share of every issued chunk has landed
    __syncthreads();
    visible = issued;
    const int lim = consumed + RING < NCHUNK ? consumed + RING : NCHUNK;
    while (issued < lim) { issue(issued); ++issued; }
  };
  // Before the first read of chunk cn.  voluntary: also stop when free slots could be refilled: two of
  // them, or all that is left of the stream (a barrier for a single slot is one barrier more in the
  // FFN, where nothing else needs one).
  auto boundary = [&](int cn, int consumed, bool voluntary) {
    if (cn >= NCHUNK) return;
    const int lim = consumed + RING < NCHUNK ? consumed + RING : NCHUNK;
    if (voluntary && lim > issued && (lim - issued >= 2 || lim == NCHUNK)) sync(consumed);
    while (cn >= visible) sync(consumed);
  };
  // An LDS read reaches 64 KB beyond its base register through the immediate offset; the ring can be
  // larger, so there are two bases, the second one hidden from constant folding.
  uint32_t hi_units = 4 * CF * 64;  // slots 4.. start here (u32x4 units)
  asm volatile("" : "+v"(hi_units));
  const u32x4* ring_lo = ring + lane;
  const u32x4* ring_hi = ring + hi_units + lane;
  auto slot_ptr = [&](int chunk) -> const u32x4* {
    const int slot = chunk % RING;
    return slot < 4 ? ring_lo + slot * CF * 64 : ring_hi + (slot - 4) * CF * 64;
  };

  // All that the ring holds at once, behind the rows that are already on their way: four layers of 20,011 rows, G = 50, 47.5 ->
  // 47.1 us against two chunks now and the others behind the first barrier.
#pragma unroll
  for (int c = 0; c < RING; ++c) issue(c);
  issued = RING;

  // The per-feature vectors (LayerNorm scales and shifts, biases) follow the fragments in the packed buffer as
  // fp32 in the order of ParamOff: they go to LDS the way the weights do, 1 KB per instruction, spread over the
  // wavefronts, and are there for everyone after the first barrier.
  {
    constexpr int PIECES = LP::PARAMS / 1024;
#pragma unroll
    for (int t = 0; t < (PIECES + NW - 1) / NW; ++t) {
      const int piece = wu + t * NW;
      if ((t + 1) * NW <= PIECES || piece < PIECES) {  // wave-uniform
        const u32x4* srcp = packed + ((size_t)NCHUNK * CF + piece) * 64;
        // (LDS byte address from the ring's base: the pointer `par` sits in a vector register)
        const uint32_t dst = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)ring) +
                             (uint32_t)(RING * CF + piece) * 1024u;
        if constexpr (LEAN) {
          const u32x4* srcv = srcp + lane;
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(dst), "v"(srcv) : "memory", "m0");
        } else {
          const uint64_t src = reinterpret_cast<uint64_t>(srcp);  // wave-uniform
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                       :
                       : "s"(dst), "v"(lane * 16), "s"(src)
                       : "memory", "m0");
        }
      }
    }
  }

  // ---- gather + LN1 ---------------------------------------------------------------------------------
  f32x4 x1[NB];  // residual stream of my pillars, accumulator layout
  const bool guessed = (int64_t)g * G == start;  // wave-uniform
  const int s = part * 16 + i;
  int32_t row;        // pillar index, -1 for padding slots
  if (guessed) row = s < m ? guess : -1;
  else row = s < m ? perm[start + s] : -1;
  if (in_sorted == 2 && guessed) {  // the early fetch hit
    const bool live = s < m;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const uint2 u = early[nb];
      // (padding slots: the bits are cleared before the conversion, two instructions per block instead of a
      // branch around each block)
      const uint32_t keep = live ? 0xffffffffu : 0u;
      x1[nb] = f32x4{el_lo(u.x & keep), el_hi(u.x & keep), el_lo(u.y & keep), el_hi(u.y & keep)};
    }
  } else {
    // every lane loads (padding slots read a valid row and drop it): loads under a condition of their
    // own are waited for one by one
    uint2 raw[NB];
    const int32_t src = row >= 0 ? (in_sorted ? start + s : row) : 0;  // row of feats for my pillar
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      raw[nb] = *reinterpret_cast<const uint2*>(feats + (int64_t)src * C + 16 * nb + 4 * q);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const uint2 u = raw[nb];
      const uint32_t keep = row >= 0 ? 0xffffffffu : 0u;
      x1[nb] = f32x4{el_lo(u.x & keep), el_hi(u.x & keep), el_lo(u.y & keep), el_hi(u.y & keep)};
    }
  }
  // Positional embedding of my pillars, still bf16, in the layout of `act` (Eq. (2), second argument
  // of the attention): it is added to the LayerNorm output on the way to the query and key products.
  Frag8 pef[PE ? KB : 1];
  if constexpr (PE) {
    uint2 praw[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      praw[nb] = *reinterpret_cast<const uint2*>(pos_embed + (int64_t)(row >= 0 ? row : 0) * C + 16 * nb + 4 * q);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      pef[nb / 2].u[(nb & 1) * 2 + 0] = row >= 0 ? praw[nb].x : 0u;
      pef[nb / 2].u[(nb & 1) * 2 + 1] = row >= 0 ? praw[nb].y : 0u;
    }
  }
  if (drop && ngroups >= 0) {
    // Pillars of no group skip the layer: their rows are copied.  The wavefronts of group g take the
    // sorted positions between its end and the next group's start, those of group index 0 also the
    // positions before the first start (every position when the list is empty).  Without a list none are.
    auto copy_rows = [&](int lo, int hi) {
      constexpr int LPR = C / 8, RPW = 64 / LPR;  // 16 bytes per lane, several rows per wavefront
      const int sub = lane / LPR, col = (lane % LPR) * 8;
      hi = hi < n ? hi : n;
      for (int p = lo + part * RPW + sub; p < hi; p += WPG * RPW) {
        const int32_t pillar = perm[p];
        const u32x4 v = *reinterpret_cast<const u32x4*>(feats + (int64_t)(in_sorted ? p : pillar) * C + col);
        const int64_t at = (int64_t)(out_index ? out_index[pillar] : pillar) * C + col;
        if constexpr (OUT_F32) {
          float* dst = reinterpret_cast<float*>(out) + at;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            dst[2 * e] = el_lo(v[e]);
            dst[2 * e + 1] = el_hi(v[e]);
          }
        } else {
          *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(out) + at) = v;
        }
      }
    };
    if (g == 0) copy_rows(0, ngroups > 0 ? off0 : n);
    if (g < ngroups) copy_rows(start + m, off1);
  }
  sync(0);  // the ring's first filling and the small parameters are in LDS
  // out_index: the next layer of a block wants its input in its own sorted order.  Fetched only now:
  // the barrier above waits for every load in flight, and this one hangs on the pillar index.
  const int32_t orow = out_index && row >= 0 ? out_index[row] : row;  // row of `out` the result goes to

  // The window: fragments j .. j + PF - 1 of the stream are in registers (or on their way) while
  // fragment j is being used.
  Frag8 win[PF];
  auto fill_window = [&]() {
    const u32x4* p0 = slot_ptr(0);
#pragma unroll
    for (int f = 0; f < PF; ++f) win[f].q = p0[f * 64];
  };
  if (!LEAN) fill_window();  // early, so that the reads overlap the LayerNorm arithmetic
  __builtin_amdgcn_sched_barrier(0);

  Frag8 act[KB];  // normalised activations as B operands (LN1 output, later LN2 output)
  Frag8 actqk[PE ? KB : 1];  // LN1 output plus the positional embedding: input of Q and K
  auto layer_norm = [&](int goff_f, int boff_f, bool first) {
    float s = 0.f, ss = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
      for (int j = 0; j < 4; ++j) { s += x1[nb][j]; ss = fmaf(x1[nb][j], x1[nb][j], ss); }
    }
    const float mu = quad_sum(s) * (1.0f / C);
    const float var = fmaxf(quad_sum(ss) * (1.0f / C) - mu * mu, 0.f);
    const float sc = rsqrtf(var + eps), sh = -mu * sc;  // y = x * sc + sh
    // the affine parameters come from LDS four feature blocks at a time, all eight reads of a batch
    // issued before the first is used (read, wait, use per block exposed the LDS latency every time)
    constexpr int NBG = LEAN ? 1 : 4;  // the lean mapping has no registers for a batch
    static_assert(NB % NBG == 0, "feature blocks per parameter batch");
#pragma unroll
    for (int nb0 = 0; nb0 < NB; nb0 += NBG) {
      f32x4 gmv[NBG], btv[NBG];
#pragma unroll
      for (int u = 0; u < NBG; ++u) {
        gmv[u] = *reinterpret_cast<const f32x4*>(par + goff_f + 16 * (nb0 + u) + 4 * q);
        btv[u] = *reinterpret_cast<const f32x4*>(par + boff_f + 16 * (nb0 + u) + 4 * q);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < NBG; ++u) {
        const int nb = nb0 + u;
        const f32x4 gm = gmv[u], bt = btv[u];
        float y[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = fmaf(fmaf(x1[nb][j], sc, sh), gm[j], bt[j]);
        act[nb / 2].u[(nb & 1) * 2 + 0] = pack2(y[0], y[1]);
        act[nb / 2].u[(nb & 1) * 2 + 1] = pack2(y[2], y[3]);
        if constexpr (PE) {
          if (first) {
            const uint32_t p01 = pef[nb / 2].u[(nb & 1) * 2 + 0], p23 = pef[nb / 2].u[(nb & 1) * 2 + 1];
            actqk[nb / 2].u[(nb & 1) * 2 + 0] = pack2(y[0] + el_lo(p01), y[1] + el_hi(p01));
            actqk[nb / 2].u[(nb & 1) * 2 + 1] = pack2(y[2] + el_lo(p23), y[3] + el_hi(p23));
          }
        }
      }
    }
  };
  auto add_bias_rows = [&](int off_f) {  // x1 += per-feature vector
    constexpr int NBG = LEAN ? 1 : 8;  // reads of a batch issued together, as in layer_norm
#pragma unroll
    for (int nb0 = 0; nb0 < NB; nb0 += NBG) {
      f32x4 b[NBG];
#pragma unroll
      for (int u = 0; u < NBG; ++u) b[u] = *reinterpret_cast<const f32x4*>(par + off_f + 16 * (nb0 + u) + 4 * q);
#pragma unroll
      for (int u = 0; u < NBG; ++u) x1[nb0 + u] += b[u];
    }
  };
  // Bias of the Q rows of a unit (accumulator layout).  K and V start from zero: the key bias has no
  // effect on the softmax and the value bias is part of the folded output bias.
  f32x4 bqk[2];
  auto load_unit_bias = [&](int hp) {
#pragma unroll
    for (int c = 0; c < 2; ++c) bqk[c] = *reinterpret_cast<const f32x4*>(par + PO::BQ + 32 * hp + 16 * c + 4 * q);
  };
  if (!LEAN) load_unit_bias(0);
  layer_norm(PO::LN1G, PO::LN1B, true);
  add_bias_rows(PO::BO);  // residual + output-projection bias
  if (LEAN) { __builtin_amdgcn_sched_barrier(0); fill_window(); }
  const float qscale = rsqrtf((float)DH) * 1.44269504088896340736f;  // 1/sqrt(d) * log2(e)
  // wave-uniform: some key slots are padding.  A wavefront past the last group (m == 0) keeps all its
  // (zero) keys instead, so that it computes finite numbers it never stores rather than -inf - -inf.
  const bool short_group = m > 0 && m < NKB * 16;

  // ---- attention: one 32-wide head-dim unit per iteration (two heads of 16) --------
#pragma unroll ATT_UNROLL
  for (int hp = 0; hp < HP; ++hp) {
    const int c0 = hp * CPH;
    const u32x4* pb[CPH + 1];
#pragma unroll
    for (int k = 0; k <= CPH; ++k) pb[k] = slot_ptr(c0 + k);
    // fragment j of this unit has been used: refill its window slot with fragment j + PF
    auto refill = [&](int j) {
      const int jj = j + PF, k = jj / CF;
      __builtin_amdgcn_sched_barrier(0);
      if (jj % CF == 0) boundary(c0 + k, c0 + (j + 1) / CF, false);
      win[j % PF].q = pb[k][(jj % CF) * 64];  // a hidden unit always follows: the chunk exists
      __builtin_amdgcn_sched_barrier(0);
    };
    if (LEAN) load_unit_bias(hp);
    Frag4 Qf[2], Kf[2], Vf[2];  // bf16 fragments of my pillars, index [16-block a]
    u32x2* kv = kvx + (size_t)((hp & 1) * GPW + gl) * (2 * 2 * NKB * 64) + lane;  // this unit's exchange buffer

    // Six accumulation chains: Q a=0,1 and K a=0,1 as D[feature][pillar], V a=0,1 with the operand
    // roles swapped as D[pillar][feature].  The conversion of a finished chain is issued after the
    // first product of the next one.
    {
      f32x4 acc[2];
      auto finish = [&](int ch) {
        const int a = ch & 1;
        Frag4& dst = ch < 2 ? Qf[a] : ch < 4 ? Kf[a] : Vf[a];
        dst.u[0] = pack2(acc[ch & 1][0], acc[ch & 1][1]);
        dst.u[1] = pack2(acc[ch & 1][2], acc[ch & 1][3]);
        // K/V of the whole group go through LDS: [K|V][16-block a][key block][lane]
        if (ch >= 2) kv[(((ch >= 4 ? 1 : 0) * 2 + a) * NKB + part) * 64] = dst.d;
      };
      // Stream order (kQkvOrder): K and V first, so that their way to LDS overlaps the Q products
      // instead of standing between the last product and the barrier.
#pragma unroll
      for (int p = 0; p < 6; ++p) {
        const int ch = kQkvOrder[p];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const int j = p * KB + kb;
          const Frag8 wf = win[j % PF];
          if (kb == 0) {  // the accumulator starts from the bias
              acc[ch & 1] = ch < 2 ? bqk[ch] : f32x4{0.f, 0.f, 0.f, 0.f};
          }
            acc[ch & 1] = ch < 4 ? mfma32(wf, PE ? actqk[PE ? kb : 0] : act[kb], acc[ch & 1])
                                     : mfma32(act[kb], wf, acc[ch & 1]);
          if (kb == 0 && p > 0) finish(kQkvOrder[p - 1]);
          refill(j);
        }
      }
      finish(kQkvOrder[5]);
    }
    sync(c0 + (6 * KB) / CF);         // K/V of the group are in LDS
    if (!LEAN) load_unit_bias(hp + 1 < HP ? hp + 1 : hp);
    auto Kget = [&](int a, int jb) -> Frag4 { Frag4 f; f.d = kv[((0 * 2 + a) * NKB + jb) * 64]; return f; };
    auto Vget = [&](int a, int jb) -> Frag4 { Frag4 f; f.d = kv[((1 * 2 + a) * NKB + jb) * 64]; return f; };
    Frag8 Of;                         // attention output of this unit as B operand of the output projection
    // The unit's two heads are independent; they go through the softmax in lockstep stages so that the long
    // dependency chains interleave, if there are registers for both heads' score tiles (168 of them with three
    // wavefronts on a SIMD).
    constexpr int HJ = 2 * NKB <= (MINW == 3 ? 8 : 16) && MINW < 4 ? 2 : 1;
#pragma unroll
    for (int h0 = 0; h0 < 2; h0 += HJ) {
      f32x4 S[HJ][NKB];               // scores, transposed: S[key 16*jb + 4q + j][query i]
#pragma unroll
      for (int hh = 0; hh < HJ; ++hh)
#pragma unroll
        for (int jb = 0; jb < NKB; ++jb)
          // the only k=16 products left: their accumulator input is zero, so they depend on no
          // earlier product (see the note at the odd key block below)
          S[hh][jb] = mfma16_from_zero(Kget(h0 + hh, jb), Qf[h0 + hh]);
      if (short_group) {  // keys beyond the group's real members
#pragma unroll
        for (int hh = 0; hh < HJ; ++hh)
#pragma unroll
          for (int jb = 0; jb < NKB; ++jb)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (16 * jb + 4 * q + j >= m) S[hh][jb][j] = -INFINITY;
      }
      float mxs[HJ];
#pragma unroll
      for (int hh = 0; hh < HJ; ++hh) {
        float mx = S[hh][0][0];
#pragma unroll
        for (int jb = 0; jb < NKB; ++jb)
#pragma unroll
          for (int j = 0; j < 4; ++j) mx = fmaxf(mx, S[hh][jb][j]);
        mxs[hh] = mx;
      }
#pragma unroll
      for (int hh = 0; hh < HJ; ++hh) mxs[hh] = -quad_max(mxs[hh]) * qscale;
      // p = 2^((s - max) * log2(e) / sqrt(d)): the score scale lives in the exponent argument
#pragma unroll
      for (int hh = 0; hh < HJ; ++hh)
#pragma unroll
        for (int jb = 0; jb < NKB; ++jb)
#pragma unroll
          for (int j = 0; j < 4; ++j) S[hh][jb][j] = __builtin_amdgcn_exp2f(fmaf(S[hh][jb][j], qscale, mxs[hh]));
      // O^T[d][query] = sum over keys V^T[d][key] P^T[key][query], two key blocks per product.
      // The row sums of P come from the matrix cores as well: an all-ones A operand makes every
      // accumulator row the sum over keys of the (16-bit rounded) probabilities.
      f32x4 O[HJ], rowsum[HJ];
#pragma unroll
      for (int hh = 0; hh < HJ; ++hh) {
        const int h = h0 + hh;
        Frag8 ones;
        ones.u[0] = ones.u[1] = ones.u[2] = ones.u[3] = kOnePair;
        rowsum[hh] = f32x4{0.f, 0.f, 0.f, 0.f};
        O[hh] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int jb = 0; jb + 1 < NKB; jb += 2) {
          Frag8 p8, v8;
          p8.u[0] = pack2(S[hh][jb][0], S[hh][jb][1]); p8.u[1] = pack2(S[hh][jb][2], S[hh][jb][3]);
          p8.u[2] = pack2(S[hh][jb + 1][0], S[hh][jb + 1][1]); p8.u[3] = pack2(S[hh][jb + 1][2], S[hh][jb + 1][3]);
          const Frag4 v0 = Vget(h, jb), v1 = Vget(h, jb + 1);
          v8.u[0] = v0.u[0]; v8.u[1] = v0.u[1]; v8.u[2] = v1.u[0]; v8.u[3] = v1.u[1];
          O[hh] = mfma32(v8, p8, O[hh]);
          rowsum[hh] = mfma32(ones, p8, rowsum[hh]);
        }
        if (NKB & 1) {
          // The odd last key block: a k=32 product whose upper half multiplies zeros.  A k=16
          // product here was wrong on this chip: issued right behind a k=32 product into the same
          // accumulator it read the accumulator before that product had written it (row sums of 48
          // instead of 80, whenever the scheduler put the two back to back), so every product of an
          // accumulation chain is of one kind.  The k=16 product takes the same 16 cycles anyway.
          constexpr int jb = NKB - 1;
          Frag8 p8, v8;
          p8.u[0] = pack2(S[hh][jb][0], S[hh][jb][1]); p8.u[1] = pack2(S[hh][jb][2], S[hh][jb][3]);
          p8.u[2] = p8.u[3] = 0u;
          const Frag4 v0 = Vget(h, jb);
          v8.u[0] = v0.u[0]; v8.u[1] = v0.u[1]; v8.u[2] = v8.u[3] = 0u;
          O[hh] = mfma32(v8, p8, O[hh]);
          rowsum[hh] = mfma32(ones, p8, rowsum[hh]);
        }
      }
#pragma unroll
      for (int hh = 0; hh < HJ; ++hh) {
        const float inv = __builtin_amdgcn_rcpf(rowsum[hh][0]);
        Of.u[(h0 + hh) * 2 + 0] = pack2(O[hh][0] * inv, O[hh][1] * inv);
        Of.u[(h0 + hh) * 2 + 1] = pack2(O[hh][2] * inv, O[hh][3] * inv);
      }
    }
    // output projection of this unit, accumulated into the residual stream
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int j = 6 * KB + nb;
      const Frag8 wf = win[j % PF];
      x1[nb] = mfma32(wf, Of, x1[nb]);
      refill(j);
    }
  }

  // ---- FFN ------------------------------------------------------------------------------------------
  f32x4 b1r[2];
  auto load_b1 = [&](int fc) {
#pragma unroll
    for (int a = 0; a < 2; ++a) b1r[a] = *reinterpret_cast<const f32x4*>(par + PO::B1 + 32 * fc + 16 * a + 4 * q);
  };
  if (!LEAN) load_b1(0);
  layer_norm(PO::LN2G, PO::LN2B, false);
  add_bias_rows(PO::B2);
#pragma unroll FFN_UNROLL
  for (int fc = 0; fc < FC; ++fc) {
    const int c0 = HP * CPH + fc * CPF;
    const u32x4* pb[CPF + 1];
#pragma unroll
    for (int k = 0; k <= CPF; ++k) pb[k] = slot_ptr(c0 + k);
    auto refill = [&](int j) {
      const int jj = j + PF, k = jj / CF;
      __builtin_amdgcn_sched_barrier(0);
      if (jj % CF == 0) boundary(c0 + k, c0 + (j + 1) / CF, true);
      if (k < CPF || fc + 1 < FC) win[j % PF].q = pb[k][(jj % CF) * 64];
      __builtin_amdgcn_sched_barrier(0);
    };
    Frag8 Hf;
    if (LEAN) load_b1(fc);
    {
      f32x4 acc[2];
      auto finish = [&](int a) {
        Hf.u[a * 2 + 0] = pack2(gelu2_fast(acc[a][0]), gelu2_fast(acc[a][1]));
        Hf.u[a * 2 + 1] = pack2(gelu2_fast(acc[a][2]), gelu2_fast(acc[a][3]));
      };
#pragma unroll
      for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const int j = a * KB + kb;
          const Frag8 wf = win[j % PF];
          if (kb == 0) acc[a] = b1r[a];
          acc[a] = mfma32(wf, act[kb], acc[a]);
          if (kb == 0 && a == 1) finish(0);
          refill(j);
        }
      }
      finish(1);
    }
    if (!LEAN) load_b1(fc + 1 < FC ? fc + 1 : fc);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int j = 2 * KB + nb;
      const Frag8 wf = win[j % PF];
      x1[nb] = mfma32(wf, Hf, x1[nb]);
      refill(j);
    }
  }

  // ---- scatter -------------------------------------------------------------------------------------
  if (row < 0) return;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const size_t o = (size_t)orow * C + 16 * nb + 4 * q;
    if (OUT_F32) {
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + o) =
          make_float4(x1[nb][0], x1[nb][1], x1[nb][2], x1[nb][3]);
    } else {
      *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + o) =
          make_uint2(pack2(x1[nb][0], x1[nb][1]), pack2(x1[nb][2], x1[nb][3]));
    }
  }
}

template <int WPG, int NW, int MINW>
int launch_cfg(const void* feats, void* out, const void* pos_embed, const int32_t* perm, const int32_t* goff,
               const int32_t* num_groups,
               int32_t max_groups, const u32x4* packed, float eps, bool out_f32, int n, int G,
               int drop, const int32_t* out_index, int in_sorted, hipStream_t stream) {
  constexpr int GPW = NW / WPG;
  const size_t lds_bytes = LdsPlan<WPG, NW, MINW>::TOTAL;
  const unsigned blocks = (unsigned)((max_groups + GPW - 1) / GPW);
  // The dynamic LDS size has to be allowed once per kernel and device (output type and positional
  // embedding make four kernels of a mapping).
  static std::atomic<uint64_t> allowed[4] = {{0}, {0}, {0}, {0}};  // bit d: done on device d
  auto go = [&](auto kern, int which) -> int {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return FF_ERR_LAUNCH;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(allowed[which].load(std::memory_order_acquire) & bit)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds_bytes) != hipSuccess)
        return FF_ERR_LAUNCH;
      allowed[which].fetch_or(bit, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(NW * 64), lds_bytes, stream, (const uint16_t*)feats, perm, packed,
                       n, G, in_sorted, (int)max_groups, goff, num_groups, out_index, out, (const uint16_t*)pos_embed, drop, eps);
    return launch_status();
  };
  if (pos_embed) {
    if (out_f32) return go(k_layer_mfma<WPG, NW, MINW, true, true>, 3);
    return go(k_layer_mfma<WPG, NW, MINW, false, true>, 2);
  }
  if (out_f32) return go(k_layer_mfma<WPG, NW, MINW, true, false>, 1);
  return go(k_layer_mfma<WPG, NW, MINW, false, false>, 0);
}

}  // namespace

// Shapes with a fused kernel: (C, head dim, F) = (128, 16, 256), (256, 32, 512) and (64, 16, 128), G <= 128.
static int shape_id(const ff_layer_weights* w) {
  const int C = w->C, F = w->F, d = C / w->heads;
  if (C == 128 && d == 16 && F == 256) return 1;
  if (C == 256 && d == 32 && F == 512) return 2;
  if (C == 64 && d == 16 && F == 128) return 3;
  return 0;
}

#ifndef FF_LAYER_F16  // the same for both formats
bool layer_mfma_supported(const ff_layer_weights* w, int G) { return shape_id(w) != 0 && G <= 128; }
#endif

static size_t layer_mfma_frag_count(const ff_layer_weights* w) {
  const int C = w->C, F = w->F;
  return (size_t)((C / 32) * frags_per_hp(C) + (F / 32) * frags_per_fc(C));
}

#ifndef FF_LAYER_F16
size_t layer_mfma_packed_bytes(const ff_layer_weights* w) {
  return layer_mfma_frag_count(w) * (size_t)1024 + (size_t)pack_param_bytes(w->C, w->F);
}
#endif

// Packs `count` layers of identical shape; layer l goes to packed + l * stride_bytes.
int FF_LAYER_SYM(layer_mfma_pack)(const ff_layer_weights* w, int count, void* packed, size_t stride_bytes,
                                  hipStream_t stream) {
  for (int l0 = 0; l0 < count; l0 += kPackBatch) {
    const int nl = count - l0 < kPackBatch ? count - l0 : kPackBatch;
    PackJob job;
    make_pack_job(w + l0, nl, (char*)packed + (size_t)l0 * stride_bytes, stride_bytes, kHalf ? kPackF16 : kPackBf16, &job);
    hipLaunchKernelGGL(k_pack_weights, dim3((unsigned)job.blocks, (unsigned)nl), dim3(256), 0, stream, job.pb, job.C,
                       job.F, job.total_frags);
  }
  return launch_status();
}

// variant: 0 = chosen from the shape; 1.. = a specific wave/group mapping (tuning and tests).
int FF_LAYER_SYM(layer_mfma_launch)(const void* feats, void* out, int64_t n, const int32_t* perm, const int32_t* group_offsets,
                      const int32_t* num_groups, int32_t max_groups, const ff_layer_weights* w, int G,
                      bool out_f32, bool drop, const void* packed, int variant, const int32_t* out_index,
                      int in_sorted, hipStream_t stream) {
  if (max_groups == 0 || n == 0) return FF_OK;
  const u32x4* pk = (const u32x4*)packed;
#define FF_GO(WPG, NW, MINW) \
  return launch_cfg<WPG, NW, MINW>(feats, out, w->pos_embed, perm, group_offsets, num_groups, max_groups, pk, \
                                                  w->ln_eps, out_f32, (int)n, G, drop ? 1 : 0, out_index, in_sorted, stream)
  const int shape = shape_id(w);
  const bool pe = w->pos_embed != nullptr;
  if (shape != 3) {
    // 128 and 256 features: wavefronts that cut the features.  They are ahead of wavefronts that cut the rows, which served
    // these widths before, nearly everywhere (us a layer, before / now, 30,000 rows: C = 128, G = 64 16.5 / 14.7, G = 69 23.6 /
    // 21.9, G = 100 32.8 / 26.8; C = 256, G = 64 43.8 / 40.9; 2,000 rows, C = 256 40 / 16; the other way round for groups of more
    // than 112 in one or two rounds at C = 128, 20.8 / 21.4 and with float32 results 23.3 / 24.4); at 64 features, two wavefronts a
    // group, they are not (20,000 rows, G = 50: 8.9 / 10.9).
    // Mapping numbers are forms of that kernel, each with its largest group; the forms differ in which rows and registers a
    // wavefront has, not in the operations on a row or their order, so all that hold G give the same bits.  (Numbers that have never
    // taken a positional embedding, and groups beyond the size a number has stood for, are still refused.)
    struct Mapping { int slots; bool embeds; int blocks, waves; bool whole; };
    static constexpr Mapping kNone = {0, false, 0, 0, false};
    static constexpr Mapping k128[16] = {{128, true, 0, 0, false}, {32, false, 1, 2, false}, {64, true, 2, 2, true}, {80, true, 3, 0, false},
                                         {128, true, 4, 0, true}, kNone, {64, true, 2, 3, true}, {64, true, 2, 2, false},
                                         {128, false, 4, 0, true}, {128, true, 4, 0, false}, {32, true, 1, 2, false}, {64, false, 3, 0, false},
                                         {64, true, 2, 3, false}, {80, true, 3, 0, true}, {96, true, 3, 0, false}, {32, true, 1, 3, false}};
    static constexpr Mapping k256[16] = {{128, true, 0, 0, false}, {32, true, 1, 0, false}, {64, true, 2, 0, false}, {80, false, 3, 0, false},
                                         {128, true, 4, 0, false}, {64, true, 3, 0, false}, {80, true, 4, 0, true}, {96, false, 3, 0, true},
                                         {64, false, 3, 0, true}, kNone, kNone, kNone, kNone, kNone, kNone, kNone};
    const Mapping& mp = (shape == 1 ? k128 : k256)[variant & 15];
    if (G > mp.slots || (pe && !mp.embeds)) return FF_ERR_UNSUPPORTED;
    const LayerSlice call{feats, out, (int)n, perm, group_offsets, num_groups, max_groups, w, G, drop, out_f32, packed, out_index,
                          in_sorted, mp.blocks, mp.waves, mp.whole};
    return FF_LAYER_SYM(layer_slice_launch)(call, stream);
  }
  // The narrow layer (64 features, 4 heads): the whole 64 KB weight stream stays in the ring.  A launch runs in rounds of one
  // workgroup per compute unit.  A workgroup of more wavefronts does more per round, because the wavefronts of a SIMD hide each
  // other's stalls and read the staged weights together, but its round takes longer: the mapping with the smaller
  // product of rounds and measured time of a round wins.  A mapping whose wavefronts cover G with fewer padding slots
  // does less work.
  auto rounds = [&](int per_wg) { return ceil_div(ceil_div((int64_t)max_groups, per_wg), kComputeUnits); };
  if (variant == 0) {
    // G <= 32: four or eight groups per workgroup (1301 groups 14.8 / 13.2 us, 2602: 21.9 / 23.5, 9009: 63 / 56);
    // G <= 64: two or four (466 groups 12.1 / 13.5, 942: 16.6 / 14.4, 1302: 23.7 / 26.0, 3407: 54 / 51); G <= 80 and
    // <= 96: two of five or six wavefronts against one of eight (466 groups 18.8 -> 12.5 and 19.6 -> 13.7, 3400: 121
    // -> 75 and 125 -> 84); above: one or two (466: 18.9 / 16.7, 627: 27.4 / 30.1, 1172: 44.6 / 44.9, 3414: 123 / 104).
    if (G <= 32) variant = rounds(4) * 70 <= rounds(8) * 118 ? 1 : 3;
    else if (G <= 64) variant = rounds(2) * 79 <= rounds(4) * 129 ? 2 : 8;
    else if (G <= 96) variant = rounds(1) == 1 ? 4 : G <= 80 ? 5 : 6;
    else variant = rounds(1) * 90 <= rounds(2) * 151 ? 4 : 7;
  }
  // (waves per group, waves per workgroup, min waves per SIMD)
  switch (variant) {
    case 1: if (G <= 32) FF_GO(2, 8, 2); break;
    case 2: if (G <= 64) FF_GO(4, 8, 2); break;
    case 3: if (G <= 32) FF_GO(2, 16, 4); break;   // eight groups
    case 4: if (G <= 128) FF_GO(8, 8, 2); break;
    case 5: if (G <= 80) FF_GO(5, 10, 3); break;   // two groups
    case 6: if (G <= 96) FF_GO(6, 12, 3); break;   // two groups
    case 7: if (G <= 128) FF_GO(8, 16, 4); break;  // two groups
    case 8: if (G <= 64) FF_GO(4, 16, 4); break;   // four groups
    default: break;
  }
#undef FF_GO
  return FF_ERR_UNSUPPORTED;
}

}  // namespace ff
