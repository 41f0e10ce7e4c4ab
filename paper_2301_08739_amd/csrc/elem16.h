// Number format of the 16-bit layer kernels, and what all of them do element by element.  A translation unit is built
// for bfloat16, or with FF_LAYER_F16 defined for IEEE half (the precision the paper runs in, Sec. 5.1), from the same
// sources.
#pragma once
#include "common.h"

namespace ff {
namespace {

// ---- number format of the 16-bit storage and of the matrix-core operands --------------------------------
#ifdef FF_LAYER_F16
typedef _Float16 el8 __attribute__((ext_vector_type(8)));
typedef _Float16 el4 __attribute__((ext_vector_type(4)));
typedef _Float16 el2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kOnePair = 0x3c003c00u;  // two ones
__device__ __forceinline__ float el_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
__device__ __forceinline__ float el_lo(uint32_t u) { return el_to_f32((uint16_t)(u & 0xffffu)); }
__device__ __forceinline__ float el_hi(uint32_t u) { return el_to_f32((uint16_t)(u >> 16)); }
#define FF_LAYER_SYM(name) name##_f16
#else
typedef __bf16 el8 __attribute__((ext_vector_type(8)));
typedef short el4 __attribute__((ext_vector_type(4)));
typedef __bf16 el2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kOnePair = 0x3f803f80u;  // two ones
__device__ __forceinline__ float el_to_f32(uint16_t h) { return bf16_to_f32(h); }
__device__ __forceinline__ float el_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float el_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
#define FF_LAYER_SYM(name) name
#endif
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

union Frag8 {  // eight 16-bit elements = one operand of the k=32 product
  el8 v;
  uint32_t u[4];
  u32x4 q;
};
union Frag4 {  // four 16-bit elements = one operand of the k=16 product
  el4 v;
  uint32_t u[2];
  u32x2 d;
};

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  f32x2 f = {lo, hi};
  el2 r = __builtin_convertvector(f, el2);  // round to nearest even
  return *reinterpret_cast<uint32_t*>(&r);
}
__device__ __forceinline__ void load4(const uint16_t* p, float* o) {  // 4 consecutive elements -> fp32
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  o[0] = el_lo(u.x);
  o[1] = el_hi(u.x);
  o[2] = el_lo(u.y);
  o[3] = el_hi(u.y);
}
// GELU(v) = v * Phi(v) with the upper tail 1 - Phi(t) ~ 0.5 * exp(-(a t + b t^2 + c t^3)), t = |v|
// (coefficients fitted to the erf form; all positive, so the exponent is monotone for any t):
//   GELU(v) = max(v, 0) - 0.5 t e = 0.5 (v + t (1 - e)),   e = exp(-(a t + b t^2 + c t^3)),
// max abs error 8.6e-5.  This returns 2 GELU(v); the factor 0.5 is folded into the packed W2
// (exact in bf16).  Five vector operations and one transcendental per element.
__device__ __forceinline__ float gelu2_fast(float v) {
  constexpr float L2E = 1.44269504088896340736f;
  const float t = fabsf(v);
  float p = fmaf(t, -0.01916250660946074f * L2E, -0.33840941696965965f * L2E);
  p = fmaf(t, p, -0.7908370960657618f * L2E);
  const float e = __builtin_amdgcn_exp2f(p * t);
  return v + fmaf(-t, e, t);
}

}  // namespace
}  // namespace ff
