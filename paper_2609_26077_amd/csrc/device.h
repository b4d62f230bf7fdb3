// Device helpers: block-scale rules and the e4m3 cast (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace fmm {
namespace dev {

constexpr float kFltMax = 3.402823466e38f;
constexpr float kE4m3Max = 448.0f;
constexpr float kClamp = 1e-12f;  // fl32(1e-12): the block maximum is clamped from below

enum { RULE_FP32_AMAX = 0, RULE_POW2_CEIL = 1, RULE_POW2_OCP = 2 };

// Scale of one block from its absolute maximum.
//   FP32_AMAX : s = fl32(a / 448), returned in `s`; `inv_or_div` = s (divide by it)
//   POW2_*    : s = 2^e; `inv_or_div` = 2^-e (multiplying by it is exactly x / s)
// `stored` receives the stored form: the fp32 bits of s, or the E8M0 byte e + 127.
struct Scale {
  float div;       // FP32_AMAX: the divisor s
  float inv;       // FP32_AMAX: fl32(1 / s), for div_by
  float mul;       // POW2: 2^-e
  uint32_t stored;
};

// x / d rounded to nearest, given inv = fl32(1 / d): the quotient estimate's
// exact remainder corrects it.  Three instructions where the general division
// sequence takes about fourteen, which was half of the fp32-scale encoder's
// arithmetic (encodes with fp32 scales, us: 8192^3 with 128 x 128 weight blocks
// 266 -> 230, 2560x3584x2560 at block 128 41 -> 33, <2,2,3;11> 8 of
// 512x512x768 17.3 -> 14.3).
// Equal to x / d for d in [2^-49, 2^120] and |x| <= 448 d (1 + 2^-23): over every
// significand of d the quotient was compared for the numerators within 6 ulp
// of d times each boundary between two codes (1.7e9 pairs; the test keeps a
// sample), and further from a boundary the estimate's error, about 2^-46
// relative, changes no code.  Tiny x, whose remainder may be subnormal, give
// a quotient below 2^-10 of x's sign: the remainder is taken as q d - x and
// subtracted, so that it is +0 for x = +-0 and the zero keeps its sign.
__device__ __forceinline__ float div_by(float x, float d, float inv) {
  const float q = x * inv;
  return __fmaf_rn(-__fmaf_rn(q, d, -x), inv, q);
}

__device__ __forceinline__ Scale block_scale(float amax, int rule) {
  Scale sc;
  const float a = fmaxf(amax, kClamp);
  if (rule == RULE_FP32_AMAX) {
    // (= a / 448 for every significand of a, compared; a combination of finite
    // operands may overflow: its block's scale is then inf, whose finite values
    // div_by takes to zeros of their signs and whose infinite ones to NaN, as x / s does)
    const float s = a <= kFltMax ? div_by(a, kE4m3Max, 1.0f / kE4m3Max) : a;
    sc.div = fminf(s, kFltMax);
    sc.inv = __fdiv_rn(1.0f, s);
    sc.mul = 1.0f;
    sc.stored = __float_as_uint(s);
    return sc;
  }
  // a >= 1e-12 is a normal binary32: a = m 2^E, m in [1, 2).
  const uint32_t bits = __float_as_uint(a);
  const int E = (int)((bits >> 23) & 0xffu) - 127;
  int e = E - 8;
  // POW2_CEIL: least e with a <= 448 2^e = 1.75 2^(e+8): e = E-8 iff m <= 1.75.
  if (rule == RULE_POW2_CEIL && (bits & 0x7fffffu) > 0x600000u) e += 1;
  sc.div = 1.0f;
  sc.inv = 1.0f;
  sc.mul = __uint_as_float((uint32_t)(127 - e) << 23);  // 2^-e, e in [-48, 121]
  sc.stored = (uint32_t)(e + 127);
  return sc;
}

// e4m3 codes of four scaled values, packed little-endian into a word.
// v_cvt_pk_fp8_f32 rounds to nearest even and keeps the sign, but turns
// magnitudes above 448 into NaN, so saturate first: rounding then clamping to
// 448 equals clamping then rounding.
__device__ __forceinline__ uint32_t e4m3_pack4(float v0, float v1, float v2, float v3) {
  v0 = __builtin_amdgcn_fmed3f(v0, -kE4m3Max, kE4m3Max);
  v1 = __builtin_amdgcn_fmed3f(v1, -kE4m3Max, kE4m3Max);
  v2 = __builtin_amdgcn_fmed3f(v2, -kE4m3Max, kE4m3Max);
  v3 = __builtin_amdgcn_fmed3f(v3, -kE4m3Max, kE4m3Max);
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(v0, v1, 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(v2, v3, w, true);
  return (uint32_t)w;
}

// Codes of four values under a power-of-two scale s = 2^e, e in [-48, 120]:
// the e4m3 code of x / s with round to nearest even, saturated to 448.
// v_cvt_scalef32_pk_fp8_f32 divides by the power of two that its scale
// operand holds (exactly, subnormal binary32 inputs included) and rounds to
// nearest even, but, like the plain cast, does not saturate; clamping x to
// +-448 s first is exact because 448 s is.  Where 448 s overflows binary32
// (e = 120, reached only by the ceiling rule) |x| <= 448 s holds already and
// the clamp to +-inf is the identity.
__device__ __forceinline__ uint32_t e4m3_pack4_pow2(float v0, float v1, float v2, float v3, float s) {
  typedef short v2i16 __attribute__((ext_vector_type(2)));
  const float lim = 448.0f * s;
  v0 = __builtin_amdgcn_fmed3f(v0, -lim, lim);
  v1 = __builtin_amdgcn_fmed3f(v1, -lim, lim);
  v2 = __builtin_amdgcn_fmed3f(v2, -lim, lim);
  v3 = __builtin_amdgcn_fmed3f(v3, -lim, lim);
  v2i16 w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32((v2i16){0, 0}, v0, v1, s, false);
  w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w, v2, v3, s, true);
  return __builtin_bit_cast(uint32_t, w);
}

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// Eight codes (two little-endian words) -> their values times the power of two
// whose exponent field `s` carries, as bf16 (exact).
__device__ __forceinline__ v8bf dequant8(uint32_t lo, uint32_t hi, float s) {
  typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
  const v2bf a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)lo, s, false);
  const v2bf b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)lo, s, true);
  const v2bf c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)hi, s, false);
  const v2bf d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)hi, s, true);
  v8bf r;
  r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1];
  r[4] = c[0]; r[5] = c[1]; r[6] = d[0]; r[7] = d[1];
  return r;
}

// A float whose exponent field is E8M0 byte i of word w, as the scale operand
// of v_cvt_scalef32_pk_bf16_fp8, which reads the exponent field alone (its sign
// and mantissa bits, here parts of the neighbouring bytes, leave the result
// unchanged: every code at every exponent -48 .. 120 measured), so one shift
// places the byte.
__device__ __forceinline__ float e8m0_at(uint32_t w, int i) {
  return __uint_as_float(i == 3 ? w >> 1 : w << (23 - 8 * i));
}

}  // namespace dev
}  // namespace fmm
