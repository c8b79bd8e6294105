// Device-side building blocks shared by the HiFA4 kernels (gfx950).
//
// HIF4 group quantization (paper, Background "HIF4" paragraph; Section 4.1)
// under the library's reading: unsigned E6M2 base b = smallest value with
// 1.75*b >= max|x| (bias 31); level-2 (8 elements) and level-3 (4 elements)
// one-bit micro-exponents that halve the scale when the block's maximum fits
// in half of the range; element code u = round-half-away(|x| / step),
// step = b * 2^-(E2+E3) / 4.
//
// MFMA operand encoding.  A HIF4 element equals o * b/4 with o = u * 2^-sh,
// u in 0..7 and sh = E2+E3 in 0..2.  Every such o is exactly representable in
// the OCP FP6 E2M3 format (values m/8 and (1+m/8)*2^(e-1)), which E2M1 (FP4)
// cannot hold (5 and 7 need three significant bits).  The kernels therefore
// feed o as FP6 E2M3 to the block-scaled F8F6F4 MFMA (same issue rate as
// FP4) with unit E8M0 scales, so every group dot product sum(o_q * o_k) is
// exact in the fp32 accumulator, and apply the E6M2 bases (which carry two
// mantissa bits that an E8M0 scale cannot) in an fp32 epilogue.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hifa4 {

typedef _Float16 half_t;
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef _Float16 h32_t __attribute__((ext_vector_type(32)));
typedef float f16v_t __attribute__((ext_vector_type(16)));
typedef int i6_t __attribute__((ext_vector_type(6)));
typedef int i8_t __attribute__((ext_vector_type(8)));

// fp32 bits of the smallest E6M2 value b with 1.75*b >= A (A >= 0, an fp16 or
// fp16-softmax value held exactly in fp32); A = 0 gives 0.  b is A/1.75 rounded
// up to two mantissa bits.  The product with 4/7 (1 - 2^-20) stands for the
// quotient: where A = 1.75 b exactly it lies just below b and rounds up to b;
// any other fp16 A lies at least 2^-12 (relative) from such a value, far more
// than the bias and the rounding of the product, so it rounds up to the same
// value as the quotient.  Three instructions against the fourteen of counting
// significand thresholds.
__device__ __forceinline__ uint32_t e6m2_cover_bits(float A) {
  const float y = A * 0x1.249236p-1f;                  // 4/7 (1 - 2^-20)
  return (__float_as_uint(y) + 0x1FFFFFu) & 0xFFE00000u;
}

// E6M2 byte of the value with fp32 bits b (0 for b = 0).
__device__ __forceinline__ uint32_t e6m2_code_of(uint32_t b) { return b ? (b - 0x30000000u) >> 21 : 0u; }

// Smallest E6M2 byte whose value b satisfies 1.75*b >= A; A = 0 gives 0.
__device__ __forceinline__ uint32_t e6m2_ceil(float A) { return e6m2_code_of(e6m2_cover_bits(A)); }

// E6M2 value b = (1 + m/4) * 2^(e-31) of byte e<<2|m, built from its bits.
__device__ __forceinline__ float e6m2_bits_value(uint32_t code) {
  return __uint_as_float((code << 21) + 0x30000000u);
}

// R = (4/b) * (1 + 2^-18), rounded: for the 4 base mantissas the constant
// fp32(16/(4+m) * (1 + 2^-18)), then an exact power-of-two scaling by
// 2^(31-e) applied to the exponent field.
//
// Element rounding uses o = fl(a*R + C_sh) - C_sh with C_sh = 1.5*2^(23-sh)
// (fp32) or 1.5*2^(10-sh) (fp16 destination): the fused multiply-add rounds
// the exact product a*R once onto the grid 2^-sh, which is u*2^-sh with
// u = round-half-to-even(a/step * (1+beta)).  a/step is an fp16 value divided
// by (4+m)*2^k: a non-tie lies at least 2^-12 (relative) from a half-integer
// while beta ~ 2^-18, so those round as exactly as without beta; an exact tie
// n+1/2 is pushed strictly above and rounds away from zero.  The result is
// exactly round-half-away(a/step).
__device__ __forceinline__ float hif4_rcp_step(uint32_t code) {
  const uint32_t m = code & 3u;
  const uint32_t lo = (m & 1u) ? 0x404ccd00u : 0x40800020u;   // m = 1 : 0
  const uint32_t hi = (m & 1u) ? 0x40124949u : 0x402aaad5u;   // m = 3 : 2
  const uint32_t cb = (m & 2u) ? hi : lo;
  return __uint_as_float(cb + (uint32_t)((31 - (int)(code >> 2)) << 23));
}

// E6M2 value of a base byte: (1 + m/4) * 2^(e - 31).
__device__ __forceinline__ float e6m2_value(uint32_t code) { return e6m2_bits_value(code); }

__device__ __forceinline__ float round_const(int sh) {
  return sh == 0 ? 12582912.0f : (sh == 1 ? 6291456.0f : 3145728.0f);
}

// fp16 softmax exponential E(x) = fp16(2^x) for a pair of fp16 x (x = -inf
// gives 0): v_exp_f16 on the low half, then its SDWA form on the high half,
// which keeps the low half of the destination.  The SDWA form reads the
// destination to preserve it, so it must wait for the transcendental result
// (the s_nop; the compiler does not see this dependency inside the asm).
// On gfx950 v_exp_f16 returns the correctly rounded value for every fp16
// input x <= 0 (checked exhaustively; the library's exp2 self-test entry
// point re-checks this routine on the device).
__device__ __forceinline__ h2_t exp2_h2(h2_t x) {
  h2_t y;
  asm("v_exp_f16 %0, %1\n\ts_nop 1\n\tv_exp_f16_sdwa %0, %1 dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:WORD_1"
      : "=&v"(y)
      : "v"(x));
  return y;
}

// Pack fp16(fp32(a*c)) and fp16(fp32(b*c)): the products are rounded to fp32,
// then converted to fp16 (round to nearest even) by one packed conversion.
__device__ __forceinline__ h2_t scale2_to_f16(float a, float b, float c) {
  const float ya = a * c, yb = b * c;
  h2_t y;
  asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(y) : "v"(ya), "v"(yb));
  return y;
}

// Pack fp16(a) and fp16(b) (round to nearest even) into one register.
__device__ __forceinline__ h2_t pack2_f16(float a, float b) {
  h2_t y;
  asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(y) : "v"(a), "v"(b));
  return y;
}

// fp16 nearest to the exact quotient k/s (k an fp16 value, s > 0 fp32): the
// correctly rounded fp32 quotient rounds to the same fp16 unless it sits
// exactly on an fp16 midpoint; there the exact remainder k - q*s (exact in
// fp32 for a correctly rounded q) tells on which side the true quotient lies.
__device__ __forceinline__ half_t div_rn16(float k, float s) {
  const float q = k / s;
  const half_t h = (half_t)q;
  const float hv = (float)h;
  if (hv == q) return h;
  const uint16_t hb = __builtin_bit_cast(uint16_t, h);
  // neighbour of h on q's side (magnitude up if |q| > |h|)
  const uint16_t nbb = (fabsf(q) > fabsf(hv)) ? (uint16_t)(hb + 1) : (uint16_t)(hb - 1);
  const half_t nb = __builtin_bit_cast(half_t, nbb);
  const float mid = 0.5f * (hv + (float)nb);
  if (q != mid) return h;
  const float r = __builtin_fmaf(-q, s, k);        // exact remainder
  if (r == 0.0f) return h;                          // exact tie: h is the even one
  const bool above = r > 0.0f;                      // true quotient > q (s > 0)
  const bool nb_above = (float)nb > q;
  return (above == nb_above) ? nb : h;
}

}  // namespace hifa4
