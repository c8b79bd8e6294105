// Packed-fp16 building blocks of the HIF4 quantizers (gfx950), shared by the
// attention kernels and the K/V pre-pass.
//
// HIF4 group quantization under the library's reading (the paper's HIF4
// paragraph in Background; Section 4.1): E6M2 base b = the smallest value with
// 1.75 b >= max|x|, level-2 and level-3 micro-exponents that halve the scale
// of 8- and 4-element blocks whose maximum fits in half of the range, element
// code u = round-half-away(|x| / step).  A group of 64 is held by a lane
// pair (l, l^32), 32 elements each as 16 packed fp16 pairs; every decision is
// taken on exact fp16 values: maxima with packed fp16 max, the base from the
// fp32 bits of the maximum, the shift of each 4-block by saturating 16-bit
// arithmetic on the bit patterns, and each magnitude rounded onto its grid by
// one mixed-precision fused multiply-add.
#pragma once

#include "hifa4_device.h"

namespace hifa4 {

// Lane-pair exchange with v_permlane32_swap(v, v): it swaps the upper 32
// lanes of the first copy with the lower 32 lanes of the second, so lanes
// 0..31 see (own, partner) and lanes 32..63 see (partner, own).  Symmetric
// combinations need no select.
struct Pair32 {
  uint32_t x, y;
};
__device__ __forceinline__ Pair32 pair32(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return Pair32{r[0], r[1]};
}
__device__ __forceinline__ h2_t max_with_partner(h2_t v) {
  const Pair32 p = pair32(__builtin_bit_cast(uint32_t, v));
  h2_t y;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(y) : "v"(p.x), "v"(p.y));
  return y;
}
__device__ __forceinline__ float add_with_partner(float v) {
  const Pair32 p = pair32(__builtin_bit_cast(uint32_t, v));
  return __builtin_bit_cast(float, p.x) + __builtin_bit_cast(float, p.y);
}
// The partner lane's value (h = lane / 32).
__device__ __forceinline__ h2_t partner_h2(h2_t v, int h) {
  const Pair32 p = pair32(__builtin_bit_cast(uint32_t, v));
  return __builtin_bit_cast(h2_t, h ? p.x : p.y);
}

// o = fp16(p*R + C) - C for both halves of p (fp16), R fp32 and C half SEL
// of cp (fp16).  The fused value is rounded once to fp16, onto the grid of C;
// the subtraction is exact.
template <int SEL>
__device__ __forceinline__ h2_t grid_round2(h2_t p, float R, h2_t cp) {
  h2_t y;
  if (SEL == 0)
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,0,1]\n\t"
        "v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,1]\n\t"
        "v_pk_add_f16 %0, %0, %3 op_sel:[0,0] op_sel_hi:[1,0] neg_lo:[0,1] neg_hi:[0,1]"
        : "=&v"(y)
        : "v"(p), "v"(R), "v"(cp));
  else
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel:[0,0,1] op_sel_hi:[1,0,1]\n\t"
        "v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,1] op_sel_hi:[1,0,1]\n\t"
        "v_pk_add_f16 %0, %0, %3 op_sel:[0,1] op_sel_hi:[1,1] neg_lo:[0,1] neg_hi:[0,1]"
        : "=&v"(y)
        : "v"(p), "v"(R), "v"(cp));
  return y;
}

// Rounding constants of a pair of 4-blocks (low / high half): with A4 the
// 4-block maximum, A8 its 8-block maximum and thr = (h, q) the fp16 floors of
// 0.875b and 0.4375b, the block's shift is sh = [A8 <= h] + [A4 <= (A8 <= h ?
// q : h)] = 2 - n with n = [A4 > h] + ([A8 > h] | [A4 > q]), and its constant
// 1.5 * 2^(k - sh) has the fp16 bits c0 + n * 0x400, c0 those of 1.5 * 2^(k-2)
// in both halves.  Non-negative fp16 values order like their bit patterns, so
// each test is a saturating 16-bit subtraction clamped to 1.
__device__ __forceinline__ h2_t grid_consts(h2_t a4, h2_t a8, h2_t thr, uint32_t c0) {
  h2_t n;
  uint32_t t, w;
  asm("v_pk_sub_u16 %0, %3, %5 op_sel:[0,0] op_sel_hi:[1,0] clamp\n\t"       // n = sat(A4 - h)
      "v_pk_sub_u16 %1, %4, %5 op_sel:[0,0] op_sel_hi:[1,0] clamp\n\t"       // t = sat(A8 - h)
      "v_pk_sub_u16 %2, %3, %5 op_sel:[0,1] op_sel_hi:[1,1] clamp\n\t"       // w = sat(A4 - q)
      "v_pk_max_u16 %1, %1, %2\n\t"
      "v_pk_min_u16 %0, %0, 1 op_sel_hi:[1,0]\n\t"
      "v_pk_min_u16 %1, %1, 1 op_sel_hi:[1,0]\n\t"
      "v_pk_add_u16 %0, %0, %1\n\t"
      "v_pk_mad_u16 %0, %0, %6, %7"
      : "=&v"(n), "=&v"(t), "=&v"(w)
      : "v"(a4), "v"(a8), "v"(thr), "s"(0x04000400u), "v"(c0));
  return n;
}
constexpr uint32_t kGrid10 = 0x5E005E00u;     // 1.5 * 2^8, both halves: the grids 2^-sh at 1.5 * 2^(10-sh)
constexpr uint32_t kGrid6 = 0x4E004E00u;      // 1.5 * 2^4: the grids 2^(-4-sh) at 1.5 * 2^(6-sh)

// (h, q) of a base: the fp16 floors of 0.875b and 0.4375b (round-toward-zero
// conversion); an fp16 value x satisfies x <= 0.875b iff x <= floor16(0.875b).
__device__ __forceinline__ h2_t range_floors(float b) {
  return __builtin_bit_cast(h2_t, __builtin_amdgcn_cvt_pkrtz(0.875f * b, 0.4375f * b));
}

// Packed fp16 max.  Written as an instruction so that the compiler does not
// canonicalize its (finite or -inf, never NaN) operands first.
__device__ __forceinline__ h2_t hmax2(h2_t a, h2_t b) {
  h2_t y;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(y) : "v"(a), "v"(b));
  return y;
}
// max of the two halves, in both halves
__device__ __forceinline__ h2_t hmax_halves(h2_t a) {
  h2_t y;
  asm("v_pk_max_f16 %0, %1, %1 op_sel:[0,1] op_sel_hi:[1,0]" : "=v"(y) : "v"(a));
  return y;
}
// max(a.lo, a.hi) in the low half and max(b.lo, b.hi) in the high half
// (two SDWA maxima in one block).
__device__ __forceinline__ h2_t hmax_pairs(h2_t a, h2_t b) {
  h2_t y;
  asm("v_max_f16_sdwa %0, %1, %1 dst_sel:WORD_0 dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n\t"
      "v_max_f16_sdwa %0, %2, %2 dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:WORD_0 src1_sel:WORD_1"
      : "=&v"(y)
      : "v"(a), "v"(b));
  return y;
}

// The value of lane l^32 through the LDS crossbar (ds_bpermute; `addr` is
// 4 * (l ^ 32)).  Used where several exchanges are independent so that their
// latency overlaps and the VALU stays free.
__device__ __forceinline__ uint32_t partner_bperm(uint32_t v, int addr) {
  return (uint32_t)__builtin_amdgcn_ds_bpermute(addr, (int)v);
}

// fp16(x * s) for both halves of x with per-half fp32 scales: the exact
// product rounded once (v_fma_mix with an fp16 destination).
__device__ __forceinline__ h2_t smooth_mul2(h2_t x, float s0, float s1) {
  h2_t y;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0 op_sel:[0,0,0] op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixhi_f16 %0, %1, %3, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
      : "=&v"(y)
      : "v"(x), "v"(s0), "v"(s1));
  return y;
}

// |x| for both halves (max(x, -x); the values are finite).
__device__ __forceinline__ h2_t habs2(h2_t x) {
  h2_t y;
  asm("v_pk_max_f16 %0, %1, %1 neg_lo:[0,1] neg_hi:[0,1]" : "=v"(y) : "v"(x));
  return y;
}

// max(a, b) for both halves, written as an instruction (no canonicalization).
__device__ __forceinline__ h2_t hmax2_q(h2_t a, h2_t b) {
  h2_t y;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(y) : "v"(a), "v"(b));
  return y;
}

// fp16 nearest to a float64 value (ties to even), rounded once: the value is
// first rounded to odd in fp32 (which keeps 13 more significand bits than
// fp16, enough for the second rounding to be exact), then to fp16.
__device__ __forceinline__ half_t rn16_from_f64(double x) {
  const float f = (float)x;
  uint32_t b = __float_as_uint(f);
  const double fd = (double)f;
  if (fd != x) {
    if (fabs(fd) > fabs(x)) b -= 1u;      // one fp32 step toward zero
    b |= 1u;                             // sticky bit: round to odd
  }
  return (half_t)__uint_as_float(b);
}

// Eight packed pairs of values 0 <= p <= 1 to whole units of 2^(E-7), rounded
// down: w = floor(p * 2^(7-E)) <= 392 for p <= 1.75b, b = (1 + m/4) 2^E.  The
// product with scale = 2^(-17-E) (low half) lands in fp16's subnormals, whose
// spacing 2^-24 is the unit, so one multiply in round-toward-zero mode
// truncates exactly; the mode holds inside the statement only.
__device__ __forceinline__ void floor_units8(const h2_t (&p)[8], h2_t scale, h2_t (&w)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) w[i] = p[i];
  asm("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3\n\t"
      "v_pk_mul_f16 %0, %0, %8 op_sel_hi:[1,0]\n\t"
      "v_pk_mul_f16 %1, %1, %8 op_sel_hi:[1,0]\n\t"
      "v_pk_mul_f16 %2, %2, %8 op_sel_hi:[1,0]\n\t"
      "v_pk_mul_f16 %3, %3, %8 op_sel_hi:[1,0]\n\t"
      "v_pk_mul_f16 %4, %4, %8 op_sel_hi:[1,0]\n\t"
      "v_pk_mul_f16 %5, %5, %8 op_sel_hi:[1,0]\n\t"
      "v_pk_mul_f16 %6, %6, %8 op_sel_hi:[1,0]\n\t"
      "v_pk_mul_f16 %7, %7, %8 op_sel_hi:[1,0]\n\t"
      "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 0"
      : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), "+v"(w[7])
      : "v"(scale));
}

// o/16 = fp16(w*R + C) - C for both halves of w, R the low half of `r` and C
// half SEL of cp.
template <int SEL>
__device__ __forceinline__ h2_t grid_round_units(h2_t w, h2_t r, h2_t cp) {
  h2_t y;
  if (SEL == 0)
    asm("v_pk_fma_f16 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,0,0]\n\t"
        "v_pk_add_f16 %0, %0, %3 op_sel:[0,0] op_sel_hi:[1,0] neg_lo:[0,1] neg_hi:[0,1]"
        : "=&v"(y)
        : "v"(w), "v"(r), "v"(cp));
  else
    asm("v_pk_fma_f16 %0, %1, %2, %3 op_sel:[0,0,1] op_sel_hi:[1,0,1]\n\t"
        "v_pk_add_f16 %0, %0, %3 op_sel:[0,1] op_sel_hi:[1,1] neg_lo:[0,1] neg_hi:[0,1]"
        : "=&v"(y)
        : "v"(w), "v"(r), "v"(cp));
  return y;
}

// P^ = HIF4(P) of one 64-key block held in the S^T accumulator layout (lane
// half h holds keys 32t + 8j + 4h + [0,4) of 4-block (t, j) in the packed
// registers p2[t][2j], p2[t][2j+1]; the 8-blocks pair with lane l^32).  A is
// the block maximum (an fp16 value, at most 1).  Returns the operand values
// o/16 = u * 2^(-4-sh) (kPScale) in the order of the packed registers (slot
// 16t + 2v2 + e = half e of p2[t][v2]) and the base value b (0 where A is 0).
// With DEBUG, a non-null dcodes / dmeta receive the lane's share of the
// canonical codes and the metadata word.
//
// Rounding on packed fp16 alone.  Every threshold (u - 1/2) step of the
// codes is a whole number T = (2u-1)(4+m) 2^(2-sh) <= 364 of units 2^(E-7),
// so truncating P to whole units (floor_units8) moves no value across one.
// u 2^-sh / 16 is then w 2^-24 * R on the grid 2^(-4-sh), R = 2^15 / (1+m/4)
// taken just above as an fp16 (relative excess eps, 2^-12 < eps <= 2^-10):
// w = T lands above the half and rounds up (half away from zero),
// w <= T - 1 stays below it since eps < 1/363.  Three packed instructions per
// pair (12 cycles) against two mixed-precision fused multiply-adds of 8 cycles
// each and a subtraction: the block's rounding takes 192 instead of 320 issue
// cycles, and the attention kernels are bound by these.
constexpr float kPScale = 0.0625f;
struct PQuant {
  h32_t ov;
  float bval;
};

template <bool DEBUG>
__device__ __forceinline__ PQuant quantize_p_block(const h2_t (&p2)[2][8], float A, int lane, int h, uint8_t* dcodes,
                                                   uint32_t* dmeta) {
  PQuant out;
  // Maxima are packed in pairs of 4-blocks: a4[t][jp] = (A4(t, 2jp), A4(t, 2jp+1)).
  h2_t cst[2][2];       // rounding constants of 4-blocks (t, 2jp), (t, 2jp+1)
  h2_t a4s[2][2], a4p[2][2];
  const int paddr = 4 * (lane ^ 32);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int jp = 0; jp < 2; ++jp) {
      const h2_t m0 = hmax2(p2[t][4 * jp], p2[t][4 * jp + 1]);       // 4-block 2jp, two partial maxima
      const h2_t m1 = hmax2(p2[t][4 * jp + 2], p2[t][4 * jp + 3]);   // 4-block 2jp+1
      a4s[t][jp] = hmax_pairs(m0, m1);
      a4p[t][jp] = __builtin_bit_cast(h2_t, partner_bperm(__builtin_bit_cast(uint32_t, a4s[t][jp]), paddr));
    }
  const uint32_t bb = e6m2_cover_bits(A);
  out.bval = __uint_as_float(bb);
  // 2^(-17-E) as fp16 (b = 0: the largest fp16, which multiplies zeros)
  const float sc = __uint_as_float((237u << 23) - (bb & 0x7F800000u));
  const h2_t scale = __builtin_bit_cast(h2_t, __builtin_amdgcn_cvt_pkrtz(sc, sc));
  // R of the four mantissas m: 32800, 26224, 21856, 18736 as fp16, picked by byte
  const uint32_t m = (bb >> 21) & 3u;
  const h2_t R = __builtin_bit_cast(
      h2_t, __builtin_amdgcn_perm(0x74937556u, 0x76677801u, __umul24(m, 0x0202u) + 0x0C0C0100u));
  const h2_t thr = range_floors(out.bval);
  uint32_t c0;          // written here so that it holds no register between blocks
  asm volatile("v_mov_b32 %0, %1" : "=v"(c0) : "i"(kGrid6));
  uint32_t e2bits = 0, e3bits = 0;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int jp = 0; jp < 2; ++jp) {
      const h2_t a4 = a4s[t][jp];
      const h2_t a8 = hmax2(a4, a4p[t][jp]);
      cst[t][jp] = grid_consts(a4, a8, thr, c0);
      if (DEBUG) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int j = 2 * jp + e;
          const bool e2 = a8[e] <= thr[0];
          const bool e3 = a4[e] <= (e2 ? thr[1] : thr[0]);
          e2bits |= (uint32_t)e2 << (4 * t + j);
          e3bits |= (uint32_t)e3 << (8 * t + 2 * j + h);
          const bool e3o = a4p[t][jp][e] <= (e2 ? thr[1] : thr[0]);
          e3bits |= (uint32_t)e3o << (8 * t + 2 * j + (h ^ 1));
        }
      }
    }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    h2_t w[8];
    floor_units8(p2[t], scale, w);
#pragma unroll
    for (int v2 = 0; v2 < 8; ++v2) {
      // 4-block j = v2/2 of tile t: its constant is half (j & 1) of cst[t][j >> 1]
      const h2_t cp = cst[t][v2 >> 2];
      const h2_t tt = ((v2 >> 1) & 1) ? grid_round_units<1>(w[v2], R, cp) : grid_round_units<0>(w[v2], R, cp);
      out.ov[16 * t + 2 * v2] = tt[0];
      out.ov[16 * t + 2 * v2 + 1] = tt[1];
    }
  }
  if (DEBUG && dcodes) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q4 = 8 * t + 2 * j + h;
        const int sh = (int)((e2bits >> (4 * t + j)) & 1u) + (int)((e3bits >> q4) & 1u);
        uint32_t nib[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) nib[i] = (uint32_t)((float)out.ov[16 * t + 4 * j + i] * (float)(16 << sh));
        dcodes[16 * t + 4 * j + 2 * h] = (uint8_t)(nib[0] | (nib[1] << 4));
        dcodes[16 * t + 4 * j + 2 * h + 1] = (uint8_t)(nib[2] | (nib[3] << 4));
      }
    if (h == 0) *dmeta = e6m2_code_of(bb) | (e2bits << 8) | (e3bits << 16);
  }
  return out;
}

// The quantizer's output for one lane: its 32 FP6 E2M3 fields, the group's
// E6M2 base byte and base value.
struct GroupOps {
  i6_t pk;
  uint32_t base;
  float bval;
};

// HIF4 of a group in row layout: lane half h holds elements 32h..32h+31 as
// x[i] = (element 32h+2i, 32h+2i+1), i.e. 4-blocks 8h..8h+7 and 8-blocks
// 4h..4h+3, so only the group maximum needs the partner lane.  FP6 slot s =
// element 32h + s, value +-u*2^-sh (a negative value whose code is 0 becomes
// -0, which the MFMA treats as 0).  Used for Q and K along the head dimension.
__device__ __forceinline__ GroupOps rows_quantize(const h2_t (&x)[16]) {
  h2_t ax[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) ax[i] = habs2(x[i]);
  // 4-block k = pairs 2k, 2k+1; a4p[j] = (A4[2j], A4[2j+1]) = 8-block j's halves
  h2_t a4p[4], a8[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const h2_t m0 = hmax2_q(ax[4 * j], ax[4 * j + 1]);
    const h2_t m1 = hmax2_q(ax[4 * j + 2], ax[4 * j + 3]);
    a4p[j] = hmax_pairs(m0, m1);
    a8[j] = hmax_halves(a4p[j]);
  }
  const h2_t lane_max = hmax2_q(hmax2_q(a8[0], a8[1]), hmax2_q(a8[2], a8[3]));
  const h2_t gmax = max_with_partner(lane_max);
  const float A = (float)gmax[0];
  GroupOps r;
  r.base = e6m2_ceil(A);
  r.bval = e6m2_value(r.base);
  const float R = hif4_rcp_step(r.base);
  const h2_t thr = range_floors(r.bval);
  h32_t ov;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const h2_t cst = grid_consts(a4p[j], a8[j], thr, kGrid10);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 4 * j + e;                 // pair i belongs to 4-block 2j + e/2
      const h2_t o = (e >> 1) ? grid_round2<1>(ax[i], R, cst) : grid_round2<0>(ax[i], R, cst);
      const uint32_t sgn = __builtin_bit_cast(uint32_t, x[i]) & 0x80008000u;
      const h2_t os = __builtin_bit_cast(h2_t, __builtin_bit_cast(uint32_t, o) | sgn);
      ov[2 * i] = os[0];
      ov[2 * i + 1] = os[1];
    }
  }
  r.pk = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(ov, 1.0f);
  return r;
}

// HIF4 of a signed group in key layout (that of P^ in the S^T accumulator:
// x[t][v2] holds elements 32t + 8(v2/2) + 4h + 2(v2%2) + {0, 1}; 8-blocks pair
// with lane l^32).  FP6 slot 16t + 2v2 + e = half e of x[t][v2].  Used for V
// along tokens.
__device__ __forceinline__ GroupOps keys_quantize(const h2_t (&x)[2][8], int lane, int h) {
  h2_t ax[2][8];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v2 = 0; v2 < 8; ++v2) ax[t][v2] = habs2(x[t][v2]);
  h2_t m = ax[0][0];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v2 = 0; v2 < 8; ++v2)
      if (t > 0 || v2 > 0) m = hmax2_q(m, ax[t][v2]);
  const h2_t gmax = hmax_halves(max_with_partner(m));
  GroupOps r;
  r.base = e6m2_ceil((float)gmax[0]);
  r.bval = e6m2_value(r.base);
  const float R = hif4_rcp_step(r.base);
  const h2_t thr = range_floors(r.bval);
  const int paddr = 4 * (lane ^ 32);
  h2_t a4s[2][2], a4p[2][2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int jp = 0; jp < 2; ++jp) {
      a4s[t][jp] = hmax_pairs(hmax2(ax[t][4 * jp], ax[t][4 * jp + 1]), hmax2(ax[t][4 * jp + 2], ax[t][4 * jp + 3]));
      a4p[t][jp] = __builtin_bit_cast(h2_t, partner_bperm(__builtin_bit_cast(uint32_t, a4s[t][jp]), paddr));
    }
  h32_t ov;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v2 = 0; v2 < 8; ++v2) {
      const int jp = v2 >> 2;
      const h2_t cst = grid_consts(a4s[t][jp], hmax2(a4s[t][jp], a4p[t][jp]), thr, kGrid10);
      const h2_t o = ((v2 >> 1) & 1) ? grid_round2<1>(ax[t][v2], R, cst) : grid_round2<0>(ax[t][v2], R, cst);
      const uint32_t sgn = __builtin_bit_cast(uint32_t, x[t][v2]) & 0x80008000u;
      const h2_t os = __builtin_bit_cast(h2_t, __builtin_bit_cast(uint32_t, o) | sgn);
      ov[16 * t + 2 * v2] = os[0];
      ov[16 * t + 2 * v2 + 1] = os[1];
    }
  r.pk = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(ov, 1.0f);
  return r;
}

}  // namespace hifa4
