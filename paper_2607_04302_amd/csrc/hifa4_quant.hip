// HIF4 quantization kernels: canonical Q^/K^/V^ outputs, the attention
// pre-pass that writes MFMA-ready K and V operands, calibration reductions,
// and the exponential self-test.
//
// Paper: Algorithm 1 (Smooth-QK step, HIF4 of Q, K, V); Eq. 1 (q*s, k/s
// after RoPE); Appendix C (GQA: s is per key-head channel).
#include "hifa4_device.h"
#include "hifa4_internal.h"
#include "hifa4_packed.h"

#include <algorithm>

namespace hifa4 {

// Token index (row of the [T, H, D] view) of position i in sequence b.
__device__ __forceinline__ int seq_start(const int* cu, int b, int S) {
  return cu ? cu[b] : b * S;
}
// a length above max_seqlen is outside the contract; clamping it keeps every
// access inside the caller's buffers
__device__ __forceinline__ int seq_len(const int* cu, int b, int S) {
  return cu ? min(cu[b + 1] - cu[b], S) : S;
}

// Packed-fp16 pieces of the canonical quantizers.
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u16x2_t as_u16(h2_t x) { return __builtin_bit_cast(u16x2_t, x); }

// Level-2 and level-3 decisions of both halves of a pair of 4-block maxima a4
// whose 8-block maxima are a8, against the half- and quarter-range floors
// (per half): n = 2 - (E2 + E3) and the complement of E2, as 0..2 and 0..1 in
// 16-bit halves (non-negative fp16 values order like their bit patterns).
__device__ __forceinline__ void block_levels(h2_t a4, h2_t a8, h2_t th_h, h2_t th_q, u16x2_t& n, u16x2_t& not_e2) {
  const u16x2_t one = {1, 1};
  const u16x2_t big4 = __builtin_elementwise_min(__builtin_elementwise_sub_sat(as_u16(a4), as_u16(th_h)), one);
  not_e2 = __builtin_elementwise_min(__builtin_elementwise_sub_sat(as_u16(a8), as_u16(th_h)), one);
  const u16x2_t quarter = __builtin_elementwise_min(__builtin_elementwise_sub_sat(as_u16(a4), as_u16(th_q)), one);
  n = big4 + __builtin_elementwise_max(not_e2, quarter);
}

// fp16(a*R + C) per half (R fp32 per half, C fp16 per half): the code u sits in
// the low mantissa bits, since C = 1.5 * 2^(10-sh) has the grid 2^-sh as its
// last place.  Returns u in 0..7 per half.
__device__ __forceinline__ uint32_t codes2(h2_t a, float r0, float r1, u16x2_t n) {
  const u16x2_t c = n * (unsigned short)0x400 + (unsigned short)(kGrid10 & 0xFFFFu);
  h2_t y;
  asm("v_fma_mixlo_f16 %0, %1, %2, %4 op_sel:[0,0,0] op_sel_hi:[1,0,1]\n\t"
      "v_fma_mixhi_f16 %0, %1, %3, %4 op_sel:[1,0,1] op_sel_hi:[1,0,1]"
      : "=&v"(y)
      : "v"(a), "v"(r0), "v"(r1), "v"(__builtin_bit_cast(uint32_t, c)));
  return __builtin_bit_cast(uint32_t, y) & 0x00070007u;
}

// Sign-magnitude nibbles of both halves: u | sign << 3, a zero code without a
// sign (u + 7 carries into bit 3 exactly where u > 0).
__device__ __forceinline__ uint32_t nibbles2(uint32_t u, h2_t x) {
  const uint32_t s = (__builtin_bit_cast(uint32_t, x) >> 12) & 0x00080008u;
  return u | ((u + 0x00070007u) & s);
}

// fp16(k/s) for a pair of fp16 values from r0, r1 = RN32(1/s) of each: with the
// reciprocal taken two units in the last place (ulps) down and up, the fp32
// products bracket the exact quotient (two ulps exceed the reciprocal's half
// ulp and the product's rounding together), so where both ends round to the
// same fp16 the quotient does too.  `open` collects the bits in which they
// differ (about one value in 2000): those take the exact division.
__device__ __forceinline__ h2_t divide2(h2_t k, float r0, float r1, uint32_t& open) {
  const float d0 = __uint_as_float(__float_as_uint(r0) - 2u), u0 = __uint_as_float(__float_as_uint(r0) + 2u);
  const float d1 = __uint_as_float(__float_as_uint(r1) - 2u), u1 = __uint_as_float(__float_as_uint(r1) + 2u);
  float a, b, c, d;
  asm("v_fma_mix_f32 %0, %4, %5, 0 op_sel:[0,0,0] op_sel_hi:[1,0,0]\n\t"
      "v_fma_mix_f32 %1, %4, %6, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\t"
      "v_fma_mix_f32 %2, %4, %7, 0 op_sel:[0,0,0] op_sel_hi:[1,0,0]\n\t"
      "v_fma_mix_f32 %3, %4, %8, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
      : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d)
      : "v"(k), "v"(d0), "v"(d1), "v"(u0), "v"(u1));
  const h2_t lo = pack2_f16(a, b), hi = pack2_f16(c, d);
  open |= __builtin_bit_cast(uint32_t, lo) ^ __builtin_bit_cast(uint32_t, hi);
  return lo;
}

// fp16(k/s) of N pairs: s and rs are the scales and their reciprocals.
template <int N, typename S>
__device__ __forceinline__ void divide_pairs(h2_t (&x)[N], const S& s, const S& rs) {
  h2_t y[N];
  uint32_t any = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) y[i] = divide2(x[i], rs[2 * i], rs[2 * i + 1], any);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(any != 0) != 0, 0)) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      uint32_t open = 0;
      divide2(x[i], rs[2 * i], rs[2 * i + 1], open);
      if (open) y[i] = h2_t{div_rn16((float)x[i][0], s[2 * i]), div_rn16((float)x[i][1], s[2 * i + 1])};
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = y[i];
}

// Reductions over aligned sets of eight lanes (quad permutes, then the mirror
// of eight, which pairs the two quads).
template <typename F>
__device__ __forceinline__ uint32_t reduce8(uint32_t v, F f) {
  v = f(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
  v = f(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
  return f(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true));  // row_half_mirror
}

// ---------------------------------------------------------------------------
// Canonical Q^ / K^ (hifa4_quantize_qk).  Eight lanes per group: a lane holds
// one 8-block (16 bytes of input, 4 bytes of codes), so a wave reads 1 KiB and
// writes 256 bytes of codes in one piece each, E2 and E3 stay in the lane and
// only the group maximum and the metadata word are reduced over the eight
// lanes.  Bound by HBM (164 bytes moved per group).  A thread steps over the
// rows at a stride that is a whole number of rows, so it keeps its column's
// smoothing scales and reciprocals in registers, with kRowsAhead loads in
// flight.  The K^ of 8 x 4096 tokens of 8 heads, D=128, took 84 us with a lane
// pair per group (64-byte steps between lanes, fp32 arithmetic, a division per
// element).
constexpr int kRowsAhead = 4;

template <bool kIsK>
__global__ void __launch_bounds__(256) k_quant_rows(const half_t* __restrict__ x, const float* __restrict__ s,
                                                    uint8_t* __restrict__ codes, uint32_t* __restrict__ meta,
                                                    long n_pieces, long stride, int heads, int heads_kv, int D) {
  const long tid = (long)blockIdx.x * 256 + threadIdx.x;
  if (tid >= stride) return;                  // whole sets of eight lanes exit together
  const int j = threadIdx.x & 7;
  float sc[8], rc[8];
  if (s) {
    const int ch = (int)(tid % (heads * D / 8)) * 8;
    const int hk = (ch / D) / (heads / heads_kv);
    const float4* sp = reinterpret_cast<const float4*>(s + (size_t)hk * D + ch % D);
    const float4 a = sp[0], b = sp[1];
    const float t[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sc[i] = t[i];
      rc[i] = kIsK ? 1.0f / t[i] : 0.0f;
    }
  }
  for (long i0 = tid; i0 < n_pieces; i0 += kRowsAhead * stride) {
    uint4 in[kRowsAhead];
#pragma unroll
    for (int r = 0; r < kRowsAhead; ++r) {
      const long i = i0 + r * stride;
      in[r] = *reinterpret_cast<const uint4*>(x + 8 * (i < n_pieces ? i : tid));
    }
#pragma unroll
    for (int r = 0; r < kRowsAhead; ++r) {
      const long i = i0 + r * stride;
      if (i >= n_pieces) break;               // whole sets of eight lanes again (n_pieces is a multiple of 8)
      h2_t v[4] = {__builtin_bit_cast(h2_t, in[r].x), __builtin_bit_cast(h2_t, in[r].y),
                   __builtin_bit_cast(h2_t, in[r].z), __builtin_bit_cast(h2_t, in[r].w)};
      if (s) {
        if (kIsK) {
          divide_pairs(v, sc, rc);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = smooth_mul2(v[e], sc[2 * e], sc[2 * e + 1]);
        }
      }
      h2_t a[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = habs2(v[e]);
      const h2_t a4 = hmax_pairs(hmax2(a[0], a[1]), hmax2(a[2], a[3]));     // both 4-blocks
      // (integer maxima here: the lane exchanges read registers right after they
      // are written, which the compiler must be able to see)
      const u16x2_t a8u = __builtin_elementwise_max(as_u16(a4), __builtin_shufflevector(as_u16(a4), as_u16(a4), 1, 0));
      const h2_t a8 = __builtin_bit_cast(h2_t, a8u);
      const uint32_t gm = reduce8(__builtin_bit_cast(uint32_t, a8u), [](uint32_t p, uint32_t q) {
        return __builtin_bit_cast(
            uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, p), __builtin_bit_cast(u16x2_t, q)));
      });
      const uint32_t base = e6m2_ceil((float)__builtin_bit_cast(h2_t, gm)[0]);
      const float R = hif4_rcp_step(base);
      const h2_t thr = range_floors(e6m2_value(base));
      u16x2_t n, ne2;
      block_levels(a4, a8, h2_t{thr[0], thr[0]}, h2_t{thr[1], thr[1]}, n, ne2);
      uint32_t word = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned short ne = n[e >> 1];
        const uint32_t nib = nibbles2(codes2(a[e], R, R, u16x2_t{ne, ne}), v[e]);
        word |= ((nib | (nib >> 12)) & 0xFFu) << (8 * e);
      }
      reinterpret_cast<uint32_t*>(codes)[i] = word;
      // E2 = 1 - ne2, E3 = 2 - n - E2 per 4-block
      const uint32_t e2 = 1u - ne2[0];
      const uint32_t e3 = (2u - n[0] - e2) | ((2u - n[1] - e2) << 1);
      const uint32_t bits = reduce8((e2 << (8 + j)) | (e3 << (16 + 2 * j)), [](uint32_t p, uint32_t q) { return p | q; });
      if (j == 0) meta[i >> 3] = base | bits;
    }
  }
}

// ---------------------------------------------------------------------------
// Canonical V^ (hifa4_quantize_v): group = 64 tokens of one (kv head, channel)
// column, aligned to the sequence start.  A lane holds four consecutive
// columns (of the heads_kv * D of a token) and 32 of the group's tokens; lane
// l^32 holds the other 32.  Both halves of every packed register are two
// channels, so all decisions but the group maximum stay in the lane; a load
// reads two whole 256-byte runs of columns per wave, all 32 issued before the
// first is used.  Bound by HBM (the groups' 128 bytes in, 36 out).  V^ of 8 x
// 4096 tokens of 8 heads, D=128, took 41 us with a lane per channel reading 2
// bytes at a time.
__global__ void __launch_bounds__(256) k_quant_v_canon(const half_t* __restrict__ v, const int* __restrict__ cu,
                                                       uint8_t* __restrict__ codes, uint32_t* __restrict__ meta,
                                                       int batch, int S, int NB, int cols) {
  const int lane = threadIdx.x & 63;
  const int h = lane >> 5;
  const long item = ((long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 32 + (lane & 31);
  const int per_block = cols / 4;
  if (item >= (long)batch * NB * per_block) return;      // whole lane pairs
  const int c0 = 4 * (int)(item % per_block);
  const int J = (int)((item / per_block) % NB);
  const int b = (int)(item / per_block / NB);
  const int t0 = seq_start(cu, b, S);
  const int L = seq_len(cu, b, S);
  const int p0 = 64 * J + 32 * h;
  h2_t x[32][2];
  if (64 * J < L) {
    uint2 in[32];
#pragma unroll
    for (int k = 0; k < 32; ++k)
      in[k] = *reinterpret_cast<const uint2*>(v + (size_t)(t0 + min(p0 + k, L - 1)) * cols + c0);
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const bool live = p0 + k < L;
      x[k][0] = __builtin_bit_cast(h2_t, live ? in[k].x : 0u);
      x[k][1] = __builtin_bit_cast(h2_t, live ? in[k].y : 0u);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 32; ++k) x[k][0] = x[k][1] = h2_t{(half_t)0, (half_t)0};
  }
  const size_t g0 = (size_t)item * 4;                     // first of the lane's four groups
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    h2_t a4[8], gm = {(half_t)0, (half_t)0};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      a4[q] = hmax2(hmax2(habs2(x[4 * q][w]), habs2(x[4 * q + 1][w])),
                    hmax2(habs2(x[4 * q + 2][w]), habs2(x[4 * q + 3][w])));
      gm = hmax2(gm, a4[q]);
    }
    gm = max_with_partner(gm);
    const uint32_t base0 = e6m2_ceil((float)gm[0]), base1 = e6m2_ceil((float)gm[1]);
    const float r0 = hif4_rcp_step(base0), r1 = hif4_rcp_step(base1);
    const h2_t f0 = range_floors(e6m2_value(base0)), f1 = range_floors(e6m2_value(base1));
    const h2_t th_h = {f0[0], f1[0]}, th_q = {f0[1], f1[1]};
    uint32_t acc[8];           // four tokens' nibbles per half
    uint32_t lev = 0;          // per half: E2 of the lane's four 8-blocks, then E3 of its eight 4-blocks
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      u16x2_t n, ne2;
      block_levels(a4[q], hmax2(a4[q & ~1], a4[q | 1]), th_h, th_q, n, ne2);
      acc[q] = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[q] |= nibbles2(codes2(habs2(x[4 * q + i][w]), r0, r1, n), x[4 * q + i][w]) << (4 * i);
      const uint32_t e2 = 0x00010001u - __builtin_bit_cast(uint32_t, ne2);
      if ((q & 1) == 0) lev |= e2 << (q >> 1);
      lev |= (0x00020002u - __builtin_bit_cast(uint32_t, n) - e2) << (4 + q);
    }
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      lo[d] = __builtin_amdgcn_perm(acc[2 * d + 1], acc[2 * d], 0x05040100u);
      hi[d] = __builtin_amdgcn_perm(acc[2 * d + 1], acc[2 * d], 0x07060302u);
    }
    uint8_t* dst = codes + (g0 + 2 * w) * 32 + 16 * h;
    *reinterpret_cast<uint4*>(dst) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    *reinterpret_cast<uint4*>(dst + 32) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    const Pair32 pl = pair32(lev);                        // x: tokens 0..31, y: tokens 32..63
    const uint32_t l0 = h ? pl.x >> 16 : pl.x, l1 = h ? pl.y >> 16 : pl.y;      // lane half h writes channel 2w + h
    meta[g0 + 2 * w + h] = (h ? base1 : base0) | ((l0 & 0xFu) << 8) | ((l1 & 0xFu) << 12) | (((l0 >> 4) & 0xFFu) << 16) |
                           (((l1 >> 4) & 0xFFu) << 24);
  }
}

// ---------------------------------------------------------------------------
// Attention pre-pass (HIF4 operands).  Two workgroups of 2G waves per
// (sequence b, kv head, 64-key block J): in the K workgroup wave w quantizes
// K half-tile t = w/G, group g = w%G; in the V workgroup wave w quantizes V
// channel tile w.
// Writes, for the chunk:
//   K operands [2 halves][G groups][2] operand records (64 lanes x dwords
//     0..3, then 64 lanes x dwords 4..5 of the lane's 6): lane l holds key
//     32t + l%32 and channels 64g + 32(l/32) + [0,32) in FP6 E2M3, i.e. the
//     A operand of S^T = K^ Q^T for the 32x32x64 MFMA, as the two operands of
//     the key's split base (below);
//   K scale words [2][G][32]: their two E8M0 bytes per key and group;
//   V operands [D/32 tiles][2] operand records: lane l holds channel
//     32dt + l%32 and, at FP6 slot s, the key 32(s/16) + 8((s%16)/4) +
//     4(l/32) + s%4 -- the key order in which the attention kernel's P^
//     operand arrives (the S^T accumulator registers of both 32-key halves in
//     order) -- again as the two operands of the split base;
//   V scale words [D]: their two E8M0 bytes per channel.
// Two-operand form of a HIF4 group for the FP6 MFMA.  The base
// b = (1 + m/4) 2^(e-31) is not an E8M0 power of two, so the group's codes
// enter two MFMAs whose E8M0 scales add up to b/4 exactly:
//   m = 0:  1    = 1                 operand B all zero
//   m = 1:  1.25 = 1 + 1/4           B = codes,          scale 2^(e-35)
//   m = 2:  1.5  = 1 + 1/2           B = codes,          scale 2^(e-34)
//   m = 3:  1.75 = 2 - 1/4           B = negated codes,  scale 2^(e-35)
// operand A = codes with scale 2^(e-33), or 2^(e-32) for m = 3.  The E8M0
// byte of 2^k is k + 127.  Byte 0 of the scale word serves operand A, byte 1
// operand B.
__device__ __forceinline__ uint32_t split_scale_word(uint32_t base) {
  const uint32_t e = base >> 2, m = base & 3u;
  const uint32_t sa = e + 94u + (m == 3u ? 1u : 0u);
  const uint32_t sb = e + (m == 2u ? 93u : 92u);
  return sa | (sb << 8);
}

// Stores a lane's operand A (its 24 code bytes) into the operand record at
// rec and operand B into the next record.  A record holds dwords 0..3 of the
// 64 lanes (16 bytes each), then dwords 4..5 (8 bytes each).  The E2M3 sign is
// bit 5 of each 6-bit field.
__device__ __forceinline__ void store_split_operand(uint8_t* rec, int lane, const i6_t& pk, uint32_t base) {
  constexpr uint32_t kSign[3] = {0x20820820u, 0x08208208u, 0x82082082u};   // fields 6s+5, period 96 bits
  const uint32_t m = base & 3u;
  uint32_t wa[6], wb[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    wa[i] = (uint32_t)pk[i];
    wb[i] = m == 0u ? 0u : (m == 3u ? wa[i] ^ kSign[i % 3] : wa[i]);
  }
  *reinterpret_cast<uint4*>(rec + 16 * lane) = make_uint4(wa[0], wa[1], wa[2], wa[3]);
  *reinterpret_cast<uint2*>(rec + 1024 + 8 * lane) = make_uint2(wa[4], wa[5]);
  *reinterpret_cast<uint4*>(rec + kOpRecord + 16 * lane) = make_uint4(wb[0], wb[1], wb[2], wb[3]);
  *reinterpret_cast<uint2*>(rec + kOpRecord + 1024 + 8 * lane) = make_uint2(wb[4], wb[5]);
}

__global__ void __launch_bounds__(512) k_prep_kv_hif4(const half_t* __restrict__ k, const half_t* __restrict__ v,
                                                      const float* __restrict__ s, const int* __restrict__ cu,
                                                      uint8_t* __restrict__ ws, int S, int NB, int heads_kv, int G,
                                                      bool qmean) {
  // workgroup (J, hk, 2b + role): role 0 quantizes K, role 1 V, of block J
  extern __shared__ __align__(16) uint8_t sm[];
  const int J = blockIdx.x, hk = blockIdx.y, b = blockIdx.z >> 1;
  const bool is_v = (blockIdx.z & 1) != 0;
  const int D = 64 * G;
  const int t0 = seq_start(cu, b, S);
  const int L = seq_len(cu, b, S);
  if (64 * J >= L) return;
  const ChunkLayout lay = chunk_layout_hif4(G, qmean);
  uint8_t* chunk = ws + ((size_t)(b * heads_kv + hk) * NB + J) * lay.bytes;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5;
  if (!is_v) {
    const int t = wave / G, g = wave % G;
    const int key = 32 * t + (lane & 31);
    const int pos = 64 * J + key;
    // the key's 32 channels 64g + 32h + [0, 32) as 16 fp16 pairs, requested
    // before the smoothing scales are staged so that both loads overlap
    h2_t x[16];
    if (pos < L) {
      typedef uint32_t u4v_t __attribute__((ext_vector_type(4)));
      const u4v_t* src = reinterpret_cast<const u4v_t*>(k + ((size_t)(t0 + pos) * heads_kv + hk) * D + 64 * g + 32 * h);
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const u4v_t w = src[v4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t wi = w[i];     // copy first: bit-casting an ext_vector element in place misreads it
          x[4 * v4 + i] = __builtin_bit_cast(h2_t, wi);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = h2_t{(half_t)0, (half_t)0};
    }
    if (s) {
      // this head's smoothing scales and their reciprocals (one division per
      // channel), staged in LDS; then k~ = fp16(k/s) per element
      float* rs = reinterpret_cast<float*>(sm);
      float* ss = rs + D;
      for (int c = threadIdx.x; c < D; c += blockDim.x) {
        const float sc = s[(size_t)hk * D + c];
        ss[c] = sc;
        rs[c] = 1.0f / sc;
      }
      __syncthreads();
      const float* sc = ss + 64 * g + 32 * h;
      const float* rc = rs + 64 * g + 32 * h;
      divide_pairs(x, sc, rc);
    }
    if (qmean) {
      // Q-Mean key sums (Algorithm 1's correction term): the exact sum of the
      // key's smoothed channels in float64 (any 256 fp16 values sum exactly),
      // one partial per (32-key half, group) in LDS, then rounded once to fp32.
      double part = 0.0;
#pragma unroll
      for (int i = 0; i < 16; ++i) part += (double)(float)x[i][0] + (double)(float)x[i][1];
      part += __shfl_xor(part, 32);
      double* parts = reinterpret_cast<double*>(sm + 2 * D * sizeof(float));     // [2][G][32]
      if (h == 0) parts[(t * G + g) * 32 + (lane & 31)] = part;
      __syncthreads();
      if (g == 0 && h == 0) {
        double sum = 0.0;
        for (int gg = 0; gg < G; ++gg) sum += parts[(t * G + gg) * 32 + (lane & 31)];
        reinterpret_cast<float*>(chunk + lay.kappa)[32 * t + (lane & 31)] = (float)sum;
      }
    }
    const GroupOps go = rows_quantize(x);
    store_split_operand(chunk + lay.k_op + (size_t)(t * G + g) * 2 * kOpRecord, lane, go.pk, go.base);
    if (h == 0)
      reinterpret_cast<uint32_t*>(chunk + lay.k_scale)[(t * G + g) * 32 + (lane & 31)] = split_scale_word(go.base);
  } else {
    // stage V rows [64J, 64J+64) of this head, zero past the sequence end:
    // 64 * D / 8 pieces of 16 bytes, 4 per thread, all loads issued before
    // the first store (rows past the end load the last row, then store zero)
    half_t* vt = reinterpret_cast<half_t*>(sm);        // [64 keys][D]
    const int pieces_per_row = D / 8;
    uint4 val[4];
    bool live[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = threadIdx.x + r * blockDim.x;
      const int pos = 64 * J + i / pieces_per_row;
      live[r] = pos < L;
      const int row = live[r] ? pos : L - 1;             // L > 64 J >= 0 here
      val[r] = *reinterpret_cast<const uint4*>(v + ((size_t)(t0 + row) * heads_kv + hk) * D +
                                               8 * (i % pieces_per_row));
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      reinterpret_cast<uint4*>(vt)[threadIdx.x + r * blockDim.x] = live[r] ? val[r] : make_uint4(0, 0, 0, 0);
    __syncthreads();
    const int dt = wave;
    const int d = 32 * dt + (lane & 31);
    // the lane's 32 keys in the order of the attention kernel's P^ operand:
    // x[t][v2] = keys 32t + 8(v2/2) + 4h + 2(v2%2) + {0, 1} of channel d
    h2_t x[2][8];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v2 = 0; v2 < 8; ++v2) {
        const int k0 = 32 * t + 8 * (v2 >> 1) + 4 * h + 2 * (v2 & 1);
        x[t][v2] = h2_t{vt[k0 * D + d], vt[(k0 + 1) * D + d]};
      }
    const GroupOps go = keys_quantize(x, lane, h);
    store_split_operand(chunk + lay.v_op + (size_t)dt * 2 * kOpRecord, lane, go.pk, go.base);
    if (h == 0) reinterpret_cast<uint32_t*>(chunk + lay.v_scale)[d] = split_scale_word(go.base);
  }
}

// ---------------------------------------------------------------------------
// Attention pre-pass (FP16 operands, the C16V16 reference).  Same chunking;
//   K operand [2][D/16][64 lanes][8 halves]: lane l holds key 32t + l%32,
//     channels 16kc + 8(l/32) + [0,8) -- A operand of the 32x32x16 f16 MFMA;
//   V operand [D/32][4 chunks][64 lanes][8 halves]: lane l holds channel
//     32dt + l%32 and, at slot e of key chunk c = 2t + jp, the key
//     32t + 8(2jp + e/4) + 4(l/32) + e%4.
__global__ void __launch_bounds__(256) k_prep_kv_fp16(const half_t* __restrict__ k, const half_t* __restrict__ v,
                                                      const int* __restrict__ cu, uint8_t* __restrict__ ws, int S,
                                                      int NB, int heads_kv, int D) {
  const int J = blockIdx.x, hk = blockIdx.y, b = blockIdx.z;
  const int t0 = seq_start(cu, b, S);
  const int L = seq_len(cu, b, S);
  if (64 * J >= L) return;
  const ChunkLayout lay = chunk_layout_fp16(D);
  uint8_t* chunk = ws + ((size_t)(b * heads_kv + hk) * NB + J) * lay.bytes;
  const int lane = threadIdx.x & 63, h = lane >> 5;
  // K: items (t, kc, lane)
  const int nk = 2 * (D / 16) * 64;
  for (int it = threadIdx.x; it < nk; it += blockDim.x) {
    const int ln = it & 63, kc = (it >> 6) % (D / 16), t = (it >> 6) / (D / 16);
    const int pos = 64 * J + 32 * t + (ln & 31);
    uint4 val = make_uint4(0, 0, 0, 0);
    if (pos < L)
      val = *reinterpret_cast<const uint4*>(k + ((size_t)(t0 + pos) * heads_kv + hk) * D + 16 * kc + 8 * (ln >> 5));
    reinterpret_cast<uint4*>(chunk + lay.k_op)[it] = val;
  }
  // V: items (dt, c, lane)
  const int nv = (D / 32) * 4 * 64;
  for (int it = threadIdx.x; it < nv; it += blockDim.x) {
    const int ln = it & 63, c = (it >> 6) & 3, dt = (it >> 8);
    const int hh = ln >> 5, d = 32 * dt + (ln & 31);
    const int t = c >> 1, jp = c & 1;
    h8_t val;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int pos = 64 * J + 32 * t + 8 * (2 * jp + (e >> 2)) + 4 * hh + (e & 3);
      val[e] = pos < L ? v[((size_t)(t0 + pos) * heads_kv + hk) * D + d] : (half_t)0.0f;
    }
    reinterpret_cast<h8_t*>(chunk + lay.v_op)[it] = val;
  }
  (void)h;
}

// ---------------------------------------------------------------------------
// Calibration reductions.  stats layout: [n][2][Hkv][D] uint32 holding the
// bits of non-negative floats (order-preserving): index 0 = max|K|, 1 = max|Q|
// (over the query heads of the group).  hist: 32768 uint64 bins of the fp16
// magnitude bit pattern of every K element.
__global__ void k_fill_u32(uint32_t* __restrict__ p, size_t n, uint32_t val) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = val;
}

// One pass over Q and K (bound by HBM: each is read once).  A workgroup takes
// a run of tokens; a thread holds one 16-byte piece of channels of one kv head
// (the same piece of each query head of its group for Q) and steps over the
// run with eight loads in flight, so a wave reads whole runs of 128 bytes or
// more.  Its maxima meet those of the workgroup in LDS and reach memory once
// per sequence of the run.  K's magnitudes also go into the workgroup's
// histogram in LDS (32-bit counters; the totals in memory have 64), flushed
// once: a flush costs an atomic per bin that occurs.  Odd workgroups take
// their Q tokens first, so that flushes run under other workgroups' loads.
// One kernel per statistic (2-byte loads, K read twice, a flush per 32768
// elements) took 890 us for 16 sequences of 4096 tokens with 32 + 8 heads,
// D=128.
constexpr int kCalibThreads = 1024;
constexpr int kCalibLoads = 8;
constexpr int kCalibBins = 32768;

struct CalibArgs {
  const half_t* q;
  const half_t* k;
  uint32_t* stats;
  unsigned long long* hist;
  int n, S, hkv, grp, D;
  int per_wg;                // tokens per workgroup
};

// Maximum bits of |x| over tokens [r0, r1) of x [.., hkv * grp, D] (grp heads
// per piece) into st[hkv * D], with COUNT every magnitude counted in bins.
// mx: LDS words of the pieces in hand, zero on entry and on return.
template <bool COUNT>
__device__ __forceinline__ void calib_run(const half_t* __restrict__ x, uint32_t* __restrict__ st, int r0, int r1,
                                          int hkv, int grp, int D, uint32_t* bins, uint32_t* mx) {
  const int pieces = hkv * D / 8;
  for (int p0 = 0; p0 < pieces; p0 += kCalibThreads) {
    // threads per token: the pieces, and as many tokens side by side as fit
    const int width = min(pieces - p0, kCalibThreads);
    const int par = kCalibThreads / width;
    const int sub = (int)threadIdx.x / width, slot = (int)threadIdx.x % width;
    if (sub < par) {
      const int c = (p0 + slot) * 8;
      const size_t row = (size_t)hkv * grp * D;
      const half_t* base = x + (size_t)(c / D) * grp * D + c % D;
      u16x2_t m[4] = {};
      for (int g = 0; g < grp; ++g, base += D) {
        for (int i0 = r0 + sub; i0 < r1; i0 += par * kCalibLoads) {
          uint4 in[kCalibLoads];
#pragma unroll
          for (int u = 0; u < kCalibLoads; ++u)        // past the end: the last token again (not counted below)
            in[u] = *reinterpret_cast<const uint4*>(base + (size_t)min(i0 + u * par, r1 - 1) * row);
#pragma unroll
          for (int u = 0; u < kCalibLoads; ++u) {
            const uint32_t w[4] = {in[u].x & 0x7FFF7FFFu, in[u].y & 0x7FFF7FFFu, in[u].z & 0x7FFF7FFFu,
                                   in[u].w & 0x7FFF7FFFu};
            const bool live = i0 + u * par < r1;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              m[e] = __builtin_elementwise_max(m[e], __builtin_bit_cast(u16x2_t, w[e]));
              if (COUNT && live) {
                atomicAdd(&bins[w[e] & 0xFFFFu], 1u);
                atomicAdd(&bins[w[e] >> 16], 1u);
              }
            }
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        atomicMax(&mx[slot + width * e],
                  __float_as_uint((float)__builtin_bit_cast(half_t, (unsigned short)m[e >> 1][e & 1])));
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 8 * width; i += kCalibThreads) {
      const uint32_t v = mx[i];
      mx[i] = 0;
      uint32_t* dst = &st[(size_t)(p0 + i % width) * 8 + i / width];
      if (v > *dst) atomicMax(dst, v);          // a stale value is only too small: no needed update is skipped
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kCalibThreads) k_calib(CalibArgs a) {
  extern __shared__ __align__(16) uint32_t lh[];           // the bins, then 8 words per piece in hand
  uint32_t* mx = lh + kCalibBins;
  const int hd = a.hkv * a.D;
  const int words = kCalibBins + min(hd, 8 * kCalibThreads);
  for (int i = threadIdx.x; i < words; i += kCalibThreads) lh[i] = 0;
  __syncthreads();
  const long t0 = (long)blockIdx.x * a.per_wg, t1 = min(t0 + a.per_wg, (long)a.n * a.S);
  for (int phase = 0; phase < 2; ++phase) {
    const bool is_q = (phase == 0) == ((blockIdx.x & 1) != 0);
    for (long t = t0; t < t1;) {                           // the run's part in each sequence
      const int n = (int)(t / a.S), r0 = (int)(t % a.S), r1 = (int)min((long)a.S, r0 + (t1 - t));
      if (is_q)
        calib_run<false>(a.q + (size_t)n * a.S * hd * a.grp, a.stats + ((size_t)n * 2 + 1) * hd, r0, r1, a.hkv, a.grp,
                         a.D, lh, mx);
      else
        calib_run<true>(a.k + (size_t)n * a.S * hd, a.stats + (size_t)n * 2 * hd, r0, r1, a.hkv, 1, a.D, lh, mx);
      t += r1 - r0;
    }
    if (!is_q) {                                           // calib_run ends with a barrier
      for (int i = threadIdx.x; i < kCalibBins; i += kCalibThreads) {
        const uint32_t c = lh[i];
        if (c) atomicAdd(&a.hist[i], (unsigned long long)c);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The gate of one layer, in float64: one workgroup reads the histogram (each
// thread a run of bins) and the channel maxima, and leaves rho, T, the branch
// and alpha in place of the first bins.  The formulas are evaluated step by
// step (no contraction into fused multiply-adds).
//
// On the GPU and not on the host, where the same sums need a copy of 390 KB
// through pageable memory, three passes over the bins and two pow() per
// channel: 16 x 4096 tokens of 32 + 8 heads, D = 128, take 193 us a call against
// 273, of which the pass over Q and K is 145 us.
constexpr int kGateThreads = 1024;

__global__ void __launch_bounds__(kGateThreads) k_calib_gate(const uint32_t* __restrict__ stats,
                                                             unsigned long long* hist, int n, int hd, float alpha) {
#pragma clang fp contract(off)
  constexpr int kPer = kCalibBins / kGateThreads, kWaves = kGateThreads / 64;
  __shared__ unsigned long long wave_sum[kWaves];
  __shared__ float wave_max[2][kWaves];
  __shared__ double stat_at[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  unsigned long long c[kPer], own = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) c[i] = hist[kPer * tid + i];
  // largest statistic of K and of Q (a NaN never replaces a maximum)
  float mk = 0.0f, mq = 0.0f;
  for (int i = tid; i < hd; i += kGateThreads) {
#pragma unroll 8
    for (int r = 0; r < n; ++r) {
      const float k = __uint_as_float(stats[(size_t)(2 * r) * hd + i]);
      const float q = __uint_as_float(stats[(size_t)(2 * r + 1) * hd + i]);
      mk = mk < k ? k : mk;
      mq = mq < q ? q : mq;
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float k = __shfl_xor(mk, o), q = __shfl_xor(mq, o);
    mk = mk < k ? k : mk;
    mq = mq < q ? q : mq;
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) own += c[i];
  unsigned long long incl = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wave_sum[wave] = incl;
  if (lane == 0) {
    wave_max[0][wave] = mk;
    wave_max[1][wave] = mq;
  }
  if (tid < 2) stat_at[tid] = 0.0;
  __syncthreads();
  unsigned long long before = incl - own, total = 0;
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) before += wave_sum[w];
    total += wave_sum[w];
    mk = mk < wave_max[0][w] ? wave_max[0][w] : mk;
    mq = mq < wave_max[1][w] ? wave_max[1][w] : mq;
  }
  // P99 of |K|: linear interpolation between two order statistics
  const double pos = total > 0 ? 0.99 * (double)(total - 1) : 0.0;
  const unsigned long long lo = (unsigned long long)floor(pos);
  const unsigned long long hi = total > 0 && lo + 1 > total - 1 ? total - 1 : lo + 1;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const unsigned long long k = j == 0 ? lo : hi;
    if (k < before || k >= before + own) continue;        // the bin that holds it is another thread's
    unsigned long long at = before;
    bool found = false;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      at += c[i];
      if (!found && at > k) {
        stat_at[j] = (double)(float)__builtin_bit_cast(half_t, (uint16_t)(kPer * tid + i));
        found = true;
      }
    }
  }
  __syncthreads();
  if (tid != 0) return;
  double p99 = 0.0;
  if (total > 0) {
    const double t = pos - (double)lo, a = stat_at[0], b = stat_at[1], diff = b - a;
    p99 = t >= 0.5 ? b - diff * (1.0 - t) : a + diff * t;
  }
  CalibGate g;
  g.rho = p99 > 0 ? (double)mk / p99 : __builtin_inf();
  g.t_kq = mq > 0 ? (double)mk / (double)mq : __builtin_inf();
  if (alpha < 0) {
    g.branch = g.rho >= 6.0 && g.t_kq > 3.0 ? 2 : g.rho >= 6.0 && g.t_kq >= 2.0 && g.t_kq <= 3.0 ? 1 : 0;
    g.alpha = g.branch == 2 ? 0.5 : g.branch == 1 ? 0.25 : 0.0;
  } else {
    g.branch = alpha == 0 ? 0 : alpha >= 0.5f ? 2 : 1;
    g.alpha = alpha;
  }
  *reinterpret_cast<CalibGate*>(hist) = g;                // every thread holds its bins by now
}

// s of each channel: the RMS over the sequences of the per-sequence maxima,
// s = Kbar^alpha / Qbar^(1-alpha), rounded once to fp32.
__global__ void __launch_bounds__(64) k_calib_scales(const uint32_t* __restrict__ stats,
                                                     const CalibGate* __restrict__ gate, int n, int hd,
                                                     float* __restrict__ s_out) {
#pragma clang fp contract(off)
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= hd) return;
  const double alpha = gate->alpha;
  float s32 = 1.0f;
  if (alpha != 0.0) {
    double sk = 0.0, sq = 0.0;
#pragma unroll 4
    for (int r = 0; r < n; ++r) {
      const double kv = (double)__uint_as_float(stats[(size_t)(2 * r) * hd + i]);
      const double qv = (double)__uint_as_float(stats[(size_t)(2 * r + 1) * hd + i]);
      sk += kv * kv;
      sq += qv * qv;
    }
    const double kbar = sqrt(sk / n), qbar = sqrt(sq / n);
    const double s = pow(kbar, alpha) / pow(qbar, 1.0 - alpha);
    const bool bad = kbar == 0 || qbar == 0 || !__builtin_isfinite(s) || s == 0;
    s32 = bad ? 1.0f : (float)s;
  }
  s_out[i] = s32;
}

// ---------------------------------------------------------------------------
// Pairs of inputs go through the packed routine the attention kernels use.
__global__ void k_selftest_exp2(const half_t* __restrict__ x, half_t* __restrict__ y, long n) {
  const long i = 2 * ((long)blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= n) return;
  h2_t v = {x[i], i + 1 < n ? x[i + 1] : (half_t)0.0f};
  const h2_t r = exp2_h2(v);
  y[i] = r[0];
  if (i + 1 < n) y[i + 1] = r[1];
}

// ---------------------------------------------------------------------------
// Host launchers.
hipError_t launch_quant_rows(const half_t* x, const float* s, uint8_t* codes, uint32_t* meta, long n_rows,
                             int heads, int heads_kv, int D, bool is_k, hipStream_t st) {
  const long per_row = (long)heads * D / 8;               // pieces of 8 channels
  const long n = n_rows * per_row;
  if (n == 0) return hipSuccess;
  // six waves per SIMD on 256 compute units, rounded up to a whole number of
  // rows (four, eight or sixteen waves are 1 to 2% slower)
  constexpr long kThreads = 256L * 1536;
  const long stride = std::min(n, (kThreads + per_row - 1) / per_row * per_row);
  const dim3 grid((unsigned)((stride + 255) / 256));
  if (is_k)
    k_quant_rows<true><<<grid, dim3(256), 0, st>>>(x, s, codes, meta, n, stride, heads, heads_kv, D);
  else
    k_quant_rows<false><<<grid, dim3(256), 0, st>>>(x, s, codes, meta, n, stride, heads, heads_kv, D);
  return hipGetLastError();
}

hipError_t launch_quant_v(const half_t* v, const int* cu, uint8_t* codes, uint32_t* meta, int batch, int S, int NB,
                          int heads_kv, int D, hipStream_t st) {
  const long n_items = (long)batch * NB * heads_kv * D / 4;
  if (n_items == 0) return hipSuccess;
  const long blocks = (n_items + 127) / 128;
  k_quant_v_canon<<<dim3((unsigned)blocks), dim3(256), 0, st>>>(v, cu, codes, meta, batch, S, NB, heads_kv * D);
  return hipGetLastError();
}

hipError_t launch_prep_kv(const half_t* k, const half_t* v, const float* s, const int* cu, uint8_t* ws, int batch,
                          int S, int NB, int heads_kv, int D, bool fp16, bool qmean, hipStream_t st) {
  dim3 grid(NB, heads_kv, batch);
  if (fp16)
    k_prep_kv_fp16<<<grid, dim3(256), 0, st>>>(k, v, cu, ws, S, NB, heads_kv, D);
  else
    k_prep_kv_hif4<<<dim3(NB, heads_kv, 2 * batch), dim3(64 * 2 * (D / 64)), 64 * D * sizeof(half_t), st>>>(
        k, v, s, cu, ws, S, NB, heads_kv, D / 64, qmean);
  return hipGetLastError();
}

hipError_t launch_calib(const half_t* q, const half_t* k, int n, int S, int hq, int hkv, int D, float alpha,
                        uint32_t* stats, unsigned long long* hist, float* s_out, hipStream_t st) {
  // stats and hist are adjacent in the workspace (hist follows, rounded up to
  // 256 bytes): one fill clears both
  const size_t words = (size_t)(reinterpret_cast<uint32_t*>(hist) - stats) + 2 * 32768;
  k_fill_u32<<<dim3((unsigned)std::min<size_t>(256, (words + 255) / 256)), dim3(256), 0, st>>>(stats, words, 0u);
  // a workgroup per compute unit: the histogram takes most of its LDS
  const long tokens = (long)n * S;
  const CalibArgs a{q, k, stats, hist, n, S, hkv, hq / hkv, D, (int)((tokens + 255) / 256)};
  const size_t lds = (kCalibBins + std::min(hkv * D, 8 * kCalibThreads)) * sizeof(uint32_t);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_calib),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  k_calib<<<dim3((unsigned)((tokens + a.per_wg - 1) / a.per_wg)), dim3(kCalibThreads), lds, st>>>(a);
  k_calib_gate<<<dim3(1), dim3(kGateThreads), 0, st>>>(stats, hist, n, hkv * D, alpha);
  k_calib_scales<<<dim3((unsigned)((hkv * D + 63) / 64)), dim3(64), 0, st>>>(
      stats, reinterpret_cast<const CalibGate*>(hist), n, hkv * D, s_out);
  return hipGetLastError();
}

hipError_t launch_selftest_exp2(const half_t* x, half_t* y, long n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  k_selftest_exp2<<<dim3((unsigned)((n + 511) / 512)), dim3(256), 0, st>>>(x, y, n);
  return hipGetLastError();
}

}  // namespace hifa4
