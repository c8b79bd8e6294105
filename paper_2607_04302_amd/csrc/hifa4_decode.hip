// HiFA4 decode step on a packed HIF4 K/V cache (gfx950).
//
// Paper: Algorithm 1 for one query row per sequence (the newest token, which
// sees every cached key) with Section 4.5's P-Reordering; the cache holds K^
// and V^ in the packed 4.5-bit HIF4 format of the Background's HIF4
// paragraph.  The paper leaves decode and the KV-cache footprint open.
//
// The cache is the canonical layout (hifa4_quantize_qk, hifa4_quantize_v):
// per group 32 bytes of sign-magnitude nibbles and one metadata word.  One
// decode row has too little work per sequence for one workgroup, so the key
// range is split into runs of 64-key blocks; the split must not change any P^
// code, because P^ depends on the running maximum entering each block.  Two
// kernels keep every decision of the sequential loop:
//   1. runs: each wave takes a run of blocks of one kv head.  It smooths and
//      quantizes the query rows of the GQA group (Q^ = HIF4(fp16(q s))),
//      computes the fp16 scores S2 of its blocks into LDS, publishes each
//      row's maximum over the run, takes the running maximum the sequential
//      loop has at its first block from the maxima the earlier runs published,
//      then applies the FP16 softmax, P^ = HIF4(P) and the PV product as the
//      sequential loop does; it writes its partial O_s and l_s, both relative
//      to the running maximum at its last block;
//   2. merge: O = sum_s O_s R_s and l = sum_s l_s R_s, where R_s is the product
//      of the rescale factors r_J = E(fp16(m_{J-1} - m_J)) of all blocks after
//      run s: the sequential recurrence O <- r_J O + P^_J V^_J unrolled.
//
// Both contractions run on the block-scaled 16x16x128 MFMA with the cache
// codes as FP4 (E2M1) operands and no per-element conversion.  A code's
// magnitude u is (u & 3) + (u & 4), and both parts are E2M1 codes of value
// (u & 3)/2 and (u & 4)/2 with the cache's own sign bit, so masking a word of
// eight nibbles gives two operand registers.  Of an element's scale
// 2^-(E2+E3), E2 (one per word) is the lane's E8M0 operand scale, and
// 2^-E3 = (1 + [E3 = 0])/2 is a second pair of registers with the E3 = 1
// half-words cleared.  So one word fills the 32 K slots of its lane:
// {u&3, u&4, (u&3)[E3=0], (u&4)[E3=0]}, against the same eight query (or P^)
// elements four times, in FP6 (E2M3, which holds every u 2^-sh).  A group of
// 64 elements is two words in each of four lanes, two MFMAs.  Every product is
// a multiple of 2^-4 and every sum stays below 2^13, so each 64-element dot is
// exact in fp32; the bases (E6M2, three significant bits) are applied in an
// fp32 epilogue where every product stays exact.  The scores therefore follow
// the library's score contract bit for bit, and the PV partial sums of a block
// are exact before the fp32 rescale-and-add.
//
// What bounds it: one step of 8 sequences of 32768 tokens (Hq 32, Hkv 8, D 128)
// reads 302 MB, 59 us at the 5.1 TB/s that large reads reach on this card, and
// takes 77 us where several such caches take turns (72 us over one, part of
// which the 256 MB cache beside the memory holds); 32 sequences of 300 to 8192
// tokens take 50 us, one of 4096 tokens 15 us (12.4 into outputs that the caller brings).  The VALU is
// busy half of the time and the cache streams at 4.3 TB/s beside it.  With the
// codes turned into int8 operands (9400 VALU instructions a wave for 8 blocks,
// 512 of them quarter-rate multiplies, against 4750 here) the three took 89,
// 82.5 and 20.6 us.
//
// MFMA operand convention: lane l holds row / column n = l & 15 of A / B and
// the K slots 32q..32q+31, q = l >> 4; output value i of lane l is row 4q + i,
// column n.  Query row r of the GQA group sits in A row 4(r & 3) + (r >> 2),
// so the output rows of a lane are r = q (and q + 4 for groups of more than
// four heads): the same lanes that hold row r in the softmax, sixteen lanes of
// four keys each, and the row's factors need no exchange.
//
// Workgroups hold one wave per kv head (up to eight): the heads of a token
// share cache lines, so the lines are read once by one compute unit.
#include <atomic>
#include <random>

#include "hifa4_device.h"
#include "hifa4_decode.h"
#include "hifa4_internal.h"
#include "hifa4_packed.h"

namespace hifa4 {

namespace {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
typedef short s16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int dseq_start(const int* cu, int b, int S) { return cu ? cu[b] : b * S; }
// a length above max_seqlen is outside the contract; clamping it keeps every
// access inside the caller's buffers
__device__ __forceinline__ int dseq_len(const int* cu, int b, int S) { return cu ? min(cu[b + 1] - cu[b], S) : S; }

// The value of another lane of the same sixteen (CTRL: a DPP control word).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int kDppNext = 0xF9;           // quad_perm [1, 2, 3, 3]

template <int CTRL>
__device__ __forceinline__ h2_t max_dpp(h2_t v) {
  return hmax2(v, __builtin_bit_cast(h2_t, dpp<CTRL>(__builtin_bit_cast(uint32_t, v))));
}
// Maximum over the sixteen lanes of a row, per half.
__device__ __forceinline__ h2_t max_row16(h2_t v) {
  v = max_dpp<kDppXor1>(v);
  v = max_dpp<kDppXor2>(v);
  v = max_dpp<kDppHalfMirror>(v);
  return max_dpp<kDppMirror>(v);
}

// Where the runs leave their results.
struct RunStore {
  float* opart;            // [Hq, stride, D]
  float4* spart;           // [Hq, stride]: l, product of the run's
                           // rescale factors, running max after its last block
  uint64_t* runmax;        // [Hq, stride] run maxima, epoch-tagged; the merge
                           // kernel clears each row's words after the runs
  int stride;              // runs of a query head
};

struct DecodeArgs {
  const half_t* q;         // raw decode queries [batch, Hq, D] fp16
  const float* s;          // smoothing scales [Hkv, D] or null
  const uint8_t* kc;       // canonical K^ cache [tokens, Hkv, G, 32]
  const uint32_t* km;      // [tokens, Hkv, G]
  const uint8_t* vc;       // canonical V^ cache [batch, NB, Hkv, D, 32]
  const uint32_t* vm;      // [batch, NB, Hkv, D]
  const int* cu;
  RunStore usual, grown;   // in the workspace; `grown`: of runs that outgrew the grid
  int* runbase;            // packed runs: [batch] first run of each sequence (`usual`)
  half_t* o;               // [batch, Hq, D]
  float* lse;              // [Hq, batch]
  uint8_t* dbg_codes;      // [Hq, batch, NB, 32] or null
  uint32_t* dbg_meta;      // [Hq, batch, NB]
  int batch, S, NB, hq, hkv, D, waves;
  int bps;                 // blocks per run
  int n_split;             // ceil(NB / bps)
  int packed;              // runs are numbered over the sequences' own lengths
  int tokens;              // cached tokens that the grid of packed runs covers
  float c;
  uint32_t epoch;          // this call's tag (never 0)
  int spin_limit;          // polls before a look-back gives up
  int rescore;             // 0: a row whose look-back gave up comes out NaN (testing)
  int publish;             // 0: no run maxima are published (testing the give-up)
};

// One wave's share: kv head hk of sequence b, blocks [J0, J0 + nb), run `part`
// of the sequence, run `run` of the call.
struct WaveSpan {
  int hk, b, L, J0, nb, t0, grp, part, run;
};

// Bounds of the sequences 64 k + lane of a packed call (empty past the batch).
constexpr int kScanSteps = kMaxPackedBatch / 64;
struct Bounds {
  int first[kScanSteps], end[kScanSteps];
};
__device__ __forceinline__ Bounds load_bounds(const DecodeArgs& a, int lane) {
  Bounds s;
#pragma unroll
  for (int k = 0; k < kScanSteps; ++k) {
    const int b = 64 * k + lane;
    s.first[k] = s.end[k] = 0;
    if (64 * k < a.batch && b < a.batch) {
      s.first[k] = a.cu[b];
      s.end[k] = a.cu[b + 1];
    }
  }
  return s;
}
__device__ __forceinline__ int runs_of(int len, int bps) {
  return len > 0 ? (((len + 63) >> 6) + bps - 1) / bps : 0;
}
// Runs of the sequences before b.
__device__ __forceinline__ int runs_before(const DecodeArgs& a, const Bounds& s, int lane, int b, int bps) {
  int n = 0;
#pragma unroll
  for (int k = 0; k < kScanSteps; ++k)
    n += 64 * k + lane < b ? runs_of(min(s.end[k] - s.first[k], a.S), bps) : 0;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) n += __shfl_xor(n, o);
  return __builtin_amdgcn_readfirstlane(n);
}
// Blocks per run of a call whose lengths have grown: the fewest from the plan's
// on with which all runs fit the workspace (those of kMaxRun blocks always do).
__device__ __forceinline__ int grown_run_length(const DecodeArgs& a, const Bounds& s, int lane) {
  int bps = a.bps;
  while (bps < kMaxRun && runs_before(a, s, lane, a.batch, bps) > a.grown.stride) ++bps;
  return bps;
}

enum Span { kRun, kIdle, kGrown };

// Sequence and part of run `run`; kIdle when the wave has nothing to do in it.
// Packed: the runs are numbered densely over the sequences' own lengths, so
// the grid holds (nearly) no idle workgroup and the run length can be chosen
// from the number of cached tokens and not from the longest sequence; every
// wave finds its sequence by a prefix sum over the batch (one load latency and
// a scan over 64 lanes).
//
// The grid is that of total_tokens cached tokens, and a captured launch may be
// replayed over lengths that have grown past it since.  That gives kGrown; with
// GROWN the run length is settled anew, for a loop in which a workgroup takes
// several runs.  (Settled in every call it took 0.3 to 0.8 us of 18 to 44.)
template <bool GROWN>
__device__ __forceinline__ Span wave_span(const DecodeArgs& a, int run, int tid, WaveSpan& w) {
  w.hk = __builtin_amdgcn_readfirstlane((int)blockIdx.y * a.waves + (tid >> 6));
  if (w.hk >= a.hkv) return kIdle;
  w.grp = a.hq / a.hkv;
  w.run = run;
  int bps = a.bps;
  if (!a.packed) {
    w.b = w.run / a.n_split;
    w.part = w.run - w.b * a.n_split;
    w.L = dseq_len(a.cu, w.b, a.S);
    w.t0 = dseq_start(a.cu, w.b, a.S);
  } else {
    const int lane = tid & 63;
    const Bounds s = load_bounds(a, lane);
    if (GROWN) {
      bps = grown_run_length(a, s, lane);
    } else {
#pragma unroll
      for (int k = 0; k < kScanSteps; ++k)
        if ((a.batch - 1) / 64 == k &&
            __builtin_expect(__builtin_amdgcn_readlane(s.end[k], (a.batch - 1) & 63) > a.tokens, 0))
          return kGrown;
    }
    int before = 0;                      // runs of the sequences of earlier steps
    bool found = false;
#pragma unroll
    for (int k = 0; k < kScanSteps; ++k) {
      if (found || 64 * k >= a.batch) break;
      const int len = min(s.end[k] - s.first[k], a.S);
      const int nr = runs_of(len, bps);
      int incl = nr;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      const uint64_t over = __ballot(before + incl > w.run);
      if (over != 0) {
        const int j = __builtin_ctzll(over);
        w.b = 64 * k + j;
        w.part = w.run - (before + __builtin_amdgcn_readlane(incl - nr, j));
        w.t0 = __builtin_amdgcn_readlane(s.first[k], j);
        w.L = __builtin_amdgcn_readlane(len, j);
        found = true;
      } else {
        before += __builtin_amdgcn_readlane(incl, 63);
      }
    }
    if (!found) return kIdle;
    if (!GROWN && w.part == 0 && w.hk == 0 && lane == 0) a.runbase[w.b] = w.run;
  }
  const int nblk = (w.L + 63) >> 6;
  w.J0 = w.part * bps;
  if (w.J0 >= nblk) return kIdle;
  w.nb = min(bps, nblk - w.J0);
  return kRun;
}

// One block's codes and metadata of one kv head in LDS, as the loads lay them
// down: codes [64 rows][G groups][32 B] (V^: [64 G channels][32 B]), then the
// metadata words in the same order.  Row 16t + n of K^ is key 4n + t of the
// block, so that the four output columns n of tiles 0..3 are the four keys of
// one E3 block of P and the scores need no exchange on their way to the
// softmax.
template <int G>
struct Stage {
  static constexpr int kCodes = 2048 * G, kBytes = kCodes + 256 * G;
  static constexpr int kLoads = 3 * G;               // of a block: 2G of 1 KiB, G of 256 B
};

// Asynchronous copies of 64 lanes x 16 or 4 bytes straight into LDS: lane i
// reads at base + off and its bytes land at m0 + 16 i (4 i).  Written out with
// a scalar base; completion is counted in vmcnt, in issue order.  Nothing else
// in this file may use M0 (tests/test_m0_guard_decode.py).
__device__ __forceinline__ void dma16(const uint8_t* base, uint32_t off, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(m0) : "memory", "m0");
}
__device__ __forceinline__ void dma4(const uint8_t* base, uint32_t off, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1" : : "v"(off), "s"(base), "s"(m0) : "memory", "m0");
}
// At most N vector-memory operations of the wave outstanding; and every LDS
// read of the wave done (before its buffer is filled again).
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

// The two FP6 A operands of a lane's sixteen elements (96 bits d): each word's
// eight elements, 48 bits, fill the 32 slots four times, so three registers
// repeat.
struct AOperand {
  uint32_t r[2][3];
};
__device__ __forceinline__ AOperand a_operand(u4_t d) {
  AOperand a;
  a.r[0][0] = d.x;
  a.r[0][1] = (d.y & 0xFFFFu) | (d.x << 16);
  a.r[0][2] = __builtin_amdgcn_alignbit(d.y, d.x, 16);
  const uint32_t e = __builtin_amdgcn_alignbit(d.z, d.y, 16);
  a.r[1][0] = e;
  a.r[1][1] = (d.z >> 16) | (e << 16);
  a.r[1][2] = (e >> 16) | (d.z & 0xFFFF0000u);
  return a;
}
template <int WORD>
__device__ __forceinline__ f4_t mfma_word(const uint32_t (&ar)[3], uint32_t w, uint32_t e3, uint32_t scale, f4_t c) {
  const i8_t a = {(int)ar[0], (int)ar[1], (int)ar[2], (int)ar[0], (int)ar[1], (int)ar[2], 0, 0};
  const uint32_t lo = w & 0xBBBBBBBBu, hi = w & 0xCCCCCCCCu;
  const i8_t b = {(int)lo, (int)hi, (int)(lo & ~e3), (int)(hi & ~e3), 0, 0, 0, 0};
  // A: E2M3 codes of 4 u 2^-sh / 8, scaled by 2 = u 2^-sh; B: E2M1
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 2, 4, 0, 128, WORD, (int)scale);
}

// Lane constants of a group's metadata: shifts that bring the E3 bits of the
// lane's half-words (bits 16 + 4q.. of the metadata word) to the tops of two
// 16-bit halves, and of its E2 pair (bits 8 + 2q, 9 + 2q) to the bottom.
struct MetaShifts {
  u16x2_t e3[2];
  uint32_t e2;
};
__device__ __forceinline__ MetaShifts meta_shifts(int q) {
  const unsigned short s = (unsigned short)(15 - 4 * q);
  return MetaShifts{{u16x2_t{s, (unsigned short)(s - 1)}, u16x2_t{(unsigned short)(s - 2), (unsigned short)(s - 3)}},
                    (uint32_t)(8 + 2 * q)};
}
// 0xFFFF in each half-word with E3 = 1 (k: the shifts of its word).
__device__ __forceinline__ uint32_t e3_mask(uint32_t meta, u16x2_t k) {
  const uint16_t x = (uint16_t)(meta >> 16);
  const s16x2_t m = __builtin_bit_cast(s16x2_t, u16x2_t{x, x} << k) >> s16x2_t{15, 15};
  return __builtin_bit_cast(uint32_t, m);
}

// Exact dot products sum(u_a 2^-sh_a * u_b 2^-sh_b) of a whole 64-element group
// (b the lane's two words of it and the group's metadata): value i of lane l
// is row 4q + i with column n.
__device__ __forceinline__ f4_t group_dot(const AOperand& a, u2_t w, uint32_t meta, const MetaShifts& k) {
  const uint32_t e2 = __umul24((meta >> k.e2) & 3u, 0x81u);          // E2 of word 0 in bit 0, of word 1 in bit 8
  const uint32_t scale = 0x7E7Eu | (~e2 & 0x0101u);                  // 2^-E2 as E8M0 bytes
  const f4_t z = {};
  const f4_t c = mfma_word<0>(a.r[0], w.x, e3_mask(meta, k.e3[0]), scale, z);
  return mfma_word<1>(a.r[1], w.y, e3_mask(meta, k.e3[1]), scale, c);
}

// E6M2 value of a metadata word's base, (byte 0 << 21) + offset as fp32 bits
// (offset 0x30000000, held in a scalar register so that shift and add are one
// instruction).  Plain code on purpose: a statement of inline assembly beside
// the MFMAs may be given a register of an MFMA's unused result values, and the
// compiler does not wait for the MFMA before such a write.
__device__ __forceinline__ float meta_base(uint32_t meta, uint32_t offset) {
  return __uint_as_float(((meta & 255u) << 21) + offset);
}

// E2M3 codes of four elements u 2^-sh, as 24 bits in element order: the code
// of v = u << (2 - sh) eighths (half of the element; the operand scale doubles
// it) is v below 16 and 8 + v/2 above.  u and sh from the quantizer; neg is a
// 32-bit word with bit 5 of each of the four 6-bit fields.
__device__ __forceinline__ uint32_t e2m3_pack(const uint32_t (&v)[4]) {
  uint32_t c[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) c[j] = min(v[j], 8u + (v[j] >> 1));
  return c[0] | (c[1] << 6) | (c[2] << 12) | (c[3] << 18);
}
// The 24-bit fields of a quad of lanes as three consecutive words (the fourth
// lane's word is padding): lane j of the quad returns word j.
__device__ __forceinline__ uint32_t quad_words(uint32_t f, int lane) {
  const int j = lane & 3;
  return (f >> (8 * j)) | (dpp<kDppNext>(f) << (24 - 8 * j));
}

// LDS of one wave: two blocks in flight, and the A operands of Q^ (before the
// loop) and of P^ as [row][group][16 words] of which each quarter's first
// three are used.
template <int G, int RP>
struct WaveLds {
  alignas(16) uint8_t buf[2][Stage<G>::kBytes];
  alignas(16) uint32_t a[4 * RP * G * 16];
};

// The running maximum entering run w.part of a softmax row: the maximum of the
// earlier runs' epoch-tagged maxima of the sequence (f: the row's word of the
// sequence's first run), 16 lanes per row, kLookBatch words each per round,
// every load of a round in flight before the first is checked.  A limit on the
// polls of a look-back (some milliseconds) ends every wait; one that gives up
// sets `lost`, and the wave takes the missing maximum from the scores itself.
constexpr int kLookBatch = 4;                    // run maxima per lane per round
constexpr int kSpinLimit = 4096;

__device__ __forceinline__ float look_back(const DecodeArgs& a, const uint64_t* f, int part, int kq, bool& lost) {
  float mm = -__builtin_inff();
  int polls = a.spin_limit;
  lost = false;
  for (int q0 = 0; q0 < part; q0 += 16 * kLookBatch) {
    uint64_t wd[kLookBatch];
#pragma unroll
    for (int k = 0; k < kLookBatch; ++k) {
      const int q = q0 + 16 * k + kq;
      wd[k] = q < part ? __hip_atomic_load(f + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    }
#pragma unroll
    for (int k = 0; k < kLookBatch; ++k) {
      const int q = q0 + 16 * k + kq;
      if (q < part) {
        uint64_t v = wd[k];
        for (; (uint32_t)(v >> 32) != a.epoch && polls > 0; --polls) {
          __builtin_amdgcn_s_sleep(2);
          v = __hip_atomic_load(f + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if ((uint32_t)(v >> 32) == a.epoch) mm = fmaxf(mm, (float)__builtin_bit_cast(half_t, (uint16_t)v));
        else lost = true;
      }
    }
  }
  return mm;
}

// ---------------------------------------------------------------------------
// 1. Runs.  Wave = kv head, workgroup = (run, kv heads).  A wave never meets a
// barrier.  The earlier runs of a sequence belong to workgroups with lower
// indices, which each XCD dispatches first, so in a call that has the GPU to
// itself the lowest unfinished workgroup is always running and the waits are
// short.  No result depends on that: two calls on two streams can hold each
// other's lower workgroups off the GPU with workgroups that wait.  A wait that
// runs to its limit ends in the wave scoring the earlier blocks itself.
//
// The run's block loads (K of each block, then V of each block) form one
// stream through two LDS buffers of the wave, filled by asynchronous copies
// two blocks ahead of the arithmetic, so the first V^ blocks are in flight
// while the last scores are computed and the run maxima are awaited.  In the
// MFMA layout consecutive lanes hold consecutive rows, 8 bytes each of 32-byte
// groups; loaded straight into registers that way, the cache stream was bound
// by the number of separate L1 accesses (970 per block of 9.2 KB, 31.8 M
// in a call of 8 x 32768 tokens, on top of which the requests stalled) and the
// call took 102 us.  The copies read whole 64-byte rows of K^ and whole
// kilobytes of V^, and LDS serves the layout.
//
// Scores: A = the GQA group's query rows, B = 16 keys.  Epilogue per group:
// d_g = dot * b_K (exact), the group's exact term t_g = d_g * b_Q,g/16, the
// terms summed in order in fp32 (a fused multiply-add of the exact product
// rounds exactly the sum), S2 = fp16(fp32(sum * c)).
//
// Softmax of a block: lane i takes query row 4p + (i >> 4) (pass p < RP) and
// its keys 4(i & 15)..+3, one E3 block; E2 pairs two lanes, the row base is
// that of E(rowmax - m), which equals the largest P because E is monotone.
// l is summed per lane and over the row's lanes at the end of the run.
// PV: B = 16 channels of the block's V^ groups;
// O[row][ch] = fma(O, r_row, dot * b_V * b_P/16).
template <int G, int RP, int NORM, bool DEBUG, bool GROWN>
__device__ __forceinline__ Span decode_run(const DecodeArgs& a, WaveLds<G, RP>* lds, int run, int tid) {
  WaveSpan w;
  if (const Span sp = wave_span<GROWN>(a, run, tid, w); sp != kRun) return sp;
  constexpr int D = 64 * G, NT = 4 * G;
  const RunStore& rs = GROWN ? a.grown : a.usual;
  WaveLds<G, RP>& sl = lds[__builtin_amdgcn_readfirstlane(tid >> 6)];
  const int lane = tid & 63, n = lane & 15, q = lane >> 4, kq = n;
  const int hk = w.hk, nb = w.nb, grp = w.grp;
  const int h0 = hk * grp;                        // first query head of the group
  const size_t row0 = (size_t)w.b * a.hq + h0;
  int prow[RP];                                   // row of this lane per pass (idle lanes repeat row 0)
#pragma unroll
  for (int p = 0; p < RP; ++p) prow[p] = 4 * p + q < grp ? 4 * p + q : 0;

  // Query loads first, then the two first blocks.
  uint2 qraw[RP][G];
  float4 qs[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int ch = 64 * g + 4 * kq;
#pragma unroll
    for (int p = 0; p < RP; ++p) qraw[p][g] = *reinterpret_cast<const uint2*>(a.q + (row0 + prow[p]) * D + ch);
    qs[g] = a.s ? *reinterpret_cast<const float4*>(a.s + (size_t)hk * D + ch) : make_float4(1.0f, 1.0f, 1.0f, 1.0f);
  }

  // K^ copies: lane l of the i-th kilobyte fetches piece l % 2G of row
  // 64i/2G + l/2G, token 4 (row % 16) + row / 16 of the block; tokens past the
  // sequence's end repeat its last one (their scores are masked).
  const uint32_t krow = (uint32_t)a.hkv * (G * 32);             // bytes between tokens
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&sl.buf[0][0];
  const int crow = lane / (2 * G), mrow = lane / G;             // rows of load 0 (codes, metadata)
  const uint32_t coff = (uint32_t)(4 * (crow & 15) + (crow >> 4)) * krow, cpiece = 16 * (lane % (2 * G));
  const uint32_t moff = (uint32_t)(4 * (mrow & 15) + (mrow >> 4)) * (krow >> 3), mpiece = 4 * (lane % G);
  auto load_k = [&](int J, int slot) {
    const size_t g0 = ((size_t)(w.t0 + 64 * J) * a.hkv + hk) * G;
    const uint8_t* cb = a.kc + g0 * 32;
    const uint8_t* mb = reinterpret_cast<const uint8_t*>(a.km + g0);
    const uint32_t last = last_key_offset(w.L - 64 * J, krow);
    const uint32_t dst = lds0 + slot * Stage<G>::kBytes;
#pragma unroll
    for (int i = 0; i < 2 * G; ++i) {
      const uint32_t step = G == 4 ? 32 * (i & 1) + (i >> 1) : G == 2 ? i : 2 * i;      // tokens from load 0
      dma16(cb, min(coff + step * krow, last) + cpiece, dst + 1024 * i);
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const uint32_t step = G == 4 ? i : 2 * i;
      dma4(mb, min(moff + step * (krow >> 3), last >> 3) + mpiece, dst + Stage<G>::kCodes + 256 * i);
    }
  };
  auto load_v = [&](int J, int slot) {
    const size_t vg = (((size_t)w.b * a.NB + J) * a.hkv + hk) * D;
    const uint8_t* cb = a.vc + vg * 32;
    const uint8_t* mb = reinterpret_cast<const uint8_t*>(a.vm + vg);
    const uint32_t dst = lds0 + slot * Stage<G>::kBytes;
#pragma unroll
    for (int i = 0; i < 2 * G; ++i) dma16(cb + 1024 * i, 16 * lane, dst + 1024 * i);
#pragma unroll
    for (int i = 0; i < G; ++i) dma4(mb + 256 * i, 4 * lane, dst + Stage<G>::kCodes + 256 * i);
  };
  // item j of the stream: K of block j, then V of block j - nb; buffer j & 1
  auto fetch = [&](int j) {
    if (j < nb) load_k(w.J0 + j, j & 1);
    else load_v(w.J0 + j - nb, j & 1);
  };
  auto arrived = [&](int j) {                     // item j is in LDS (item j + 1 may be in flight)
    if (j + 1 < 2 * nb) wait_loads<Stage<G>::kLoads>();
    else wait_loads<0>();
  };
  fetch(0);
  fetch(1);

  // Q^ of the group's rows (repeated by every run of the sequence: a few
  // hundred instructions against a separate launch): q~ = fp16(q * s), the
  // exact product rounded once, HIF4 of each group (the row base over 16
  // lanes, E2 over a lane pair, E3 in-lane).
  float wq[RP][G];
#pragma unroll
  for (int p = 0; p < RP; ++p)
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const h2_t y01 = smooth_mul2(__builtin_bit_cast(h2_t, qraw[p][g].x), qs[g].x, qs[g].y);
      const h2_t y23 = smooth_mul2(__builtin_bit_cast(h2_t, qraw[p][g].y), qs[g].z, qs[g].w);
      const half_t xsm[4] = {y01[0], y01[1], y23[0], y23[1]};
      float ax[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) ax[j] = fabsf((float)xsm[j]);
      const float a4 = fmaxf(fmaxf(ax[0], ax[1]), fmaxf(ax[2], ax[3]));
      const float a8 = fmaxf(a4, __shfl_xor(a4, 1));
      float A = a8;
#pragma unroll
      for (int o = 2; o < 16; o <<= 1) A = fmaxf(A, __shfl_xor(A, o));
      const uint32_t base = e6m2_ceil(A);
      const float bval = e6m2_value(base);
      const bool e2 = a8 <= 0.875f * bval;
      const bool e3 = a4 <= (e2 ? 0.4375f : 0.875f) * bval;
      const int sh = (int)e2 + (int)e3;
      const float R = hif4_rcp_step(base);
      const float C = round_const(sh);
      uint32_t v[4], neg = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t u = __float_as_uint(__builtin_fmaf(ax[j], R, C)) - __float_as_uint(C);
        v[j] = u << (2 - sh);
        neg |= ((float)xsm[j] < 0.0f ? 32u : 0u) << (6 * j);
      }
      sl.a[((4 * p + q) * G + g) * 16 + kq] = quad_words(e2m3_pack(v) | neg, lane);
      wq[p][g] = 0.0625f * bval;
    }
  // A operands of A row n (zero where it holds no query row)
  const int arow = 4 * (n & 3) + (n >> 2);
  const bool alive = (n & 3) < RP && arow < grp;
  auto q_operands = [&](AOperand (&qa)[G]) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      u4_t d = {0, 0, 0, 0};
      if (alive) d = *reinterpret_cast<const u4_t*>(&sl.a[(arow * G + g) * 16 + 4 * q]);
      qa[g] = a_operand(d);
    }
  };
  AOperand qa[G];
  q_operands(qa);

  // --- scores ---
  // sc: the scores of the run's blocks (the lane's four keys per pass), a
  // queue whose newest entry is the last
  h2_t sc[kMaxRun][RP][2];
  h2_t rmax[RP];                                  // run maximum over the lane's keys
#pragma unroll
  for (int p = 0; p < RP; ++p) {
    rmax[p] = h2_t{(half_t)(-__builtin_inff()), (half_t)(-__builtin_inff())};
#pragma unroll
    for (int k = 0; k < kMaxRun; ++k) sc[k][p][0] = sc[k][p][1] = rmax[p];
  }
  auto shift = [&]() {
#pragma unroll
    for (int k = 0; k + 1 < kMaxRun; ++k)
#pragma unroll
      for (int p = 0; p < RP; ++p) {
        sc[k][p][0] = sc[k + 1][p][0];
        sc[k][p][1] = sc[k + 1][p][1];
      }
  };
  const MetaShifts ms = meta_shifts(q);
  uint32_t boff;
  asm("s_mov_b32 %0, 0x30000000" : "=s"(boff));
  const int clane = n * (32 * G) + 8 * q, mlane = Stage<G>::kCodes + n * (4 * G);
  // scores of a block in LDS: acc[t][p] the lane's key 4n + t of its row in pass p
  auto score = [&](const AOperand (&qa)[G], const uint8_t* blk, float (&acc)[4][RP]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const u2_t cw = *reinterpret_cast<const u2_t*>(blk + clane + 512 * G * t + 32 * g);
        const uint32_t meta = *reinterpret_cast<const uint32_t*>(blk + mlane + 64 * G * t + 4 * g);
        const f4_t dot = group_dot(qa[g], cw, meta, ms);
        const float bk = meta_base(meta, boff);
#pragma unroll
        for (int p = 0; p < RP; ++p) {
          const float d = dot[p] * bk;                              // exact
          acc[t][p] = g == 0 ? d * wq[p][0] : __builtin_fmaf(d, wq[p][g], acc[t][p]);
        }
      }
    }
    wait_lds();
  };
  for (int j = 0; j < nb; ++j) {
    const int left = w.L - 64 * (w.J0 + j);       // keys of the block and after
    arrived(j);
    float acc[4][RP];
    score(qa, &sl.buf[j & 1][0], acc);
    if (j + 2 < 2 * nb) fetch(j + 2);            // a run of one block has two items only
    shift();
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      h2_t s01 = scale2_to_f16(acc[0][p], acc[1][p], a.c), s23 = scale2_to_f16(acc[2][p], acc[3][p], a.c);
      if (left < 64) {                            // the sequence's last block: keys past its end
        const half_t ninf = (half_t)(-__builtin_inff());
        s01 = h2_t{4 * n < left ? s01[0] : ninf, 4 * n + 1 < left ? s01[1] : ninf};
        s23 = h2_t{4 * n + 2 < left ? s23[0] : ninf, 4 * n + 3 < left ? s23[1] : ninf};
      }
      sc[kMaxRun - 1][p][0] = s01;
      sc[kMaxRun - 1][p][1] = s23;
      rmax[p] = hmax2(rmax[p], hmax2(s01, s23));
    }
  }
  for (int j = nb; j < kMaxRun; ++j) shift();     // the first block's scores to the front

  // --- run maxima: publish, and take the maximum entering the run ---
  half_t m[RP];
  float l[RP], prod[RP];
  bool lost[RP];
  int any_lost = 0;
#pragma unroll
  for (int p = 0; p < RP; ++p) {
    const h2_t rm = max_row16(hmax_halves(rmax[p]));
    if (a.publish && kq == 0 && 4 * p + q < grp) {
      const uint64_t word = ((uint64_t)a.epoch << 32) | (uint64_t)__builtin_bit_cast(uint16_t, rm[0]);
      __hip_atomic_store(rs.runmax + (size_t)(h0 + 4 * p + q) * rs.stride + w.run, word, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    l[p] = 0.0f;
    prod[p] = 1.0f;
  }
#pragma unroll
  for (int p = 0; p < RP; ++p) {
    bool lp = false;
    float mm = look_back(a, rs.runmax + (size_t)(h0 + prow[p]) * rs.stride + (w.run - w.part), w.part, kq, lp);
    int lf = lp ? 1 : 0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      mm = fmaxf(mm, __shfl_xor(mm, o));
      lf |= __shfl_xor(lf, o);
    }
    m[p] = (half_t)mm;
    lost[p] = lf != 0;
    any_lost |= lf;
  }
  if (__builtin_expect(a.rescore && __ballot(any_lost != 0) != 0, 0)) {
    // a wait gave up: the maximum entering the run from the scores of the
    // sequence's earlier blocks (all of them whole); the V^ blocks that were in
    // flight to the two buffers are fetched again
    AOperand qb[G];                               // (again from LDS: held, they took others' registers)
    q_operands(qb);
    h2_t rm[RP];
#pragma unroll
    for (int p = 0; p < RP; ++p) rm[p] = h2_t{(half_t)(-__builtin_inff()), (half_t)(-__builtin_inff())};
    wait_loads<0>();
    for (int J = 0; J < w.J0; ++J) {
      load_k(J, 0);
      wait_loads<0>();
      float acc[4][RP];
      score(qb, &sl.buf[0][0], acc);
#pragma unroll
      for (int p = 0; p < RP; ++p)
        rm[p] = hmax2(rm[p], hmax2(scale2_to_f16(acc[0][p], acc[1][p], a.c), scale2_to_f16(acc[2][p], acc[3][p], a.c)));
    }
    fetch(nb);
    if (nb > 1) fetch(nb + 1);
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      m[p] = max_row16(hmax_halves(rm[p]))[0];
      lost[p] = false;
    }
  }

  // --- softmax, P^ and PV ---
  float O[NT][RP];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int p = 0; p < RP; ++p) O[t][p] = 0.0f;
  for (int i = 0; i < nb; ++i) {
    float rr[RP], sp16[RP];
#pragma unroll
    for (int p = 0; p < RP; ++p) {
      const h2_t s01 = sc[0][p][0], s23 = sc[0][p][1];
      const h2_t bm = max_row16(hmax_halves(hmax2(s01, s23)));
      const h2_t mo = {m[p], m[p]};
      const h2_t mn = hmax2(mo, bm);
      // r = E(m - m_new) and the largest P of the block, E(rowmax - m_new)
      const h2_t ra = exp2_h2(h2_t{m[p], bm[0]} - mn);
      const h2_t p01 = exp2_h2(s01 - mn), p23 = exp2_h2(s23 - mn);
      m[p] = mn[0];
      rr[p] = (float)ra[0];
      prod[p] *= rr[p];
      const float ap[4] = {(float)p01[0], (float)p01[1], (float)p23[0], (float)p23[1]};
      // P^ = HIF4(P) over the row's 64 keys
      const h2_t m4 = hmax_halves(hmax2(p01, p23));
      const float a4 = (float)m4[0], a8 = (float)max_dpp<kDppXor1>(m4)[0];
      const uint32_t base = e6m2_ceil((float)ra[1]);
      const float bval = e6m2_value(base);
      const bool e2 = a8 <= 0.875f * bval;
      const bool e3 = a4 <= (e2 ? 0.4375f : 0.875f) * bval;
      const int sh = (int)e2 + (int)e3;
      const float R = hif4_rcp_step(base);
      const float C = round_const(sh);
      uint32_t u[4], v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        u[j] = __float_as_uint(__builtin_fmaf(ap[j], R, C)) - __float_as_uint(C);   // round-half-away(a/step)
        v[j] = u[j] << (2 - sh);
      }
      sl.a[(4 * p + q) * 16 + kq] = quad_words(e2m3_pack(v), lane);
      sp16[p] = bval * 0.0625f;
      // P^ = (4 u 2^-sh) * b/16
      const float ls = NORM == 0 ? (float)(v[0] + v[1] + v[2] + v[3]) * sp16[p] : (ap[0] + ap[1]) + (ap[2] + ap[3]);
      l[p] = __builtin_fmaf(l[p], rr[p], ls);
      if (DEBUG) {
        // the row's sixteen flags (32-bit selects and shifts: a 64-bit shift
        // whose amount sits in the last allocated VGPR gave wrong bits here)
        const uint64_t b2 = __ballot(e2), b3 = __ballot(e3);
        const uint32_t f2 = (q & 2 ? (uint32_t)(b2 >> 32) : (uint32_t)b2) >> (16 * (q & 1));
        const uint32_t f3 = (q & 2 ? (uint32_t)(b3 >> 32) : (uint32_t)b3) >> (16 * (q & 1));
        if (4 * p + q < grp) {
          const size_t dj = ((size_t)(h0 + 4 * p + q) * a.batch + w.b) * a.NB + w.J0 + i;
          *reinterpret_cast<uint16_t*>(a.dbg_codes + dj * 32 + 2 * kq) =
              (uint16_t)(u[0] | u[1] << 4 | u[2] << 8 | u[3] << 12);
          if (kq == 0) {
            uint32_t w2 = 0;
            for (int k = 0; k < 8; ++k) w2 |= ((f2 >> (2 * k)) & 1u) << k;
            a.dbg_meta[dj] = base | (w2 << 8) | (f3 << 16);
          }
        }
      }
    }
    u4_t d = {0, 0, 0, 0};
    if (alive) d = *reinterpret_cast<const u4_t*>(&sl.a[arow * 16 + 4 * q]);
    const AOperand pa = a_operand(d);
    shift();
    const uint8_t* blk = &sl.buf[(nb + i) & 1][0];
    arrived(nb + i);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const u2_t cw = *reinterpret_cast<const u2_t*>(blk + n * 32 + 8 * q + 512 * t);
      const uint32_t meta = *reinterpret_cast<const uint32_t*>(blk + Stage<G>::kCodes + 4 * n + 64 * t);
      const f4_t dot = group_dot(pa, cw, meta, ms);
      const float bv = meta_base(meta, boff);
#pragma unroll
      for (int p = 0; p < RP; ++p) O[t][p] = __builtin_fmaf(O[t][p], rr[p], dot[p] * (bv * sp16[p]));
    }
    wait_lds();
    if (i + 2 < nb) fetch(nb + i + 2);
  }
#pragma unroll
  for (int p = 0; p < RP; ++p) {
    float ls = l[p];
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) ls += __shfl_xor(ls, o);
    const int r = 4 * p + q;
    if (r < grp) {
      const size_t e = (size_t)(h0 + r) * rs.stride + w.run;
      float* dst = rs.opart + e * D + n;
#pragma unroll
      for (int t = 0; t < NT; ++t) dst[16 * t] = O[t][p];
      if (kq == 0) rs.spart[e] = make_float4(lost[p] ? __builtin_nanf("") : ls, prod[p], (float)m[p], 0.0f);
    }
  }
  return kRun;
}

template <int G, int RP, int NORM, bool DEBUG>
__global__ void __launch_bounds__(64 * max_waves(G), (G * RP <= 2 ? 4 : 2)) k_decode_runs(DecodeArgs a) {
  __shared__ __align__(16) WaveLds<G, RP> lds[max_waves(G)];
  if (__builtin_expect(decode_run<G, RP, NORM, DEBUG, false>(a, lds, blockIdx.x, threadIdx.x) != kGrown, 1)) return;
  // a copy of its own: a loop around the only one holds what the runs share in
  // registers, which cost every call 0.8 us
  int run = blockIdx.x, tid;
  do {
    tid = threadIdx.x;
    asm volatile("" : "+v"(tid));         // (and so that this loop holds little)
  } while (decode_run<G, RP, NORM, DEBUG, true>(a, lds, run, tid) == kRun && (run += gridDim.x, true));
}

// ---------------------------------------------------------------------------
// 2. Merge.  One workgroup per row (b, query head), or per (row, channel
// slice) when there are few rows.  Each split wrote its l,
// the product of its blocks' rescale factors r_J = E(fp16(m_{J-1} - m_J))
// (in block order) and its running maximum after its last block.  Wave 0
// turns the products into R_s = the product over all later splits (a backward
// scan, 64 splits at a time, which also sums l_s R_s); the partial sums,
// loaded before the scan, are then weighted and added, thread (part,
// channel) taking every parts-th split, and the parts combined through LDS.
constexpr int kMergeThreads = 512;              // most per workgroup

__global__ void __launch_bounds__(kMergeThreads) k_decode_merge(DecodeArgs a) {
  extern __shared__ float R[];                    // [n_split], then partial sums, then the l sum
  const int row = blockIdx.x;                     // b * hq + head
  const int b = row / a.hq, head = row % a.hq;
  // the sequence's runs [run0, run0 + ns)
  int run0 = b * a.n_split, bps = a.bps, L = a.S;
  RunStore st = a.usual;
  if (a.packed) {
    int first = a.cu[b], next = a.cu[b + 1], end = a.cu[a.batch];
    run0 = a.runbase[b];
    asm volatile("" : "+s"(first), "+s"(next), "+s"(end), "+s"(run0));      // the loads side by side
    L = min(next - first, a.S);
    if (__builtin_expect(end > a.tokens, 0)) {
      const Bounds s = load_bounds(a, threadIdx.x & 63);
      bps = grown_run_length(a, s, threadIdx.x & 63);
      run0 = runs_before(a, s, threadIdx.x & 63, b, bps);
      st = a.grown;
    }
  } else {
    L = dseq_len(a.cu, b, a.S);
  }
  const int nblk = (L + 63) >> 6;
  if (nblk <= 0) return;
  const int ns = (nblk + bps - 1) / bps;
  const size_t first = (size_t)head * st.stride + run0;
  const int tid = threadIdx.x, lane = tid & 63, threads = blockDim.x;
  // the runs have read this row's run maxima; clearing them here
  // (a kernel write, so it is part of a captured graph too) means that no word
  // of a finished call can satisfy a later call's wait, whatever its epoch
  if (blockIdx.y == 0)
    for (int s = tid; s < ns; s += threads) st.runmax[first + s] = 0;
  const int D = a.D;
  const int CW = D / (int)gridDim.y;              // this workgroup's channels
  const int parts = threads / CW;                 // threads per channel
  float* acc_s = R + a.n_split;                   // [parts][CW]
  float* lsum_s = acc_s + parts * CW;
  const float4* sp = st.spart + first;
  // the partial sums do not depend on the scan: load them first
  const int c = tid % CW, part = tid / CW, ch = (int)blockIdx.y * CW + c;
  constexpr int kMaxHeld = 16;
  float po[kMaxHeld];
  const float* op = st.opart + first * D + ch;
#pragma unroll
  for (int k = 0; k < kMaxHeld; ++k) {
    const int s = part + k * parts;
    po[k] = s < ns ? op[(size_t)s * D] : 0.0f;
  }
  // wave 0: R_s backwards, 64 splits at a time, and l = sum_s l_s R_s
  if (tid < 64) {
    float tail = 1.0f, lpart = 0.0f;
    for (int s1 = ns; s1 > 0; s1 -= 64) {
      const int sidx = s1 - 1 - lane;
      const float4 v = sidx >= 0 ? sp[sidx] : make_float4(0.0f, 1.0f, 0.0f, 0.0f);
      float incl = v.y;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const float t = __shfl_up(incl, o);
        if (lane >= o) incl *= t;
      }
      const float excl = __shfl_up(incl, 1);
      const float rs = tail * (lane == 0 ? 1.0f : excl);
      if (sidx >= 0) {
        R[sidx] = rs;
        lpart = __builtin_fmaf(v.x, rs, lpart);
      }
      tail *= __shfl(incl, 63);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) lpart += __shfl_xor(lpart, o);
    if (lane == 0) lsum_s[0] = lpart;
  }
  __syncthreads();
  float acc = 0.0f;
#pragma unroll
  for (int k = 0; k < kMaxHeld; ++k) {
    const int s = part + k * parts;
    if (s < ns) acc = __builtin_fmaf(po[k], R[s], acc);
  }
  for (int s = part + kMaxHeld * parts; s < ns; s += parts) acc = __builtin_fmaf(op[(size_t)s * D], R[s], acc);
  acc_s[part * CW + c] = acc;
  __syncthreads();
  if (part == 0) {
    float o = acc;
    for (int p = 1; p < parts; ++p) o += acc_s[p * CW + c];
    const float lsum = lsum_s[0];
    a.o[(size_t)row * D + ch] = (half_t)(o * (1.0f / lsum));
    if (ch == 0) a.lse[(size_t)head * a.batch + b] = sp[ns - 1].z * 0.69314718055994531f + logf(lsum);
  }
}

// Epoch tags of the run maxima: a fresh value per call, starting from a
// random point.  Tags only separate eager calls; under graph replay the tag
// is the captured one, and what keeps a replay from reading the previous
// replay's words is the merge kernel clearing them (a cleared word never
// matches, the tag is never 0).
uint32_t next_epoch() {
  static std::atomic<uint32_t> counter{(uint32_t)std::random_device{}()};
  uint32_t e = counter.fetch_add(1) + 1;
  if (e == 0) e = counter.fetch_add(1) + 1;
  return e;
}

template <typename K>
hipError_t allow_lds(K kern, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

template <int G, int RP>
void launch_runs_rows(const DecodeArgs& a, int norm, bool debug, dim3 grid, dim3 block, hipStream_t st) {
  if (norm == 0) {
    if (debug) k_decode_runs<G, RP, 0, true><<<grid, block, 0, st>>>(a);
    else k_decode_runs<G, RP, 0, false><<<grid, block, 0, st>>>(a);
  } else {
    if (debug) k_decode_runs<G, RP, 1, true><<<grid, block, 0, st>>>(a);
    else k_decode_runs<G, RP, 1, false><<<grid, block, 0, st>>>(a);
  }
}

template <int G>
void launch_runs(const DecodeArgs& a, int grp, int norm, bool debug, dim3 grid, dim3 block, hipStream_t st) {
  if (grp <= 4) launch_runs_rows<G, 1>(a, norm, debug, grid, block, st);
  else launch_runs_rows<G, 2>(a, norm, debug, grid, block, st);
}

}  // namespace

hipError_t launch_decode(const DecodeLaunch& d, hipStream_t st) {
  const DecodePlan pl = plan_decode(d.batch, d.hq, d.hkv, d.D, d.NB, d.cu ? d.tokens : -1);
  uint8_t* ws = d.ws;
  const auto store = [&](long runs) {
    size_t off[4];
    decode_offsets(d.batch, d.hq, d.D, runs, pl.words(), 0, off);
    return RunStore{reinterpret_cast<float*>(ws + off[1]), reinterpret_cast<float4*>(ws + off[2]),
                    reinterpret_cast<uint64_t*>(ws + off[0]), (int)runs};
  };
  DecodeArgs a;
  a.q = d.q;
  a.s = d.s;
  a.kc = d.kc;
  a.km = d.km;
  a.vc = d.vc;
  a.vm = d.vm;
  a.cu = d.cu;
  a.usual = store(pl.runs);
  a.grown = pl.packed ? store(pl.longest) : a.usual;
  size_t off[4];
  decode_offsets(d.batch, d.hq, d.D, pl.runs, pl.words(), pl.packed, off);
  a.runbase = reinterpret_cast<int*>(ws + off[3]);
  a.epoch = next_epoch();
  a.spin_limit = d.test_no_publish ? 16 : kSpinLimit;
  a.publish = d.test_no_publish ? 0 : 1;
  a.rescore = d.test_no_publish == 1 ? 0 : 1;
  a.o = d.o;
  a.lse = d.lse;
  a.dbg_codes = d.dbg_codes;
  a.dbg_meta = d.dbg_meta;
  a.batch = d.batch;
  a.S = d.S;
  a.NB = d.NB;
  a.hq = d.hq;
  a.hkv = d.hkv;
  a.D = d.D;
  a.bps = pl.bps;
  a.n_split = (d.NB + pl.bps - 1) / pl.bps;
  a.packed = pl.packed;
  a.tokens = (int)d.tokens;
  a.waves = pl.waves;
  a.c = d.c;
  const int grp = d.hq / d.hkv;
  hipError_t e;
  const dim3 block(64 * a.waves);
  const dim3 grid((unsigned)pl.runs, (d.hkv + a.waves - 1) / a.waves);
  const bool dbg = d.dbg_codes != nullptr;
  switch (d.D) {
    case 64: launch_runs<1>(a, grp, d.norm, dbg, grid, block, st); break;
    case 128: launch_runs<2>(a, grp, d.norm, dbg, grid, block, st); break;
    default: launch_runs<4>(a, grp, d.norm, dbg, grid, block, st); break;
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (d.ev && (e = hipEventRecord(d.ev[1], st)) != hipSuccess) return e;
  // few rows: each row's channels are split over several workgroups (at
  // least 32 channels each), so that every thread holds few partials
  const long rows = (long)d.batch * d.hq;
  int slices = 1;
  while (rows * slices < kMinWorkgroups && d.D / (2 * slices) >= 32) slices *= 2;
  // two or more rows per compute unit: smaller workgroups, so that more rows
  // overlap their chains of loads (1024 rows: 7.5 us with 512 threads, 5.5 with 256)
  const int threads = rows >= 512 ? kMergeThreads / 2 : kMergeThreads;
  const size_t lds3 = ((size_t)a.n_split + threads + 1) * sizeof(float);
  if ((e = allow_lds(k_decode_merge, lds3)) != hipSuccess) return e;
  k_decode_merge<<<dim3((unsigned)rows, slices), dim3(threads), lds3, st>>>(a);
  return hipGetLastError();
}

}  // namespace hifa4
