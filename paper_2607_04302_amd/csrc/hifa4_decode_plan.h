// The decode step's plan and index arithmetic, which need nothing of the GPU:
// plain C++ that the kernels, the launcher and a host compiler all accept.
#pragma once

#include <cstddef>
#include <cstdint>

#ifdef __HIPCC__
#define HIFA4_HD __host__ __device__ __forceinline__
#else
#define HIFA4_HD inline
#endif

namespace hifa4 {

// Byte offset, from the first key of a 64-key block, of the last key that the
// block's copies may read: key 63 or the sequence's last token.  `left` is the
// number of keys from the block's first to the sequence's end.  It is clamped
// before the product: the distance to the sequence's end in bytes exceeds 32
// bits (8 million tokens of 8 kv heads at D = 128 hold 4 GiB of codes), the 63
// rows of a block never do.
HIFA4_HD uint32_t last_key_offset(int left, uint32_t row_bytes) {
  return (uint32_t)(left < 64 ? left - 1 : 63) * row_bytes;
}

constexpr int kMaxRun = 8;               // blocks per run (the scores of a run stay in registers)
// kv heads per workgroup: at D = 256 two workgroups of four fill the LDS
HIFA4_HD constexpr int max_waves(int G) { return G <= 2 ? 8 : 4; }
constexpr int kMaxSplitsPerRow = 128;
constexpr int kMinWorkgroups = 256;      // one per compute unit
constexpr int kMaxPackedBatch = 256;     // sequences whose runs the kernel enumerates itself

inline size_t pad256(size_t x) { return (x + 255) & ~(size_t)255; }

// The size callers allocate by, a function of batch, heads and ceil(max_seqlen /
// 64) alone: n splits of 8, 4 or 2 blocks per row (the longest that gives 256
// workgroups of eight kv heads, at most 128 per row), for each a partial O, l,
// factor product and maximum, and 8 bytes per split where those splits fill
// the chip, else the room of a row's fp16 scores and block maxima.  The kernels
// below keep neither scores nor that run length; the size stays what callers
// have always been told, and the plan fits its runs into it.
inline size_t decode_workspace_bytes(int batch, int hq, int hkv, int D, int NB) {
  const long groups = (long)batch * ((hkv + 7) / 8);
  size_t n = ((size_t)NB + 7) / 8;
  for (int bps = 4; bps >= 2 && groups * (long)n < 256; bps /= 2) {
    const size_t m = ((size_t)NB + bps - 1) / bps;
    if (m > 128) break;
    n = m;
  }
  const size_t rows = (size_t)batch * hq;
  const size_t b = pad256(rows * n * D * 4) + pad256(rows * n * 16);
  if (groups * (long)n >= 256) return b + pad256(rows * n * 8);
  return b + pad256(rows * NB * 128) + pad256(rows * ((NB + 7) & ~7) * 2);
}

// Run length, workgroup shape and grid of a call.  Aimed at is one round of
// waves: the run with which all waves of the call make 16 (or 8, as the
// registers allow) per compute unit; shorter runs would only add partial
// outputs, longer ones leave the chip idle.  At least ceil(NB/128) blocks, since
// every run of a row adds to its look-back and merge, and at most 8, which is
// what the registers of a wave hold; and as many as it takes for the partials to
// fit the workspace, which lengthens the runs of 4 to 7 sequences of 32768
// tokens to 8 (half a round at 4).  A workgroup's LDS is that of eight waves
// (four at D = 256) whatever it launches, so with few kv heads fewer waves are
// resident than aimed at: at D = 128 two of a compute unit with one kv head,
// four with two.  The workgroup takes fewer waves where eight per workgroup
// would leave compute units empty.  Measured at D = 128 with four query heads per
// kv head: one sequence of 8192, 32768 and 131072 tokens of 8 kv heads 14, 21 and
// 41 us; four of 32768 tokens 37 us, with 1, 2 and 4 kv heads 23, 25 and 27 us.
struct DecodePlan {
  int waves, bps, packed;
  long runs;               // runs of the grid
  long longest;            // runs of 8 blocks of `batch` sequences of max_seqlen (the workspace always
                           // holds them): where cu_seqlens have grown past the tokens of the plan
  long words() const { return packed && longest > runs ? longest : runs; }
};

// Workspace of `runs` runs; returns its size.  The run maxima stand first, in
// the same words for the planned and the grown runs (words: the larger number
// of runs): they never hold anything else, so none is taken for a maximum.
inline size_t decode_offsets(int batch, int hq, int D, long runs, long words, int packed, size_t off[4]) {
  const size_t n = (size_t)hq * (size_t)runs;
  size_t o = 0;
  off[0] = o; o += pad256((size_t)hq * (size_t)words * 8);             // run maxima
  off[1] = o; o += pad256(n * D * 4);                                  // partial O
  off[2] = o; o += pad256(n * 16);                                     // l, factor product, max
  off[3] = o; o += packed ? pad256((size_t)batch * 4) : 0;             // first run of each sequence
  return o;
}

// tokens: the cached tokens of a THD problem, or -1 (every length is max_seqlen).
inline DecodePlan plan_decode(int batch, int hq, int hkv, int D, int NB, long tokens) {
  const int waves_per_cu = (D / 64) * (hq / hkv > 4 ? 2 : 1) <= 2 ? 16 : 8;
  long slots = (long)kMinWorkgroups * waves_per_cu / hkv;              // runs resident at once
  if (slots < 1) slots = 1;
  const size_t room = decode_workspace_bytes(batch, hq, hkv, D, NB);
  DecodePlan p;
  const bool pack = tokens >= 0 && batch <= kMaxPackedBatch;
  long blocks = (long)batch * NB;
  if (pack && tokens / 64 + batch < blocks) blocks = tokens / 64 + batch;
  long bps = (blocks + slots - 1) / slots;
  const long least = (NB + kMaxSplitsPerRow - 1) / kMaxSplitsPerRow;
  if (bps < least) bps = least;
  if (bps > kMaxRun) bps = kMaxRun;
  p.longest = (long)batch * ((NB + kMaxRun - 1) / kMaxRun);
  for (;; ++bps) {
    p.bps = (int)bps;
    p.packed = pack;
    p.runs = (long)batch * ((NB + bps - 1) / bps);
    if (pack && tokens / (64 * bps) + batch < p.runs) p.runs = tokens / (64 * bps) + batch;
    size_t off[4];
    if (decode_offsets(batch, hq, D, p.runs, p.words(), p.packed, off) <= room) break;
    if (bps < kMaxRun) continue;
    p.packed = 0;                        // always fits
    p.runs = p.longest;
    break;
  }
  p.waves = hkv < max_waves(D / 64) ? hkv : max_waves(D / 64);
  while (p.waves > 1 && p.runs * ((hkv + p.waves - 1) / p.waves) < kMinWorkgroups) p.waves = (p.waves + 1) / 2;
  return p;
}

}  // namespace hifa4
