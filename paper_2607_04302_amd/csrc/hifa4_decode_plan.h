// The decode step's index arithmetic that depends on nothing of the GPU: plain
// C++ that the kernels, the launcher and a host compiler all accept.
#pragma once

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

}  // namespace hifa4
