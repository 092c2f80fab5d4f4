// Index arithmetic that the kernels and their launches rest on and that needs no GPU: host and device code share it, and
// the host tests run it over its whole range.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define TQ_HD __host__ __device__ __forceinline__
#else
#define TQ_HD inline
#endif

namespace tq {

// What a block of a listing stream writes: `tokens` tokens start in it, `base` start before it, token t stands for the values
// [4 t, 4 t + 4) of n_values (the last one of the stream possibly for fewer).  The block's tokens sit in LDS from dword
// base % 4 on, so that its output lies there as it lies in memory relative to 16-byte pieces.
// No token may start in the block: the last block holds nothing but raw values when the stream's last marker is among the
// last words of the block before.  Its `base` then counts that marker's token too, and 4 * base lies past n_values.
struct ListingOutput {
  uint64_t piece0;   // byte of the output that belongs to byte 0 of the LDS area
  uint32_t lo, hi;   // bytes of the LDS area that are output (lo == hi: none)
};
TQ_HD ListingOutput listing_output(uint32_t base, uint32_t tokens, uint64_t n_values) {
  const uint32_t lo = (base & 3u) * 4u;
  const uint64_t first = (uint64_t)base * 4u, end = first + (uint64_t)tokens * 4u, stop = end < n_values ? end : n_values;
  return {first - lo, lo, lo + (uint32_t)(stop > first ? stop - first : 0u)};
}

}  // namespace tq
