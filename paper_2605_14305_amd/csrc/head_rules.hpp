// Rules that shape the launches of the head kernels: plain host code on sizes, without HIP, so that a program for the CPU can
// check them over all sizes.
#pragma once
#include <stddef.h>

namespace fef {

// W past the caches: non-temporal loads.  A W longer than the Infinity Cache (256 MB) comes from HBM in every call, and as
// ordinary loads it pushes what else is in use, H above all, out of the caches: per round of 64 rows of d = 4096, V = 126464
// 203 -> 179 us, of 256 rows 264 -> 254, of 128 rows of d = 4096, V = 41344 (323 MiB) 89.5 -> 85; 16 fp32 rows of d = 768, V = 132096
// 104 -> 92.
// A shorter W is another matter.  Whether it still lies in the Infinity Cache depends on what the program does between two
// calls, and non-temporal loads neither find it there nor leave it there.  45 bf16 and 20 fp32 calls of 80 to 256 MiB: where nothing
// runs between the calls ordinary loads are up to 1.5 times as fast (16 rows of d = 4864, V = 17354 44.5 against 62.6 us, 190 rows of
// d = 2560, V = 40000 60 against 77), and so is the second half of a split round (8 rows of d = 5056, V = 10577 111 against 129 us
// per round); where the cache is swept in between, non-temporal ones are 0 to 4 % ahead.  Hence the line.
// Rows of W that are not whole 128-byte lines (fp32, d not a multiple of 32): the two k-steps that share a line then fetch it twice, at
// any size of W (16 fp32 rows of d = 1046, V = 150369 164 -> 191 us with non-temporal loads, 30 of d = 2548, V = 47390 129 -> 152).
// Two row tiles share W through L2 as far as they keep in step, and non-temporal loads cost a round that (144 rows of d = 7168, V = 22000
// 124 -> 144 us where nothing runs between the calls and 127 -> 150 where the cache is swept, 160 of d = 4608, V = 30000 95 -> 102
// and level, 256 of d = 5120 to 8192 level to 4 % ahead); a cross-entropy call, which writes no logits, gains 0 to 5 % (300 rows of d = 4096,
// V = 126464 315 -> 303, of d = 1024, V = 151936 120 -> 114).
inline bool streams_w(size_t V, size_t d, size_t element_bytes, int row_tiles, bool loss) {
  return row_tiles <= (loss ? 2 : 1) && d * element_bytes % 128 == 0 && V * d * element_bytes > (size_t)256 << 20;
}

}  // namespace fef
