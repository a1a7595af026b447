// Exchanges and reductions across the lanes of a 16 x 16 tile of D, shared by the head kernels that keep tokens in the rows of D.
#pragma once
#include "head_common.hpp"

namespace fef {

// Exchange between the four lane groups of 16 that share a row of D.  halves: x = [x.lo, y.lo], y = [x.hi, y.hi] by halves
// of the wavefront; quarters: x = [x0, y0, x2, y2], y = [x1, y1, x3, y3] by its rows of 16 lanes.
__device__ __forceinline__ void swap_halves(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
  x = __builtin_bit_cast(float, (unsigned)r[0]);
  y = __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ void swap_quarters(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
  x = __builtin_bit_cast(float, (unsigned)r[0]);
  y = __builtin_bit_cast(float, (unsigned)r[1]);
}
// Maximum of m0 over the four lane groups in m0 and of m1 in m1, in every lane.
__device__ __forceinline__ void group_max(float& m0, float& m1) {
  swap_halves(m0, m1);
  float m = vmax(m0, m1), o = m;
  swap_quarters(m, o);
  m0 = m1 = vmax(m, o);
  swap_halves(m0, m1);
}
// Binary tree over the 16 tokens j = 4 g + c of a 16-token tile, highest bit of j first, for two tiles at once: the sum
// of e0 in the lower half of the wavefront, that of e1 in the upper half.
__device__ __forceinline__ float group_sum(float (&e0)[4], float (&e1)[4]) {
  float r[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    swap_halves(e0[c], e1[c]);
    r[c] = e0[c] + e1[c];
  }
  swap_quarters(r[0], r[1]);
  swap_quarters(r[2], r[3]);
  float x = (r[0] + r[1]) + (r[2] + r[3]), y = x;
  swap_quarters(x, y);
  return x + y;
}

}  // namespace fef
