// Internal helpers shared by the vocabulary-head kernels.
#pragma once
#include <hip/hip_ext.h>
#include <math.h>

#include "fef_device.hpp"
#include "head_rules.hpp"

// Launch a head kernel; the dispatch-timestamp events need the extended launch call, every other
// launch uses the plain one (which a capturing stream records like any kernel node).
#define FEF_LAUNCH_HEAD(kernel, grid, block, a, ...)                                              \
  do {                                                                                            \
    if ((a).ev_begin || (a).ev_end)                                                               \
      hipExtLaunchKernelGGL(kernel, grid, block, 0, (a).stream, (a).ev_begin, (a).ev_end, 0, __VA_ARGS__); \
    else                                                                                          \
      hipLaunchKernelGGL(kernel, grid, block, 0, (a).stream, __VA_ARGS__);                        \
  } while (0)

namespace fef {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// Where a running maximum starts: finite, and finite still after the multiplication by log2(e), so that a piece of
// nothing but -inf (tokens past V) leaves the partial (lowest, 0) and no NaN.
constexpr float kLowest = -2e38f;

// Workgroup barrier that waits for this wavefront's LDS traffic only.  __syncthreads() would
// also drain the vector-memory counter and with it the W tiles prefetched for later steps.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Row r of this launch (0 <= r < nrows) is row row0 + r of the stacked [draft; target] matrix.
__device__ inline const __bf16* h_row(const HeadArgs& a, int r) {
  const int g = a.row0 + r;
  return g < a.BK ? (const __bf16*)a.h_draft + (size_t)g * a.d
                  : (const __bf16*)a.h_target + (size_t)(g - a.BK) * a.d;
}

// LDS tiles of bf16 are [rows][64 k] = 128 B per row.  The LDS has 64 four-byte banks, so two
// consecutive rows cover all banks once; the eight 16-byte chunks of a row are stored at
// chunk ^ ((row >> 1) & 7) so that 16-byte reads of one k-chunk over 16 consecutive rows
// touch every bank exactly once.
#ifndef FEF_SWZ_SHIFT
#define FEF_SWZ_SHIFT 1
#endif
__device__ inline int swz(int row, int chunk) { return row * 8 + (chunk ^ ((row >> FEF_SWZ_SHIFT) & 7)); }

// Value of the neighbouring lane, lane ^ 1 (DPP quad_perm [1, 0, 3, 2]).
__device__ inline float swap_pair(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, true));
}
// global_load_lds_dwordx4: lane l copies 16 bytes from its global address to LDS offset
// lds_off + 16 l (lds_off wavefront-uniform, carried in M0).  Written as inline assembly so
// that the compiler's wait-count pass does not tie the fragment reads of one stage to the
// loads still in flight for the others (it would drain them all once per ring cycle);
// completion is tracked by hand with vmcnt before the workgroup barrier.
__device__ inline void load_to_lds_16(const void* gptr, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(gptr), "s"(lds_off) : "memory");
}
// One to four of these behind one write of M0: load q fills the 1024 bytes at lds_off + 1024 q.  (The instruction offset moves the
// LDS address and the memory address alike, so pointer q is kept q KB low.)  NT: non-temporal.
template <bool NT, int L>
__device__ __forceinline__ void load_group_to_lds(const __bf16* const (&p)[L], uint32_t lds_off) {
  static_assert(L >= 1 && L <= 4 && (!NT || L == 2 || L == 4), "");
  if constexpr (L == 4 && NT)
    asm volatile("s_mov_b32 m0, %4\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, off nt\n\tglobal_load_lds_dwordx4 %1, off offset:1024 nt\n\t"
                 "global_load_lds_dwordx4 %2, off offset:2048 nt\n\tglobal_load_lds_dwordx4 %3, off offset:3072 nt"
                 :: "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "s"(lds_off) : "memory");
  else if constexpr (L == 4)
    asm volatile("s_mov_b32 m0, %4\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, off\n\tglobal_load_lds_dwordx4 %1, off offset:1024\n\t"
                 "global_load_lds_dwordx4 %2, off offset:2048\n\tglobal_load_lds_dwordx4 %3, off offset:3072"
                 :: "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "s"(lds_off) : "memory");
  else if constexpr (L == 3)
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, off\n\tglobal_load_lds_dwordx4 %1, off offset:1024\n\t"
                 "global_load_lds_dwordx4 %2, off offset:2048"
                 :: "v"(p[0]), "v"(p[1]), "v"(p[2]), "s"(lds_off) : "memory");
  else if constexpr (L == 2 && NT)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, off nt\n\tglobal_load_lds_dwordx4 %1, off offset:1024 nt"
                 :: "v"(p[0]), "v"(p[1]), "s"(lds_off) : "memory");
  else if constexpr (L == 2)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, off\n\tglobal_load_lds_dwordx4 %1, off offset:1024"
                 :: "v"(p[0]), "v"(p[1]), "s"(lds_off) : "memory");
  else
    load_to_lds_16(p[0], lds_off);
}
// Wait until at most N of this wavefront's vector-memory operations are outstanding.
template <int N>
__device__ inline void wait_newer() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
__device__ inline uint32_t lds_offset(const void* p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)p);
}
// max of numbers that are not NaN in one instruction (fmaxf also quiets signalling NaNs, which costs a second one)
__device__ inline float vmax(float x, float y) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  return r;
}
__device__ inline float vmax3(float x, float y, float z) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
  return r;
}

}  // namespace fef
