// The fp32 vocabulary head, one tile at a time: shared by the head kernel for fp32 inputs (head_gemm.hip) and the kernel that does the
// whole round of a toy vocabulary (verify_kernels.hip).
#pragma once
#include <float.h>

#include <type_traits>

#include "head_common.hpp"

namespace fef {
namespace {

// ---------------------------------------------------------------------------------------------
// fp32 kernel: workgroup tile of 16 tokens per wavefront (64 in the head kernel) x MR rows of H (16 to 64), k in steps of 32, wavefronts of
// 16 tokens x MR rows each on v_mfma_f32_16x16x4_f32 (products and sums in binary32, like FMA).
//
// Bound: the one pass over W (HBM), or the fp32 matrix rate once there are some tens of rows (32 rows of 131 MB: 21 and 14 us).
// W and H go straight from memory to LDS, two steps ahead in a ring of three stages: rows of 128 contiguous bytes, every W element
// once per MR rows, one barrier per step, and 31 to 51 KB per workgroup, so that three to five share a CU.  The fragments of
// a step are read while the step before is multiplied.  What it measured, per call with diagnostics and logits, against the form before
// (one step ahead through registers, 32 or 64 rows), with W still in the Infinity Cache and not: 16 rows of d = 1024, V = 32000 50 -> 40 and
// 53 -> 51 us, 32 rows 52 -> 48 and 55 -> 55; 48 rows of d = 599, V = 18136 60 -> 45 and 61 -> 46; 4 rows of d = 475, V = 17778 36 -> 28 and
// 37 -> 30; 16 rows of V = 151936 (a round) 165 -> 135.  Four or six stages and eight wavefronts: equal or slower.
//
// Operand layout of the 16x16x4 multiply (lane l, i = l % 16, g = l / 16): A[i][g], B[g][i], one
// float each.  The sums run over k in ascending order, one rounding per product like a chain of FMAs: multiply c of a step takes
// columns 4 c .. 4 c + 3, one from each lane group.  A = W, B = H: D[4 g + r][i] puts four consecutive tokens of one row in a lane.
// A stage is [rows][8 chunks of 16 bytes], chunk c of row r at c ^ ((r >> 1) & 7): two rows cover the 64 banks, so the 64 reads of
// a fragment (16 rows, the four columns of a chunk) fall on different ones.  The permutation is applied on the global side of the load.
//
// TK = 64: steps of 64 columns in two stages, for rows of W that are not whole 128-byte lines.  Where a step is 128 bytes of every row it
// touches two lines per row then, and neighbouring steps ask for each line twice; of 256 bytes it touches three.  That pays with
// tiles of 32 rows and long rows: 32 rows of d = 2548, V = 47390 133 -> 120 us per round, of d = 1028, V = 90000 114 -> 107, of d = 1644,
// V = 60000 114 -> 106 (through registers, with such steps, 121, 106 and 109); with 16 rows up to 20 % behind, with 64 rows, of which
// two workgroups share a CU and not three, 4 to 12.  [rows][16 chunks], chunk c of row r at c ^ (r & 15).
//
// VEC = 4: d is a multiple of 4, rows are 16-byte aligned and come in pieces of 16 bytes; VEC = 1: any d, 4 bytes per lane.
// STREAM_W: W in non-temporal loads (see streams_w).  WIDE: rows so long that 64 of them pass 4 GB (d > 2^24): W by 64-bit addresses.
// ---------------------------------------------------------------------------------------------
// Stages of the ring.  In pieces of 4 bytes and with 48 or 64 rows a step is 14 or 16 loads per wavefront: two stages (1078 rows of d = 106,
// V = 52940 306 -> 290 us) and the loads in groups behind one write of M0 (of d = 183, V = 60000 425 -> 411) are what it takes to stay
// level with a form that loads through registers (287 and 418).  With fewer rows three stages are up to 20 % ahead, and single loads 5 %.
constexpr int f32_stages(int mr, int vec, int tk) { return tk == 64 || (vec == 1 && mr >= 48) ? 2 : 3; }

// Direct-to-LDS loads of VEC floats per lane, to LDS offset lds_off + 4 VEC l: from an address, or from an offset in bytes to a
// uniform one.
template <int VEC>
__device__ inline void load_to_lds(const float* p, uint32_t lds_off) {
  if constexpr (VEC == 4)
    load_to_lds_16(p, lds_off);
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" :: "v"(p), "s"(lds_off) : "memory");
}
template <int VEC, bool STREAM>
__device__ inline void load_to_lds(const float* base, uint32_t offset, uint32_t lds_off) {
  static_assert(!STREAM || VEC == 4, "streams_w asks for rows of whole lines");
  if constexpr (STREAM)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" :: "v"(offset), "s"(base), "s"(lds_off) : "memory");
  else if constexpr (VEC == 4)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(offset), "s"(base), "s"(lds_off) : "memory");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" :: "v"(offset), "s"(base), "s"(lds_off) : "memory");
}
// VEC = 1: four or two loads behind one write of M0, which holds a wavefront for some tens of cycles.  The instruction's offset moves the
// LDS address and the memory address alike, 256 bytes per load, so offset (or address) j is 256 j bytes low.
__device__ inline void load_singles_to_lds(const float* base, const uint32_t (&o)[4], uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\t"
               "global_load_lds_dword %0, %4\n\tglobal_load_lds_dword %1, %4 offset:256\n\t"
               "global_load_lds_dword %2, %4 offset:512\n\tglobal_load_lds_dword %3, %4 offset:768"
               :: "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(o[3]), "s"(base), "s"(lds_off) : "memory");
}
__device__ inline void load_singles_to_lds(const float* p0, const float* p1, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, off\n\tglobal_load_lds_dword %1, off offset:256"
               :: "v"(p0), "v"(p1), "s"(lds_off) : "memory");
}
// Wait until all loads but those of the last `stages` (at most MAX) stages of PER loads are done.
template <int MAX, int PER>
__device__ inline void wait_stages(int stages) {
  if constexpr (MAX == 0) wait_newer<0>();
  else if (stages >= MAX) wait_newer<MAX * PER>();
  else wait_stages<MAX - 1, PER>(stages);
}

// One tile: 16 TW tokens from token n0 on (64-token partial n0 / 64 first) x rows m0 .. m0 + rows - 1 of the launch, by TW wavefronts of
// 16 tokens each.  h_of(m): row m.  logits, partials: of row 0, rows ldl and a.nT apart.  ring: f32_ring_floats<TW, MR, VEC, TK>() floats,
// free when the function is entered; everybody leaves it behind a barrier.
template <int TW, int MR, int VEC, int TK>
constexpr int f32_ring_floats() { return f32_stages(MR, VEC, TK) * (16 * TW + MR) * TK; }

template <int TW, int MR, int VEC, int TK, bool STREAM_W, bool WIDE, class RowPtr>
__device__ __forceinline__ void f32_tile(const HeadArgs& a, long n0, int m0, int rows, RowPtr h_of, float* logits, long ldl, float2* partials,
                                         float* ring, float (*tile_max)[TW]) {
  constexpr int NR = MR / 16;                 // 16-row groups of H
  constexpr int ST = f32_stages(MR, VEC, TK), HALVES = TK / 32, TOKENS = 16 * TW;
  constexpr int LW = TK / (4 * VEC);                                                      // load instructions per wavefront and stage
  constexpr int kLoadsH = MR * TK / (64 * VEC), LH = (kLoadsH + TW - 1) / TW;
  constexpr int kStage = (TOKENS + MR) * TK;  // floats: the rows of W, then MR rows of H
  constexpr bool MANY = VEC == 1 && MR >= 48;  // see f32_stages
  static_assert(TW % 4 == 0 && MR % 16 == 0 && kLoadsH >= LH, "whole 64-token partials");
  static_assert(!MANY || (!WIDE && LW % 4 == 0 && LH % 2 == 0), "loads in groups of four and two");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  const int d = a.d;
  const int nk = (d + 31) / 32, nsteps = (d + TK - 1) / TK;
  // 16-byte chunk c of row r of a stage lies at chunk c ^ twist(r)
  auto twist = [](int r) { return TK == 32 ? (r >> 1) & 7 : r & 15; };
  // Load instruction j of a wavefront fills 64 VEC floats of a stage, lane l the VEC of them from float l VEC on.
  uint32_t wo[LW];        // offset in bytes to the tile's first row
  const float* wp[WIDE ? LW : 1];
  const float* hp[LH];
  int wc[LW], hc[LH];     // the lane's first column within a step
  auto aim = [&](int f, int& col) __attribute__((always_inline)) -> int {
    const int r = f / TK, at = f % TK;
    col = (((at >> 2) ^ twist(r)) << 2) | (at & 3);
    return r;
  };
  const int last_v = (int)min((long)TOKENS - 1, a.V - 1 - n0);
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int r = min(aim((wave * LW + j) * 64 * VEC + lane * VEC, wc[j]), last_v);
    wo[j] = ((uint32_t)r * (uint32_t)d + (uint32_t)wc[j]) * 4u;
    if constexpr (WIDE) wp[j] = (const float*)a.W + (size_t)(n0 + r) * d + wc[j];
  }
  const float* wbase = (const float*)a.W + (size_t)n0 * d;
  const int hfirst = min(wave * LH, kLoadsH - LH);  // where the rows do not divide, the last wavefronts repeat some
#pragma unroll
  for (int j = 0; j < LH; ++j) {
    const int r = min(aim((hfirst + j) * 64 * VEC + lane * VEC, hc[j]), rows - 1);
    hp[j] = h_of(m0 + r) + hc[j];
  }
  const uint32_t slot = lds_offset(ring);
  auto fetch = [&](int k0, int stage) __attribute__((always_inline)) {
    const uint32_t at = slot + stage * (kStage * 4);
    const uint32_t at_w = at + wave * (LW * 256 * VEC), at_h = at + TOKENS * TK * 4 + hfirst * (256 * VEC);
    // (uniform; with steps of 64 the compiler has to be told)
    const float* wk = wbase + k0;
    if constexpr (TK != 32) {
      const uint64_t x = (uint64_t)(uintptr_t)wk;
      wk = (const float*)(uintptr_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x) |
                                     (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32);
    }
    auto all = [&](auto whole) __attribute__((always_inline)) {
      const auto back = [&](int col) __attribute__((always_inline)) { return whole || k0 + col < d ? 0 : col; };
      if constexpr (MANY) {
#pragma unroll
        for (int j = 0; j < LW; j += 4) {  // the offsets low by 256 bytes each, from a base that is 768 bytes low: none passes zero
          uint32_t o[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = wo[j + i] - back(wc[j + i]) * 4u + (3 - i) * 256u;
          load_singles_to_lds(wk - 3 * 64, o, at_w + j * 256);
        }
#pragma unroll
        for (int j = 0; j < LH; j += 2)
          load_singles_to_lds(hp[j] + k0 - back(hc[j]), hp[j + 1] + k0 - back(hc[j + 1]) - 64, at_h + j * 256);
      } else {
#pragma unroll
        for (int j = 0; j < LW; ++j) {
          if constexpr (WIDE) load_to_lds<VEC>(wp[j] + k0 - back(wc[j]), at_w + j * 256 * VEC);
          else load_to_lds<VEC, STREAM_W>(wk, wo[j] - back(wc[j]) * 4u, at_w + j * 256 * VEC);
        }
#pragma unroll
        for (int j = 0; j < LH; ++j) load_to_lds<VEC>(hp[j] + k0 - back(hc[j]), at_h + j * 256 * VEC);
      }
    };
    if (k0 + TK <= d) all(std::true_type{});
    else all(std::false_type{});  // columns past the row: the step's first instead, which exist; the multiplies leave them out
  };

  floatx4 acc[NR];
#pragma unroll
  for (int n = 0; n < NR; ++n) acc[n] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int t = 0; t < ST - 1 && t < nsteps; ++t) fetch(t * TK, t);
  int stage = 0;
  // The fragments of 32 columns are read while the 32 before are multiplied: a step, or half of one (the parity says which).
  float wv[2][8], hv[2][NR][8];
  int at[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) at[c] = (c ^ (twist(i16) & 7)) * 4;
  const int half0 = TK == 32 ? 0 : (i16 & 8) * 4;
  auto read = [&](int kt, auto set_tag) __attribute__((always_inline)) {
    constexpr int S = decltype(set_tag)::value;
    if constexpr (HALVES == 1 || S == 0) {
      const int step = kt / HALVES;
      wait_stages<ST - 2, LW + LH>(nsteps - 1 - step);
      lds_barrier();  // the step has arrived, and everybody is done with the one before
      if (step + ST - 1 < nsteps) fetch((step + ST - 1) * TK, stage == 0 ? ST - 1 : stage - 1);
    }
    const int half = HALVES == 1 ? 0 : S == 0 ? half0 : 32 - half0;
    const float* ws = ring + stage * kStage + (wave * 16 + i16) * TK + half + g;
    const float* hs = ring + stage * kStage + (TOKENS + i16) * TK + half + g;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      wv[S][c] = ws[at[c]];
#pragma unroll
      for (int n = 0; n < NR; ++n) hv[S][n][c] = hs[n * 16 * TK + at[c]];
    }
    if constexpr (HALVES == 1 || S == 1) stage = stage == ST - 1 ? 0 : stage + 1;
  };
  auto multiply = [&](auto set_tag) __attribute__((always_inline)) {
    constexpr int S = decltype(set_tag)::value;
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
      for (int n = 0; n < NR; ++n) acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[S][c], hv[S][n][c], acc[n], 0, 0, 0);
  };
  auto mask = [&](auto set_tag) __attribute__((always_inline)) {  // last step: columns at and past d count as zero
    constexpr int S = decltype(set_tag)::value;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const bool in = (nk - 1) * 32 + 4 * c + g < d;
      wv[S][c] = in ? wv[S][c] : 0.f;
#pragma unroll
      for (int n = 0; n < NR; ++n) hv[S][n][c] = in ? hv[S][n][c] : 0.f;
    }
  };
  using Even = std::integral_constant<int, 0>;
  using Odd = std::integral_constant<int, 1>;
  read(0, Even{});
  int kt = 1;
  for (; kt + 1 < nk; kt += 2) {
    read(kt, Odd{});
    multiply(Even{});
    read(kt + 1, Even{});
    multiply(Odd{});
  }
  if (kt < nk) {
    read(kt, Odd{});
    multiply(Even{});
    if (d % 32 != 0) mask(Odd{});
    multiply(Odd{});
  } else {
    if (d % 32 != 0) mask(Even{});
    multiply(Even{});
  }

  // epilogue: lane holds tokens v .. v + 3 of row m0 + 16 n + i16
  const long v = n0 + wave * 16 + 4 * g;
#pragma unroll
  for (int n = 0; n < NR; ++n) {
    const int rl = 16 * n + i16;
    const floatx4 l = acc[n] * a.inv_tau;
    if (rl < rows) {
      const int m = m0 + rl;
      if (a.labels) {  // cross-entropy use: keep only the label token's logit
        const long c = (long)a.labels[m] - v;
        if (c >= 0 && c < 4 && v + c < a.V) a.label_logit[m] = c == 0 ? l[0] : c == 1 ? l[1] : c == 2 ? l[2] : l[3];
      } else {
        float* dst = logits + (size_t)m * ldl + v;
        if (v + 3 < a.V) {
          *reinterpret_cast<floatx4*>(dst) = l;
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (v + c < a.V) dst[c] = l[c];
        }
      }
    }
    acc[n] = l;
    float mx = -FLT_MAX;  // not -inf: tokens past V, or of logit -inf, bring no NaN
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (v + c < a.V) mx = fmaxf(mx, l[c]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (g == 0) tile_max[rl][wave] = mx;
  }
  __syncthreads();  // also: the last reads of the ring are done
  // exponentials to LDS, [wavefront][row][token % 16]; then a quad of threads per row adds them as a binary tree over
  // the token number, highest bit first
  auto max_of = [&](int rl, int part) __attribute__((always_inline)) -> float {
    const float* m = &tile_max[rl][4 * part];
    return fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
  };
  floatx4* ex = reinterpret_cast<floatx4*>(ring);
  static_assert(TW * MR * 16 <= ST * kStage, "the exponentials fit where the stages were");
#pragma unroll
  for (int n = 0; n < NR; ++n) {
    const int rl = 16 * n + i16;
    const float mx = max_of(rl, wave >> 2);
    floatx4 e;
#pragma unroll
    for (int c = 0; c < 4; ++c) e[c] = v + c < a.V ? expf(acc[n][c] - mx) : 0.f;
    ex[(wave * MR + rl) * 4 + g] = e;
  }
  __syncthreads();
  if (tid < TW * MR) {  // whole wavefronts
    const int part = tid / (4 * MR), rl = tid / 4 % MR, q = tid & 3;
    const floatx4* p = ex + (size_t)(4 * part * MR + rl) * 4 + q;
    floatx4 e = (p[0] + p[2 * MR * 4]) + (p[MR * 4] + p[3 * MR * 4]);
#pragma unroll
    for (int c = 0; c < 4; ++c) e[c] += __shfl_xor(e[c], 2, 64);
#pragma unroll
    for (int c = 0; c < 4; ++c) e[c] += __shfl_xor(e[c], 1, 64);
    const float sum = (e[0] + e[2]) + (e[1] + e[3]);
    if (q == 0 && rl < rows && n0 + 64 * part < a.V)
      partials[(size_t)(m0 + rl) * a.nT + n0 / 64 + part] = make_float2(max_of(rl, part), sum);
  }
  __syncthreads();  // the next tile's first stages overwrite the exponentials
}

}  // namespace
}  // namespace fef
