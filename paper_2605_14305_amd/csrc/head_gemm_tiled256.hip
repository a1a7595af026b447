// Vocabulary-head kernel for all row counts and hidden sizes that the kernels with H in registers (head_gemm.hip) do not
// take, and for the cross-entropy use of the head.
//
// Workgroup tile 32 NR rows of H (NR = 1 to 8) x up to 256 tokens, k-steps of 64, v_mfma_f32_16x16x32_bf16 with the W tile
// as the A operand and H as the B operand.  Two forms:
//   WN = 2  four wavefronts in a 2 x 2 grid (rows x tokens), each 16 NR rows x 128 tokens: M > 256, d >= 1024
//   WN = 4  eight wavefronts in a 2 x 4 grid, each 16 NR rows x 64 tokens: M <= 256, and M > 256 with small d
//
// What bounds it, and what follows.
// (1) Power.  With every matrix unit busy on real data the chip lowers its clock, so energy per multiply is time.  A
// loop of nothing but multiplies on random operands runs at 2100 TFLOP/s with the 16x16x32 instruction and at 1840
// with 32x32x16 (2430 and 2480 with zeros): per product the smaller tile moves half the binary32 accumulators and
// rounds half as often, which outweighs its twice as many 16-bit operands.
// (2) Issue slots.  With one wavefront per SIMD the matrix unit idles for the length of any run of other
// instructions (it holds one multiply beyond the one in work), so fragment reads and operand loads are dealt out singly
// between the multiplies, and pointer additions are pinned behind their loads.
// (3) The epilogue, during which the matrix units idle.  With the tokens in the rows of D a lane holds four consecutive
// tokens of ONE row of H per tile: logits leave as 16-byte stores, and the (max, sum exp) of a row runs inside the
// lane over all its tiles; nothing crosses lanes at all (each of the four lane groups that share a row writes
// the partial of its own tokens to LDS, where a thread per row merges them).
// (4) Rows that do not exist.  M is cut into ceil(M / 256) row tiles of equal height, a multiple of 32 (300 rows:
// two tiles of 160, not 256 + 44), one instantiation per height.
//
// Measured (head kernel, rocprofv3; before: 32x32x16, tokens in the columns of D, 256-row tiles only):
// M = 2048 (d = 4096, V = 126464) 1697 -> 1610 us with logits, 1600 -> 1470 without (cross-entropy: 1.44 PFLOP/s, matrix
// units busy 0.72 of the cycles at 1.78 GHz); M = 300 without logits (d = 2048, V = 50257) 138 -> 67; M = 256 250 -> 238.
// Up to 128 rows, where two kernels built around streaming W stood before (persistent workgroups; W into LDS or straight
// into registers): 48 rows 189 -> 176 us, 64 rows 188 -> 178, 96 rows 207 -> 181, 128 rows 200 -> 187, and 159 -> 110 at
// 110 rows of d = 2560, V = 100003.
//
// Operand slabs go HBM/L2 -> LDS directly (global_load_lds_dwordx4: lane l of a wavefront deposits its 16 bytes at
// LDS base + 16 l): no register staging and no ds_write in the main loop.  A row of a stage is 128 bytes, so one load
// instruction fetches eight rows of 128 contiguous bytes (whole L2 lines; 64-byte segments move at about 60 % of that
// rate out of L2), and there is one workgroup barrier per 64 columns of k.  The loads are inline assembly with
// hand-counted vmcnt before each barrier: with the builtin, the compiler's wait-count pass ties the fragment reads of
// one stage to the loads in flight for the others.
//
// LDS (all 160 KB of the CU with 256 rows): H ring of two stages, W ring of three.  H comes from L2 / the Infinity
// Cache and is requested one k-step ahead; W comes from HBM and is requested two ahead.  A stage is [rows][8 chunks of
// 16 B]; the LDS has 64 four-byte banks, i.e. two such rows per sweep, so chunk c of row r is kept at position
// c ^ ((r >> 1) & 7) and the 16-byte fragment reads of 16 consecutive rows touch every bank once.  The permutation is
// applied on the global side of the load (lane l lands at LDS base + 16 l and fetches the chunk that belongs there).
//
// A k-step is two 32-wide slices.  The fragments of a slice are read while the slice before it is multiplied; the last
// slice of a step is multiplied behind the next step's barrier, under the first fragment reads of the new stage, so the
// barrier does not idle the matrix unit for the latency of those reads.
//
// Tile order: workgroup ids go round-robin over the 8 XCDs; within an XCD consecutive workgroups take the row tiles of
// one token tile, so a W tile comes from HBM once and is shared through that XCD's L2.
#include <type_traits>
#include <utility>

#include "head_common.hpp"

namespace fef {
namespace {

constexpr int BN = kTiled256Tn, BK = 64;
constexpr int kUnit = kTiled256Unit;
constexpr int kStageW = BN * 8;  // 16-byte chunks per W stage

// Which of `cnt` instructions spread evenly over `total` multiplies follows multiply m; -1: none.  cnt <= total.
constexpr int spread_at(int m, int cnt, int total) {
  for (int q = 0; q < cnt; ++q)
    if ((2 * q + 1) * total / (2 * cnt) == m) return q;
  return -1;
}
// f(integral_constant 0), f(1), .. f(N - 1), in order: an unrolled loop whose index is a constant expression.
template <class F, int... I>
__device__ __forceinline__ void for_each(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// c += w h^T on 16 tokens x 16 rows x 32 columns of k, in place.  As inline assembly because the compiler gives the
// builtin's result other registers than its addend (16x16 tiles may overlap freely), and a kernel whose accumulators
// wander needs 80 registers more than one whose accumulators stay.  The hazards that the compiler would look after: a
// multiply finds its own accumulator two dozen multiplies old or older; operands come from LDS reads, which it does
// wait for; and settle() stands between zeroing and the first multiply, and between the last and the first other use.
template <bool AGPR>
__device__ __forceinline__ void mfma16(floatx4& c, const bf16x8& w, const bf16x8& h) {
  if constexpr (AGPR) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(h));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(w), "v"(h));
}
// The same with a direct-to-LDS load (lane l: 16 bytes from p to lds + 16 l) around it: the write of M0 in front, the load
// behind, so that neither is a run of instructions between two multiplies and the multiply is the wait state that a
// load needs after a write of M0.
template <bool AGPR>
__device__ __forceinline__ void mfma16_load(floatx4& c, const bf16x8& w, const bf16x8& h, const void* p, uint32_t lds) {
  if constexpr (AGPR)
    asm volatile("s_mov_b32 m0, %4\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tglobal_load_lds_dwordx4 %3, off"
                 : "+a"(c) : "v"(w), "v"(h), "v"(p), "s"(lds) : "memory");
  else
    asm volatile("s_mov_b32 m0, %4\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tglobal_load_lds_dwordx4 %3, off"
                 : "+v"(c) : "v"(w), "v"(h), "v"(p), "s"(lds) : "memory");
}
// Every accumulator in its registers, and no multiply or move to them in flight: behind the zeroing and behind the last
// multiply.  (The empty statements keep the writers in front of the wait and the readers behind it.)
template <bool AGPR, int NT, int NR>
__device__ __forceinline__ void settle(floatx4 (&acc0)[NT][NR], floatx4 (&acc1)[NT][NR]) {
  auto pin = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        if constexpr (AGPR) asm volatile("" : "+a"(acc0[t][n]), "+a"(acc1[t][n]));
        else asm volatile("" : "+v"(acc0[t][n]), "+v"(acc1[t][n]));
      }
  };
  pin();
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  pin();
}

template <int NR, int WN, bool SHARES, bool CE>
__global__ __launch_bounds__(128 * WN) void head_tiled256_kernel(HeadArgs a, int m_tiles) {
  constexpr int NT = 16 / WN;                        // 16-token tiles per wavefront
  constexpr int BM = 32 * NR, WROWS = 16 * NR;       // rows of the workgroup tile, of a wavefront
  constexpr int LW = 16 / WN, LH = (2 * NR + WN - 1) / WN;  // load instructions per wavefront and stage (8 rows each)
  constexpr bool ONE = WN == 4;                      // two wavefronts per SIMD; as a rule one row tile
  constexpr bool ROLL = ONE;                         // H fragments in one set of registers, each re-read behind its last use
  constexpr int kStageH = BM * 8;                    // 16-byte chunks per H stage
  // Stages in LDS.  Narrow shares make short k-steps, so H is requested two steps ahead there like W, where 160 KB allow
  // (25.8 -> 22.9 us at 32 rows of d = 1536, V = 32000; 116 -> 110 at 110 rows of d = 2560, V = 100003; a fourth stage of
  // both measured nothing).  With whole tiles a third H stage costs 2 % (178 against 184 us at 64 rows of d = 4096,
  // V = 126464).
  constexpr int kRingW = 3, kRingH = SHARES && NR <= 5 ? 3 : 2;
  __shared__ bf16x8 ringH[kRingH * kStageH];
  __shared__ bf16x8 ringW[kRingW * kStageW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int i16 = lane & 15, g = lane >> 4;
  const int M = a.nrows;
  const int nk = a.d / BK;

  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int nt = xcd + 8 * (seq / m_tiles), mt = seq % m_tiles;
  if (nt >= a.nT) return;
  // tokens [n0, n_end) of this workgroup, at most 256: a whole tile, or an equal share of the vocabulary in units of 32
  // tokens (see tiled256_tiles)
  const int n_units = (a.V + kUnit - 1) / kUnit;
  const int m0 = mt * BM;
  const int n0 = SHARES ? (int)((long)nt * n_units / a.nT) * kUnit : nt * BN;
  const int n_end = min(a.V, SHARES ? (int)((long)(nt + 1) * n_units / a.nT) * kUnit : n0 + BN);

  // Every row of W starts at a multiple of 2 d bytes, so workgroups that walk k from 0 in step ask HBM for the
  // same low address bits at the same moment: with eight wavefronts each token tile starts its walk at another k-step and
  // wraps (with four and several row tiles per token tile, which share H in time through L2, that measured 2 % slower).
  const int k0 = ONE ? (int)((unsigned)(nt * 37) % (unsigned)nk) : 0;
  int h_left = nk - k0, w_left = nk - k0;  // steps until the walk is back at k = 0

  // Direct-to-LDS loads: wavefront w fills rows [8 LH w, + 8 LH) of an H stage and [8 LW w, + 8 LW) of a W stage,
  // 8 rows per instruction; lane l owns LDS slot (row 8 q + l / 8, position l % 8).  Every wavefront issues as many
  // loads as the others (the waits count them); where the rows of H do not divide, the last wavefronts repeat some.
  const int hrow0 = 8 * min(wave * LH, 4 * NR - LH);
  const __bf16* gh[LH];
  const __bf16* gw[LW];
  // With two wavefronts per SIMD up to four loads go out behind one write of M0 (the instruction offset moves the LDS
  // address and the memory address alike, so the pointers are kept 0, 1, 2, 3 KB low): every write of M0 in front of
  // a direct-to-LDS load holds the wavefront for some tens of cycles (2.7 % at M = 256).  With one wavefront per SIMD
  // single loads between two multiplies cost nothing measurable and a group would be a run.
  constexpr int kLow = ONE ? 512 : 0;
#pragma unroll
  for (int q = 0; q < LH; ++q) {
    const int rl = hrow0 + q * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((rl >> 1) & 7);
    gh[q] = h_row(a, min(m0 + rl, M - 1)) + c * 8 + k0 * BK - q * kLow;  // rows past M re-read the last row; masked later
  }
#pragma unroll
  for (int q = 0; q < LW; ++q) {
    const int rl = wave * (8 * LW) + q * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((rl >> 1) & 7);
    gw[q] = (const __bf16*)a.W + (size_t)min(n0 + rl, n_end - 1) * a.d + c * 8 + k0 * BK - q * kLow;  // past the share: its last row, masked later
  }
  const uint32_t slotH = lds_offset(ringH + hrow0 * 8), slotW = lds_offset(ringW + wave * LW * 64);
  constexpr uint32_t kBytesH = kStageH * 16, kBytesW = kStageW * 16;
  // Elements the pointers move on by after the loads of a step: one k-step, and back to k = 0 where the walk wraps.
  auto advance = [&](int& left) __attribute__((always_inline)) -> long {
    if constexpr (ONE) return --left == 0 ? (long)BK - a.d : (long)BK;
    else return BK;
  };
  // One load of this wavefront for the k-step the pointer stands at, which then moves on (the empty statement pins the
  // addition there: left alone, the compiler gathers the 64-bit additions of a step in front of the barrier).
  auto issue_one = [&](const __bf16*& p, int q, uint32_t lds, long move) __attribute__((always_inline)) {
    load_to_lds_16(p + q * kLow, lds + q * 1024);
    p += move;
    asm volatile("" : "+v"(p));
  };
  auto all_h = [&](int stage) __attribute__((always_inline)) {
    const long move = advance(h_left);
#pragma unroll
    for (int q = 0; q < LH; ++q) issue_one(gh[q], q, slotH + stage * kBytesH, move);
  };
  auto all_w = [&](int stage) __attribute__((always_inline)) {
    const long move = advance(w_left);
#pragma unroll
    for (int q = 0; q < LW; ++q) issue_one(gw[q], q, slotW + stage * kBytesW, move);
  };
  auto group = [&](auto& p, uint32_t base, int& left) __attribute__((always_inline)) {
    constexpr int L = sizeof(p) / sizeof(p[0]);
    if constexpr (L == 4)
      asm volatile("s_mov_b32 m0, %4\n\ts_nop 0\n\t"
                   "global_load_lds_dwordx4 %0, off\n\tglobal_load_lds_dwordx4 %1, off offset:1024\n\t"
                   "global_load_lds_dwordx4 %2, off offset:2048\n\tglobal_load_lds_dwordx4 %3, off offset:3072"
                   :: "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "s"(base) : "memory");
    else if constexpr (L == 3)
      asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\t"
                   "global_load_lds_dwordx4 %0, off\n\tglobal_load_lds_dwordx4 %1, off offset:1024\n\t"
                   "global_load_lds_dwordx4 %2, off offset:2048"
                   :: "v"(p[0]), "v"(p[1]), "v"(p[2]), "s"(base) : "memory");
    else if constexpr (L == 2)
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\t"
                   "global_load_lds_dwordx4 %0, off\n\tglobal_load_lds_dwordx4 %1, off offset:1024"
                   :: "v"(p[0]), "v"(p[1]), "s"(base) : "memory");
    else
      load_to_lds_16(p[0], base);
    const long move = advance(left);
#pragma unroll
    for (int q = 0; q < L; ++q) p[q] += move;
  };
  static_assert(!ONE || (LH <= 4 && LW <= 4), "groups of loads");

  // prologue: W as far ahead as its ring reaches, H likewise (one step where its ring is the shorter one)
#pragma unroll
  for (int t = 0; t < kRingW - 1; ++t) {
    if (t >= nk) break;
    if (t < kRingH - 1) all_h(t);
    all_w(t);
  }

  // acc(t, n): tokens 16 t + 4 g .. + 3 of row 16 n + i16 of the wavefront's tile
  // (two arrays: one of 1 KB per lane is not taken apart into registers)
  floatx4 acc0[NT / 2][NR], acc1[NT / 2][NR];
  auto acc_at = [&](int t, int n) __attribute__((always_inline)) -> floatx4& {
    return t < NT / 2 ? acc0[t][n] : acc1[t - NT / 2][n];
  };
#pragma unroll
  for (int t = 0; t < NT / 2; ++t)
#pragma unroll
    for (int n = 0; n < NR; ++n) acc0[t][n] = acc1[t][n] = floatx4{0.f, 0.f, 0.f, 0.f};
  settle<!ONE>(acc0, acc1);
  bf16x8 wf[2][NT], hf[ROLL ? 1 : 2][NR];

  // fragment addresses in a stage (chunks): row 16 n + i16 of this wavefront's rows, chunk 4 ks + g; the swizzle term
  // depends on i16 only because a wavefront's rows start at a multiple of 16
  int fo[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) fo[ks] = i16 * 8 + ((ks * 4 + g) ^ ((i16 >> 1) & 7));

  // none of this wavefront's rows, or none of its tokens, exists: loads and barriers only (wavefront-uniform, and said so)
  const int vw = n0 + wn * (16 * NT);  // first token of the wavefront
  const bool idle = __builtin_amdgcn_readfirstlane((int)(m0 + wm * WROWS >= M || vw >= n_end)) != 0;

  // Slice KS of the step in work is read into fragment set KS while the slice before it (set KS ^ 1; KS = 0: the last
  // slice of the step before) is multiplied.  LOADS: phase 0 requests the H stage of the next step, phase 1 the W
  // stage of the step after that.
  auto phase = [&](auto ks_tag, auto mul_tag, auto full, const bf16x8* Hs, const bf16x8* Ws, bool more, int stage)
      __attribute__((always_inline)) {
    constexpr int KS = decltype(ks_tag)::value;
    constexpr bool MUL = decltype(mul_tag)::value, FULL = decltype(full)::value;
    constexpr int TOTAL = NT * NR, LOADS = KS == 0 ? LH : LW;
    // Eight wavefronts: the multiply behind which the group of loads goes out.  At once where the lead of a k-step is
    // short for the load latency (many rows: 237 -> 224 us at M = 256, 207 -> 201 at 192; narrow shares: 216 -> 211 at 128
    // rows of d = 3584, V = 151936); in mid-phase where the pass over W is all it costs (128 rows: 187 against 191 us).
    constexpr int kLoadAt = SHARES || NR >= 5 ? 1 : TOTAL / 2 + (NR > 1 ? 2 : 0);
    bf16x8(&wr)[NT] = wf[KS];
    bf16x8(&wm_)[NT] = wf[KS ^ 1];
    bf16x8(&hr)[NR] = hf[ROLL ? 0 : KS];
    bf16x8(&hm)[NR] = hf[ROLL ? 0 : KS ^ 1];
    auto read_w = [&](int t) __attribute__((always_inline)) { wr[t] = Ws[(wn * NT + t) * 128 + fo[KS]]; };
    auto read_h = [&](int n) __attribute__((always_inline)) { hr[n] = Hs[(wm * NR + n) * 128 + fo[KS]]; };
    for_each(std::make_integer_sequence<int, TOTAL>{}, [&](auto m_tag) __attribute__((always_inline)) {
      constexpr int m = decltype(m_tag)::value, n = m / NT, t = m % NT;
      // four wavefronts: the load that goes with this multiply, and the pointer that moved with the multiply before
      constexpr int q = ROLL ? -1 : spread_at(m, LOADS, TOTAL), qb = ROLL ? -1 : spread_at(m - 1, LOADS, TOTAL);
      if constexpr (MUL) {
        if constexpr (q >= 0 && FULL)
          mfma16_load<!ONE>(acc_at(t, n), wm_[t], hm[n], KS == 0 ? gh[q < LH ? q : 0] : gw[q < LW ? q : 0],
                            (KS == 0 ? slotH + stage * kBytesH : slotW + stage * kBytesW) + q * 1024);
        else
          mfma16<!ONE>(acc_at(t, n), wm_[t], hm[n]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (q >= 0 && !(MUL && FULL)) {  // first and last steps: the load may not exist
        if (more) load_to_lds_16(KS == 0 ? gh[q < LH ? q : 0] : gw[q < LW ? q : 0],
                                 (KS == 0 ? slotH + stage * kBytesH : slotW + stage * kBytesW) + q * 1024);
      }
      if constexpr (ROLL) {
        // W fragments under the first row groups, an H fragment behind the last multiply that uses its registers
        constexpr int r = spread_at(m, NT, NR < NT ? TOTAL : NT * NT);  // one per row group where there are enough
        if constexpr (r >= 0) {
          read_w(r);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (t == NT - 1) {
          read_h(n);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (m == kLoadAt) {
          if (more) {
            if constexpr (KS == 0) group(gh, slotH + stage * kBytesH, h_left);
            else group(gw, slotW + stage * kBytesW, w_left);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        // a read after every third multiply or so, in the order the next phase wants them: h0, w0.., h1..
        constexpr int r = spread_at(m, NT + NR, TOTAL - TOTAL / 8);
        if constexpr (r >= 0) {
          if constexpr (r == 0) read_h(0);
          else if constexpr (r <= NT) read_w(r - 1);
          else read_h(r - NT);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (qb >= 0) {
          if (more) {
            const __bf16*& p = KS == 0 ? gh[qb < LH ? qb : 0] : gw[qb < LW ? qb : 0];
            p += BK;
            asm volatile("" : "+v"(p));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    });
  };

  // One k-step; outstanding loads of this wavefront on entry, oldest first: H(kt), W(kt+1) (H ring of two, W ring of
  // three), or those of the steps from kt on (rings of equal length); the barrier needs H(kt) and W(kt).  FULL:
  // kt + kRingW - 1 < nk, every refill exists and the step is one basic block.
  auto step = [&](int kt, int sw, auto parity, auto full, auto idle_tag, auto mul_tag) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full)::value;
    constexpr bool IDLE = decltype(idle_tag)::value;
    const bool more_h = FULL || kt + kRingH - 1 < nk, more_w = FULL || kt + kRingW - 1 < nk;
    const int sw2 = sw == 0 ? kRingW - 1 : sw - 1;               // stage of W(kt + kRingW - 1)
    const int sh = kRingH == kRingW ? sw : (int)decltype(parity)::value, sh1 = kRingH == kRingW ? sw2 : sh ^ 1;
    constexpr int kStep = kRingH == kRingW ? LH + LW : LW;       // younger loads per step that may stay in flight
    __builtin_amdgcn_sched_barrier(0);
    if (FULL || kt + 1 < nk) wait_newer<kStep>();
    else wait_newer<0>();
    lds_barrier();
    if constexpr (IDLE) {
      if (more_h) all_h(sh1);
      if (more_w) all_w(sw2);
    } else {
      const bf16x8* Hs = ringH + sh * kStageH;
      const bf16x8* Ws = ringW + sw * kStageW;
      phase(std::integral_constant<int, 0>{}, mul_tag, full, Hs, Ws, more_h, sh1);
      phase(std::integral_constant<int, 1>{}, std::true_type{}, full, Hs, Ws, more_w, sw2);
    }
  };
  // Two copies of the loop, chosen once: a wavefront without rows only loads and meets the barriers.  (With the choice
  // inside the step the two paths meet again in every step, and the compiler reconciles their registers there with
  // sixteen moves in front of the barrier.)
  auto walk = [&](auto idle_tag) __attribute__((always_inline)) {
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    step(0, 0, Even{}, std::false_type{}, idle_tag, std::false_type{});  // nothing to multiply yet in its first phase
    int kt = 1, sw = 1;
    for (; kt + kRingW < nk; kt += 2) {  // two full steps
      step(kt, sw, Odd{}, std::true_type{}, idle_tag, std::true_type{});
      sw = sw == kRingW - 1 ? 0 : sw + 1;
      step(kt + 1, sw, Even{}, std::true_type{}, idle_tag, std::true_type{});
      sw = sw == kRingW - 1 ? 0 : sw + 1;
    }
    for (; kt < nk; kt += 2) {  // what is left
      step(kt, sw, Odd{}, std::false_type{}, idle_tag, std::true_type{});
      sw = sw == kRingW - 1 ? 0 : sw + 1;
      if (kt + 1 == nk) break;
      step(kt + 1, sw, Even{}, std::false_type{}, idle_tag, std::true_type{});
      sw = sw == kRingW - 1 ? 0 : sw + 1;
    }
  };

  // Partials in LDS (the H ring is free by then): [slot][row of the tile], slot = 4 wn + g.
  float2* lp = reinterpret_cast<float2*>(ringH);
  if (idle) {
    walk(std::true_type{});
    lds_barrier();
#pragma unroll
    for (int n = 0; n < NR; ++n) lp[(4 * wn + g) * BM + wm * WROWS + 16 * n + i16] = make_float2(kLowest, 0.f);
  } else {
    walk(std::false_type{});
#pragma unroll
    for (int n = 0; n < NR; ++n)  // last slice of the last step
#pragma unroll
      for (int t = 0; t < NT; ++t)
        mfma16<!ONE>(acc_at(t, n), wf[1][t], hf[ROLL ? 0 : 1][n]);
    settle<!ONE>(acc0, acc1);
    lds_barrier();  // nobody reads the rings any more

    // Epilogue.  Straight from the registers, row group by row group.
    constexpr float kLog2e = 1.4426950408889634f;
    const float sc = a.inv_tau;
    const int v0 = vw + 4 * g;  // first token of the lane's piece of 16-token tile 0
    auto rows = [&](auto edge) __attribute__((always_inline)) {
      constexpr bool EDGE = decltype(edge)::value;  // some of the wavefront's tokens lie past the workgroup's
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        const int rl = wm * WROWS + 16 * n + i16, row = m0 + rl;
        const bool row_ok = row < M;
        floatx4 l[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) l[t] = acc_at(t, n) * sc;
        if constexpr (CE) {
          // The lane that holds the row's label token stores its logit.  Most row groups hold none of their labels among
          // these tokens; where one does, the lanes pass their values through LDS (the W ring is free) to index them.
          const int off = row_ok ? a.labels[row] - vw : -1;
          const bool mine = (unsigned)off < (unsigned)(16 * NT) && ((off >> 2) & 3) == g && vw + off < n_end;
          if (__builtin_amdgcn_ballot_w64(mine) != 0) {  // wavefront-uniform
            floatx4* own = reinterpret_cast<floatx4*>(ringW) + wave * (NT * kWave) + lane;
#pragma unroll
            for (int t = 0; t < NT; ++t) own[t * kWave] = l[t];
            if (mine) a.label_logit[row] = reinterpret_cast<const float*>(own + (off >> 4) * kWave)[off & 3];
          }
        } else {
          // A store instruction should write whole 128-byte lines, i.e. 8 lanes per row, but a row's values sit in four
          // lanes.  So neighbouring lanes (rows 2j, 2j + 1) trade one of every two tiles: row 2j's pair of tiles then lies
          // in both lanes, row 2j + 1's likewise (64-byte pieces cost 6 % of the kernel's time at M = 2048).
          // Non-temporal: the logits are read next by another kernel, and as ordinary stores they sit dirty in L2
          // and push out the W and H lines the neighbouring workgroups are about to ask for (6 % at M = 256).
          const bool odd = i16 & 1;
          const int row2 = row & ~1;
          const int pairs = EDGE ? (n_end - vw) / 32 : NT / 2;  // whole pairs of tiles, wavefront-uniform
          float* dst = a.logits + (size_t)row2 * a.ldl + v0 + (odd ? 16 : 0);
          floatx4 x[NT / 2], y[NT / 2];
#pragma unroll
          for (int t = 0; t < NT; t += 2)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const float near = swap_pair(l[t][c]), far = swap_pair(l[t + 1][c]);
              x[t / 2][c] = odd ? far : l[t][c];
              y[t / 2][c] = odd ? l[t + 1][c] : near;
            }
          if (row2 < M)
#pragma unroll
            for (int t = 0; t < NT; t += 2)
              if (!EDGE || t / 2 < pairs) __builtin_nontemporal_store(x[t / 2], reinterpret_cast<floatx4*>(dst + 16 * t));
          dst += a.ldl;
          if (row2 + 1 < M)
#pragma unroll
            for (int t = 0; t < NT; t += 2)
              if (!EDGE || t / 2 < pairs) __builtin_nontemporal_store(y[t / 2], reinterpret_cast<floatx4*>(dst + 16 * t));
          if constexpr (EDGE) {  // what does not fill a pair of tiles
            float* one = a.logits + (size_t)row * a.ldl + v0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              if (t / 2 < pairs || vw + 16 * t >= n_end || !row_ok) continue;
              if (v0 + 16 * t + 3 < n_end) {
                __builtin_nontemporal_store(l[t], reinterpret_cast<floatx4*>(one + 16 * t));
              } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                  if (v0 + 16 * t + c < n_end) one[16 * t + c] = l[t][c];
              }
            }
          }
        }
        if constexpr (EDGE) {
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if (v0 + 16 * t + c >= n_end) l[t][c] = -INFINITY;
        }
        float mx = kLowest;
#pragma unroll
        for (int t = 0; t < NT; ++t) mx = vmax3(vmax3(l[t][0], l[t][1], mx), l[t][2], l[t][3]);
        const float mb = mx * -kLog2e;
        float e = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          float x[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) x[c] = __builtin_amdgcn_exp2f(fmaf(l[t][c], kLog2e, mb));
          e += (x[0] + x[1]) + (x[2] + x[3]);
        }
        lp[(4 * wn + g) * BM + rl] = make_float2(mx, e);
      }
    };
    if (vw + 16 * NT <= n_end) rows(std::false_type{});  // wavefront-uniform
    else rows(std::true_type{});
  }
  lds_barrier();
  // one (max, sum exp) partial per (row, workgroup), merged in a fixed order by the thread that owns the row
  if (tid < BM && m0 + tid < M) {
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr int SLOTS = 4 * WN;
    float2 p[SLOTS];
    float mx = kLowest;
#pragma unroll
    for (int c = 0; c < SLOTS; ++c) {
      p[c] = lp[c * BM + tid];
      mx = fmaxf(mx, p[c].x);
    }
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < SLOTS; ++c) sum += p[c].y * exp2f((p[c].x - mx) * kLog2e);
    a.partials[(size_t)(m0 + tid) * a.nT + nt] = make_float2(mx, sum);
  }
}

template <int NR, int WN, bool SHARES>
hipError_t launch_tiles(const HeadArgs& a, int m_tiles) {
  const dim3 grid((unsigned)(8L * ((a.nT + 7) / 8) * m_tiles)), block(128 * WN);
  if (a.labels) FEF_LAUNCH_HEAD((head_tiled256_kernel<NR, WN, SHARES, true>), grid, block, a, a, m_tiles);
  else FEF_LAUNCH_HEAD((head_tiled256_kernel<NR, WN, SHARES, false>), grid, block, a, a, m_tiles);
  return hipGetLastError();
}

template <int NR>
hipError_t launch_one(const HeadArgs& a) {  // one row tile of 32 NR rows
  return a.nT == (a.V + BN - 1) / BN ? launch_tiles<NR, 4, false>(a, 1) : launch_tiles<NR, 4, true>(a, 1);
}

}  // namespace

// Token tiles of a launch over M rows = partials per row.  With one row tile the pass over W is what it costs, and
// workgroups of whole 256-token tiles leave many CUs without work in the last round of 256: V = 100003 is 391 tiles,
// one round and a half, V = 151936 is 594, two and a third, V = 32000 is 125, half a round.  There the tokens are dealt
// out evenly over full rounds instead, in units of 32 (128 bytes of logits): 120 -> 110 us at 110 rows (d = 2560,
// V = 100003), 233 -> 215 at 128 rows (d = 3584, V = 151936), 69 -> 51 at 64 rows (d = 4096, V = 32000), 155 -> 145 at 256
// rows.  Where the last round is nearly full (V = 126464: 494 tiles, 238 in the last round) whole tiles are 2 % ahead;
// hence the line at 200 of 256.  With several row tiles the multiplies are what it costs, and those of a partly filled
// tile are not saved.
int tiled256_tiles(int V, int M) {
  const int whole = (V + BN - 1) / BN;
  const int rounds = (whole + 255) / 256, last = whole - 256 * (rounds - 1);
  if (M > BN || last > 200) return whole;
  const int units = (V + kUnit - 1) / kUnit;
  return 256 * rounds < units ? 256 * rounds : units;
}

// ceil(M / 256) row tiles of equal height (a multiple of 32).  One row tile: eight wavefronts (two per SIMD: the kernel
// is short of memory parallelism there, not of LDS rate).  Several: four wavefronts, 160 to 256 rows; but eight where the
// walk over k is so short that prologue and epilogue, which two wavefronts per SIMD overlap better, are what a tile costs:
// 49.8 -> 46.0 us at 512 rows of d = 512, V = 50257, 95 -> 90 at 1024 rows; even at d = 1024 (68 -> 66 at 512 rows of
// V = 50257, 271 -> 274 at 1024 of V = 126464), 4 % behind at d = 4096.
hipError_t launch_head_tiled256(const HeadArgs& a) {
  const int m_tiles = (a.nrows + 255) / 256;
  const int nr = ((a.nrows + m_tiles - 1) / m_tiles + 31) / 32;
  if (m_tiles > 1 && a.d < 1024) {
    switch (nr) {
      case 5: return launch_tiles<5, 4, false>(a, m_tiles);
      case 6: return launch_tiles<6, 4, false>(a, m_tiles);
      case 7: return launch_tiles<7, 4, false>(a, m_tiles);
      default: return launch_tiles<8, 4, false>(a, m_tiles);
    }
  }
  if (m_tiles > 1) {
    switch (nr) {
      case 5: return launch_tiles<5, 2, false>(a, m_tiles);
      case 6: return launch_tiles<6, 2, false>(a, m_tiles);
      case 7: return launch_tiles<7, 2, false>(a, m_tiles);
      default: return launch_tiles<8, 2, false>(a, m_tiles);
    }
  }
  switch (nr) {
    case 1: return launch_one<1>(a);
    case 2: return launch_one<2>(a);
    case 3: return launch_one<3>(a);
    case 4: return launch_one<4>(a);
    case 5: return launch_one<5>(a);
    case 6: return launch_one<6>(a);
    case 7: return launch_one<7>(a);
    default: return launch_one<8>(a);
  }
}

}  // namespace fef
