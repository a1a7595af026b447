// Vocabulary-head kernel for all row counts, hidden sizes and vocabularies that the kernels for up to 32 rows (head_gemm.hip,
// head_slices.hip) and head_runs_kernel (short runs, runs of 257 to 512 tokens, short vocabularies: head_runs.hip) do not take, and for the
// cross-entropy use of the head but for a few hundred rows in one row tile (head_loss.hip).  Which kernel a call takes: head_rules.hpp.
//
// Workgroup tile 32 NR rows of H (NR = 1 to 8) x up to 256 tokens, k-steps of 64, v_mfma_f32_16x16x32_bf16 with the W tile
// as the A operand and H as the B operand.  Two grids of wavefronts:
//   WN = 2  four in a 2 x 2 grid (rows x tokens), each 16 NR rows x 128 tokens: M > 256
//   WN = 4  eight in a 2 x 4 grid, each 16 NR rows x 64 tokens: M <= 256, and the cross-entropy of some more (launch_head_tiled256)
// and five forms: kTiles (whole tiles of 256 tokens), kRuns64 and kRuns16 (M <= 128: one workgroup per CU takes a run of
// 64- or 16-token units, 256 tokens at a time), and the two of the cross-entropy, kLossTiles and kLossShares.
//
// The order of the sums.  A draw or an accept test can hang on the last bit of a sum, and with it the rest of the round, so
// in the first three forms the order in which terms are added is part of the result and does not follow the tiles:
//   a logit   groups of 16 columns (a 16x16x32 multiply gives bit for bit what two 32x32x16 in a row give), ascending
//             from a start that depends on the token's tile or run b alone, and round to it again: kTiles 64 (37 b mod d/64)
//             for M <= 256 and 0 above, kRuns64 32 (37 b mod d/32), kRuns16 128 (37 b mod d/128)
//   a partial (max, sum exp) of 64 neighbouring tokens: tokens j and j + 32 first, then a binary tree over the bits of
//             j < 32 in the order 3, 2, 1, 0, 4.  kTiles with M > 256, where 128 tokens x 128 rows exist (blocks aligned
//             to 128): of the 64 tokens whose number has bit 4 clear or set, (j + j32) + (j64 + j96) first, then bits 3,
//             2, 1, 0.  kRuns16: of 16 tokens, four neighbours in order, then bits 2 and 3.
//   a row's   the partials of a tile in ascending order; kRuns64 goes on from tile to tile; kRuns16 keeps eight chains,
//             every eighth tile of the run each, and adds the chains at the end.
// The sums over lanes and the runs that this takes cost nothing measurable at M = 2048 and 2 to 5 % up to 128 rows.
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
// tokens of ONE row of H per tile: logits leave as 16-byte stores, and most of the (max, sum exp) of a row runs inside the
// lane; the four lane groups that share a row trade with v_permlane16_swap / v_permlane32_swap, two sums per exchange
// (ten exchanges per 16 rows x 64 tokens), and a thread per row merges what meets in LDS.  In the cross-entropy nothing
// crosses lanes at all: each lane group writes the partial of its own tokens to LDS.
// (4) Rows that do not exist, and CUs without a workgroup.  M is cut into row tiles of equal height, a multiple of 32 (300 rows:
// two tiles of 160, not 256 + 44), more of them where the vocabulary is short (row_tiles), one instantiation per height.
//
// Measured (head kernel by HIP events, unless marked t: by trace; before: W in ordinary loads, as few row tiles as the rows take):
// d = 4096, V = 126464: 48 rows 182 -> 163 us, 64 rows 188 -> 166 (6.4 TB/s), 96 rows 187 -> 168, 128 rows 197 -> 171, 256 rows 240 -> 237
// to 238 (t, on one other machine: 223 -> 215), 512 rows 426 -> 423 to 432, 2048 rows 1590 -> 1600 to 1620 (other machines); 128 rows of
// d = 3584, V = 151936 222 -> 203.  Cross-entropy, 2048 rows 1470 to 1517 (1.40 to 1.43
// PFLOP/s, matrix units busy 0.75 of the cycles at 1.77 GHz).
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
#include "head_swaps.hpp"

namespace fef {
namespace {

constexpr int BN = kTiled256Tn, BK = 64;
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
// multiply finds its own accumulator NT NR multiplies old, 4 at the least, and would need no wait states even right behind
// the multiply that wrote it (the same instruction on the same registers is forwarded: the compiler issues such chains
// back to back); operands come from LDS reads, which it does wait for, or from drop(), which waits itself; and settle()
// stands between zeroing and the first multiply, and between the last and the first other use.  The build checks the
// assembly for it (check_accumulators_isa in build.py).
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

// What a launch is for; see "The order of the sums" above.
enum Form { kTiles, kRuns64, kRuns16, kLossTiles, kLossShares };
constexpr int form_unit(Form f) { return f == kRuns64 ? 64 : f == kRuns16 ? 16 : f == kLossShares ? kTiled256Unit : BN; }

// STREAM_W: the refills of the W ring are non-temporal loads (see streams_w).
template <int NR, int WN, Form F, bool STREAM_W>
__global__ __launch_bounds__(128 * WN) void head_tiled256_kernel(HeadArgs a, int m_tiles) {
  constexpr bool CE = F == kLossTiles || F == kLossShares;
  constexpr bool RUN = F == kRuns64 || F == kRuns16;  // a workgroup takes a run of tokens, 256 at a time
  constexpr bool SHARES = RUN || F == kLossShares;
  constexpr int NT = 16 / WN;                        // 16-token tiles per wavefront
  constexpr int BM = 32 * NR, WROWS = 16 * NR;       // rows of the workgroup tile, of a wavefront
  constexpr int LW = 16 / WN, LH = (2 * NR + WN - 1) / WN;  // load instructions per wavefront and stage (8 rows each)
  constexpr bool ONE = WN == 4;                      // two wavefronts per SIMD; as a rule one row tile
  constexpr bool ROLL = ONE;                         // H fragments in one set of registers, each re-read behind its last use
  constexpr int kStageH = BM * 8;                    // 16-byte chunks per H stage
  // Stages in LDS.  Narrow shares and runs make short k-steps, so H is requested two steps ahead there like W, where 160 KB
  // allow (rounds of 64 rows of d = 4096, V = 32000 69.2 -> 60.5 us together with the place of the loads, see kLoadAt; 254 ->
  // 238 at 128 rows of d = 3584, V = 151936; nothing at V = 126464; a fourth stage of both measured nothing).  With whole
  // tiles a third H stage costs 2 %.
  constexpr int kRingW = 3, kRingH = SHARES && NR <= 5 ? 3 : 2;
  __shared__ bf16x8 ringH[kRingH * kStageH];
  __shared__ bf16x8 ringW[kRingW * kStageW];
  constexpr int SLOTS = F == kRuns16 ? 16 : CE ? 4 * WN : 4;  // partials per row that meet in LDS
  __shared__ float2 run_part[RUN ? SLOTS * BM : 1];  // runs: their own place, the rings take the next tile's stages meanwhile
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int i16 = lane & 15, g = lane >> 4;
  const int M = a.nrows;
  const int nk = a.d / BK;

  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int nt = xcd + 8 * (seq / m_tiles), mt = seq % m_tiles;
  if (nt >= a.nT) return;
  // tokens [n0, n_stop) of this workgroup: a whole tile, or an equal share of the vocabulary in units of 16, 32 or 64
  // tokens; [n0, n_end) of the tile in work, at most 256
  constexpr int kUnit = form_unit(F);
  const int n_units = (a.V + kUnit - 1) / kUnit;
  const int m0 = mt * BM;
  int n0 = SHARES ? (int)((long)nt * n_units / a.nT) * kUnit : nt * BN;
  const int n_stop = min(a.V, SHARES ? (int)((long)(nt + 1) * n_units / a.nT) * kUnit : n0 + BN);
  int n_end = RUN ? min(n_stop, n0 + BN) : n_stop;

  // Every row of W starts at a multiple of 2 d bytes, so workgroups that walk k from 0 in step ask HBM for the
  // same low address bits at the same moment: with eight wavefronts each token tile starts its walk at another k-step and
  // wraps (with four and several row tiles per token tile, which share H in time through L2, that measured 2 % slower).
  // In units of kStart columns, which for the runs are what their order of sums is defined by.
  constexpr int kStart = F == kRuns64 ? 32 : F == kRuns16 ? 128 : BK;
  const int start = ONE ? (int)((unsigned)(nt * 37) % (unsigned)(a.d / kStart)) * kStart : 0;
  // A start in the middle of a k-step (HALF): the walk takes that step twice, its second half first of all and its first
  // half last of all.  (Steps that begin there would read every 128-byte line in two halves: 64 rows 237 against 198 us.)
  constexpr bool HALF = kStart % BK != 0;
  const bool half = HALF && start % BK != 0;
  const int k0 = start / BK, nsteps = nk + (half ? 1 : 0);
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
  auto aim_w = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < LW; ++q) {
      const int rl = wave * (8 * LW) + q * 8 + (lane >> 3);
      const int c = (lane & 7) ^ ((rl >> 1) & 7);
      // past the share: its last row, masked later
      gw[q] = (const __bf16*)a.W + (size_t)min(n0 + rl, n_end - 1) * a.d + c * 8 + k0 * BK - q * kLow;
    }
  };
  aim_w();
  const uint32_t slotH = lds_offset(ringH + hrow0 * 8), slotW = lds_offset(ringW + wave * LW * 64);
  constexpr uint32_t kBytesH = kStageH * 16, kBytesW = kStageW * 16;
  // Elements the pointers move on by after the loads of a step: one k-step, and back to k = 0 where the walk wraps.
  auto advance = [&](int& left) __attribute__((always_inline)) -> long {
    if constexpr (ONE) return --left == 0 ? (long)BK - a.d : (long)BK;
    else return BK;
  };
  // One load of this wavefront for the k-step the pointer stands at, which then moves on (the empty statement pins the
  // addition there: left alone, the compiler gathers the 64-bit additions of a step in front of the barrier).
  // (uniform; inside the loop over a run's tiles the compiler has to be told)
  auto scalar = [&](uint32_t x) __attribute__((always_inline)) -> uint32_t {
    if constexpr (RUN) return __builtin_amdgcn_readfirstlane(x);
    else return x;
  };
  auto issue_one = [&](const __bf16*& p, int q, uint32_t lds, long move) __attribute__((always_inline)) {
    load_to_lds_16(p + q * kLow, scalar(lds + q * 1024));
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
  auto group = [&](auto& p, uint32_t base, int& left, auto stream) __attribute__((always_inline)) {
    constexpr int L = sizeof(p) / sizeof(p[0]);
    static_assert(!decltype(stream)::value || L == 4, "W is streamed in groups of four");
    load_group_to_lds<decltype(stream)::value>(p, scalar(base));
    const long move = advance(left);
#pragma unroll
    for (int q = 0; q < L; ++q) p[q] += move;
  };
  static_assert(!ONE || (LH <= 4 && LW <= 4), "groups of loads");

  // prologue: W as far ahead as its ring reaches, H likewise (one step where its ring is the shorter one)
  auto prologue = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < kRingW - 1; ++t) {
      if (t >= nsteps) break;
      if (t < kRingH - 1) all_h(t);
      all_w(t);
    }
  };
  prologue();

  // acc(t, n): tokens 16 t + 4 g .. + 3 of row 16 n + i16 of the wavefront's tile
  // (two arrays: one of 1 KB per lane is not taken apart into registers)
  floatx4 acc0[NT / 2][NR], acc1[NT / 2][NR];
  auto acc_at = [&](int t, int n) __attribute__((always_inline)) -> floatx4& {
    return t < NT / 2 ? acc0[t][n] : acc1[t - NT / 2][n];
  };
  bf16x8 wf[2][NT], hf[ROLL ? 1 : 2][NR];

  // fragment addresses in a stage (chunks): row 16 n + i16 of this wavefront's rows, chunk 4 ks + g; the swizzle term
  // depends on i16 only because a wavefront's rows start at a multiple of 16
  int fo[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) fo[ks] = i16 * 8 + ((ks * 4 + g) ^ ((i16 >> 1) & 7));

  // Slice KS of the step in work is read into fragment set KS while the slice before it (set KS ^ 1; KS = 0: the last
  // slice of the step before) is multiplied.  LOADS: phase 0 requests the H stage of the next step, phase 1 the W
  // stage of the step after that.
  auto phase = [&](auto ks_tag, auto mul_tag, auto full, const bf16x8* Hs, const bf16x8* Ws, bool more, int stage)
      __attribute__((always_inline)) {
    constexpr int KS = decltype(ks_tag)::value;
    constexpr bool MUL = decltype(mul_tag)::value, FULL = decltype(full)::value;
    constexpr int TOTAL = NT * NR, LOADS = KS == 0 ? LH : LW;
    static_assert(ROLL || spread_at(TOTAL - 1, LOADS, TOTAL) < 0, "a load's pointer moves on behind the next multiply");
    // Eight wavefronts: the multiply behind which the group of loads goes out.  At once where the lead of a k-step is
    // short for the load latency (many rows: 237 -> 224 us at M = 256, 207 -> 201 at 192; narrow shares and runs: 254 -> 240
    // per round of 128 rows of d = 3584, V = 151936; level at V = 126464); in mid-phase with whole tiles of up to 128 rows,
    // where the pass over W is all it costs (187 against 191 us).
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
            if constexpr (KS == 0) group(gh, slotH + stage * kBytesH, h_left, std::false_type{});
            else group(gw, slotW + stage * kBytesW, w_left, std::bool_constant<STREAM_W>{});
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

  // The half of the first and of the last step that the walk does not take counts as zero (both operands, so that an
  // infinite one brings no NaN); the wait is for these writes in front of a multiply.
  auto drop = [&](bf16x8(&w)[NT]) __attribute__((always_inline)) {
    auto one = [&](bf16x8& f) __attribute__((always_inline)) {
      f = half ? bf16x8{} : f;
      asm volatile("" : "+v"(f));
    };
#pragma unroll
    for (int t = 0; t < NT; ++t) one(w[t]);
#pragma unroll
    for (int n = 0; n < NR; ++n) one(hf[0][n]);
    asm volatile("s_nop 7" ::: "memory");
  };

  // One k-step; outstanding loads of this wavefront on entry, oldest first: H(kt), W(kt+1) (H ring of two, W ring of
  // three), or those of the steps from kt on (rings of equal length); the barrier needs H(kt) and W(kt).  FULL:
  // kt + kRingW - 1 < nsteps, every refill exists and the step is one basic block.
  auto step = [&](int kt, int sw, auto parity, auto full, auto idle_tag, auto mul_tag) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full)::value;
    constexpr bool IDLE = decltype(idle_tag)::value;
    const bool more_h = FULL || kt + kRingH - 1 < nsteps, more_w = FULL || kt + kRingW - 1 < nsteps;
    const int sw2 = sw == 0 ? kRingW - 1 : sw - 1;               // stage of W(kt + kRingW - 1)
    const int sh = kRingH == kRingW ? sw : (int)decltype(parity)::value, sh1 = kRingH == kRingW ? sw2 : sh ^ 1;
    constexpr int kStep = kRingH == kRingW ? LH + LW : LW;       // younger loads per step that may stay in flight
    __builtin_amdgcn_sched_barrier(0);
    if (FULL || kt + 1 < nsteps) wait_newer<kStep>();
    else wait_newer<0>();
    lds_barrier();
    if constexpr (IDLE) {
      if (more_h) all_h(sh1);
      if (more_w) all_w(sw2);
    } else {
      const bf16x8* Hs = ringH + sh * kStageH;
      const bf16x8* Ws = ringW + sw * kStageW;
      phase(std::integral_constant<int, 0>{}, mul_tag, full, Hs, Ws, more_h, sh1);
      if constexpr (HALF && !decltype(mul_tag)::value) drop(wf[0]);
      phase(std::integral_constant<int, 1>{}, std::true_type{}, full, Hs, Ws, more_w, sw2);
    }
  };
  // Two copies of the loop, chosen once: a wavefront without rows only loads and meets the barriers.  (With the choice
  // inside the step the two paths meet again in every step, and the compiler reconciles their registers there with
  // sixteen moves in front of the barrier.)
  auto walk = [&](auto idle_tag) __attribute__((always_inline)) {
    using Yes = std::true_type;
    using No = std::false_type;
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    step(0, 0, Even{}, No{}, idle_tag, No{});  // nothing to multiply yet in its first phase
    int kt = 1, sw = 1;
    for (; kt + kRingW < nsteps; kt += 2) {  // two full steps
      step(kt, sw, Odd{}, Yes{}, idle_tag, Yes{});
      sw = sw == kRingW - 1 ? 0 : sw + 1;
      step(kt + 1, sw, Even{}, Yes{}, idle_tag, Yes{});
      sw = sw == kRingW - 1 ? 0 : sw + 1;
    }
    for (; kt < nsteps; kt += 2) {  // what is left
      step(kt, sw, Odd{}, No{}, idle_tag, Yes{});
      sw = sw == kRingW - 1 ? 0 : sw + 1;
      if (kt + 1 == nsteps) break;
      step(kt + 1, sw, Even{}, No{}, idle_tag, Yes{});
      sw = sw == kRingW - 1 ? 0 : sw + 1;
    }
  };

  // Partials in LDS, [slot][row of the tile].  Where a workgroup has one tile the H ring is free by then.
  float2* lp = RUN ? run_part : reinterpret_cast<float2*>(ringH);
  constexpr float kLog2e = 1.4426950408889634f;
  // Runs: (max, sum exp) of row tid over the tiles done so far, kRuns16: for each eighth 16-token tile of the run
  constexpr int CHAINS = F == kRuns16 ? 8 : 1;
  float run_m[CHAINS], run_s[CHAINS];
#pragma unroll
  for (int w = 0; w < CHAINS; ++w) {
    run_m[w] = -INFINITY;
    run_s[w] = 0.f;
  }

  for (;;) {  // once, or over the tiles of a run
  const int vw = n0 + wn * (16 * NT);  // first token of the wavefront
  // none of this wavefront's rows, or none of its tokens, exists: loads and barriers only (wavefront-uniform, and said so)
  const bool idle = __builtin_amdgcn_readfirstlane((int)(m0 + wm * WROWS >= M || vw >= n_end)) != 0;
  const int tile0 = n0, tile_end = n_end;
  // Behind the barrier after the walk nobody reads the rings any more: the first stages of the run's next tile are on
  // their way during the epilogue of this one.  (Its stores come behind them in the counter of the vector-memory
  // operations, so the waits of the next walk can only wait for more than they need.)
  auto next_tile = [&]() __attribute__((always_inline)) {
    if constexpr (RUN) {
      n0 += BN;
      if (n0 < n_stop) {
        n_end = min(n_stop, n0 + BN);
        h_left = w_left = nk - k0;  // the H pointers stand where they began, or a step behind
        if (HALF && half)
#pragma unroll
          for (int q = 0; q < LH; ++q) gh[q] -= BK;
        aim_w();
        prologue();
      }
    }
  };
  if (idle) {
    walk(std::true_type{});
    lds_barrier();
    next_tile();
#pragma unroll
    for (int n = 0; n < NR; ++n) {
      const int rl = wm * WROWS + 16 * n + i16;
      if constexpr (SLOTS == 4 * WN) lp[(4 * wn + g) * BM + rl] = make_float2(kLowest, 0.f);
      else if (g < SLOTS / WN) lp[(SLOTS / WN * wn + g) * BM + rl] = make_float2(kLowest, 0.f);
    }
  } else {
#pragma unroll
    for (int t = 0; t < NT / 2; ++t)
#pragma unroll
      for (int n = 0; n < NR; ++n) acc0[t][n] = acc1[t][n] = floatx4{0.f, 0.f, 0.f, 0.f};
    settle<!ONE>(acc0, acc1);
    walk(std::false_type{});
    if constexpr (HALF) drop(wf[1]);
#pragma unroll
    for (int n = 0; n < NR; ++n)  // last slice of the last step
#pragma unroll
      for (int t = 0; t < NT; ++t)
        mfma16<!ONE>(acc_at(t, n), wf[1][t], hf[ROLL ? 0 : 1][n]);
    settle<!ONE>(acc0, acc1);
    lds_barrier();  // nobody reads the rings any more
    next_tile();

    // Epilogue.  Straight from the registers, row group by row group.
    const float sc = a.inv_tau;
    const int v0 = vw + 4 * g;  // first token of the lane's piece of 16-token tile 0
    auto rows = [&](auto edge) __attribute__((always_inline)) {
      constexpr bool EDGE = decltype(edge)::value;  // some of the wavefront's tokens (or, kTiles with WN = 2, rows) do not exist
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
          const bool mine = (unsigned)off < (unsigned)(16 * NT) && ((off >> 2) & 3) == g && vw + off < tile_end;
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
          const int pairs = EDGE ? (tile_end - vw) / 32 : NT / 2;  // whole pairs of tiles, wavefront-uniform
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
              if (t / 2 < pairs || vw + 16 * t >= tile_end || !row_ok) continue;
              if (v0 + 16 * t + 3 < tile_end) {
                __builtin_nontemporal_store(l[t], reinterpret_cast<floatx4*>(one + 16 * t));
              } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                  if (v0 + 16 * t + c < tile_end) one[16 * t + c] = l[t][c];
              }
            }
          }
        }
        if constexpr (EDGE) {
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if (v0 + 16 * t + c >= tile_end) l[t][c] = -INFINITY;
        }
        auto max_of = [&](float mx, int t) __attribute__((always_inline)) -> float {
          return vmax3(vmax3(l[t][0], l[t][1], mx), l[t][2], l[t][3]);
        };
        // l[t] becomes exp(l[t] - mx)
        auto exps = [&](int t, float mx) __attribute__((always_inline)) {
          const float mb = mx * -kLog2e;
#pragma unroll
          for (int c = 0; c < 4; ++c) l[t][c] = __builtin_amdgcn_exp2f(fmaf(l[t][c], kLog2e, mb));
        };
        if constexpr (CE) {
          // nothing crosses lanes: the partial of the lane's own tokens
          float mx = kLowest;
#pragma unroll
          for (int t = 0; t < NT; ++t) mx = max_of(mx, t);
          float e = 0.f;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            exps(t, mx);
            e += (l[t][0] + l[t][1]) + (l[t][2] + l[t][3]);
          }
          lp[(4 * wn + g) * BM + rl] = make_float2(mx, e);
        } else if constexpr (F == kRuns16) {
          // one partial per 16-token tile: lane group g ends with that of tile g
          float m[4], e[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) m[t] = max_of(kLowest, t);
          swap_quarters(m[0], m[1]);
          swap_quarters(m[2], m[3]);
          float lo = vmax(m[0], m[1]), hi = vmax(m[2], m[3]);
          swap_halves(lo, hi);
          const float mine = vmax(lo, hi);
          m[0] = m[2] = mine;
          swap_halves(m[0], m[2]);
          m[1] = m[0];
          m[3] = m[2];
          swap_quarters(m[0], m[1]);
          swap_quarters(m[2], m[3]);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            exps(t, m[t]);
            e[t] = ((l[t][0] + l[t][1]) + l[t][2]) + l[t][3];
          }
          swap_quarters(e[0], e[1]);
          swap_quarters(e[2], e[3]);
          float x = e[0] + e[1], y = e[2] + e[3];
          swap_halves(x, y);
          lp[(4 * wn + g) * BM + rl] = make_float2(mine, x + y);
        } else {
          // sum over 64 neighbouring tokens, tiles t0 to t0 + 3, in every lane
          auto block_sum = [&](int t0, float mx) __attribute__((always_inline)) -> float {
            float e0[4], e1[4];
#pragma unroll
            for (int t = t0; t < t0 + 4; ++t) exps(t, mx);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              e0[c] = l[t0][c] + l[t0 + 2][c];
              e1[c] = l[t0 + 1][c] + l[t0 + 3][c];
            }
            float x = group_sum(e0, e1), y = x;
            swap_halves(x, y);
            return x + y;
          };
          if constexpr (NT == 4) {
            float mx = kLowest;
#pragma unroll
            for (int t = 0; t < NT; ++t) mx = max_of(mx, t);
            float o = mx;
            group_max(mx, o);
            const float e = block_sum(0, mx);
            if (g == 0) lp[wn * BM + rl] = make_float2(mx, e);
          } else {
            // 128 tokens of 128 rows that all exist: the even and the odd 16-token tiles; else the two blocks of 64
            const bool whole = !EDGE || ((row & ~15) < (M & ~127) && vw + 128 <= tile_end);  // wavefront-uniform
            float m0 = kLowest, m1 = kLowest, e;
            if (whole) {
#pragma unroll
              for (int t = 0; t < NT; t += 2) {
                m0 = max_of(m0, t);
                m1 = max_of(m1, t + 1);
              }
              group_max(m0, m1);
              float e0[4], e1[4];
#pragma unroll
              for (int t = 0; t < NT; t += 2) {
                exps(t, m0);
                exps(t + 1, m1);
              }
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                e0[c] = (l[0][c] + l[2][c]) + (l[4][c] + l[6][c]);
                e1[c] = (l[1][c] + l[3][c]) + (l[5][c] + l[7][c]);
              }
              e = group_sum(e0, e1);
            } else {
#pragma unroll
              for (int t = 0; t < NT / 2; ++t) {
                m0 = max_of(m0, t);
                m1 = max_of(m1, t + NT / 2);
              }
              group_max(m0, m1);
              const float x = block_sum(0, m0), y = block_sum(NT / 2, m1);
              e = g < 2 ? x : y;
            }
            if ((g & 1) == 0) lp[(2 * wn + (g >> 1)) * BM + rl] = make_float2(g ? m1 : m0, e);
          }
        }
      }
    };
    const bool interior = vw + 16 * NT <= tile_end && (CE || NT == 4 || m0 + (wm + 1) * WROWS <= (M & ~127));
    if (__builtin_amdgcn_readfirstlane((int)interior) != 0) rows(std::false_type{});
    else rows(std::true_type{});
  }
  lds_barrier();
  // One (max, sum exp) partial per (row, workgroup), merged in a fixed order by the thread that owns the row.  A run has
  // its next partials written behind the barriers of its next walk.
  if (tid < BM && m0 + tid < M) {
    if constexpr (F == kRuns16) {
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int w = t & 7;
        if (tile0 + 16 * t < tile_end) {
          const float2 p = lp[t * BM + tid];
          if (p.x > run_m[w]) {
            run_s[w] = run_s[w] * exp2f((run_m[w] - p.x) * kLog2e) + p.y;
            run_m[w] = p.x;
          } else {
            run_s[w] += p.y * exp2f((p.x - run_m[w]) * kLog2e);
          }
        }
      }
    } else {
      float2 p[SLOTS];
      float mx = RUN ? run_m[0] : kLowest;
#pragma unroll
      for (int c = 0; c < SLOTS; ++c) {
        p[c] = lp[c * BM + tid];
        mx = fmaxf(mx, p[c].x);
      }
      float sum = RUN ? run_s[0] * exp2f((run_m[0] - mx) * kLog2e) : 0.f;
#pragma unroll
      for (int c = 0; c < SLOTS; ++c) sum += p[c].y * exp2f((p[c].x - mx) * kLog2e);
      run_m[0] = mx;
      run_s[0] = sum;
    }
  }
  if (!RUN || n0 >= n_stop) break;
  }
  if (tid < BM && m0 + tid < M) {
    float mx = run_m[0], sum = run_s[0];
    if constexpr (CHAINS > 1) {
#pragma unroll
      for (int w = 0; w < CHAINS; ++w) mx = fmaxf(mx, run_m[w]);
      sum = 0.f;
#pragma unroll
      for (int w = 0; w < CHAINS; ++w) sum += run_s[w] * exp2f((run_m[w] - mx) * kLog2e);
    }
    a.partials[(size_t)(m0 + tid) * a.nT + nt] = make_float2(mx, sum);
  }
}

template <int NR, int WN, Form F>
hipError_t launch_form(const HeadArgs& a, int m_tiles) {
  const dim3 grid((unsigned)(8L * ((a.nT + 7) / 8) * m_tiles)), block(128 * WN);
  if (WN == 4 && streams_w(a.V, a.d, 2, m_tiles, F == kLossTiles)) {
    FEF_LAUNCH_HEAD((head_tiled256_kernel<NR, WN, F, WN == 4>), grid, block, a, a, m_tiles);
  } else {
    FEF_LAUNCH_HEAD((head_tiled256_kernel<NR, WN, F, false>), grid, block, a, a, m_tiles);
  }
  return hipGetLastError();
}

// One instantiation per height: 32 to 256 rows with eight wavefronts (runs: to 128), 96 to 256 with four.
template <int WN, Form F>
hipError_t launch_rows(const HeadArgs& a, int m_tiles) {
  constexpr int most = F == kRuns64 || F == kRuns16 ? 4 : 8;
  const int nr = ((a.nrows + m_tiles - 1) / m_tiles + 31) / 32;
  if constexpr (WN == 4) {
    if (nr == 1) return launch_form<1, WN, F>(a, m_tiles);
    if (nr == 2) return launch_form<2, WN, F>(a, m_tiles);
  }
  if (nr == 3) return launch_form<3, WN, F>(a, m_tiles);
  if (nr == 4) return launch_form<4, WN, F>(a, m_tiles);
  if constexpr (most == 8) {
    if (nr == 5) return launch_form<5, WN, F>(a, m_tiles);
    if (nr == 6) return launch_form<6, WN, F>(a, m_tiles);
    if (nr == 7) return launch_form<7, WN, F>(a, m_tiles);
    if (nr == 8) return launch_form<8, WN, F>(a, m_tiles);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Cross-entropy: token tiles of a launch over M rows = partials per row.  With one row tile the pass over W is what it costs,
// and workgroups of whole 256-token tiles leave many CUs without work in the last round of 256: V = 100003 is 391 tiles,
// one round and a half, V = 151936 is 594, two and a third, V = 32000 is 125, half a round.  There the tokens are dealt
// out evenly over full rounds instead, in units of 32: per call 121 -> 109 us at 110 rows (d = 2560, V = 100003), 233 -> 205
// at 128 rows (d = 3584, V = 151936), 50.5 -> 46.3 at 64 rows (d = 4096, V = 32000), level at 256 rows.  Where the last round
// is nearly full (V = 126464: 494 tiles, 238 in the last round) whole tiles are 2 % ahead; hence the line at 200 of 256.
// (Some more than 256 rows: loss_wide_serves.)
// With several row tiles the multiplies are what it costs, and those of a partly filled tile are not saved.  (A verify
// step's tiles and runs are fixed by the order of its sums.)
int tiled256_tiles(int V, int M) {
  if (loss_wide_serves(M, V)) return 256;
  const int whole = (V + BN - 1) / BN;
  const int rounds = (whole + 255) / 256, last = whole - 256 * (rounds - 1);
  if (M > BN || last > 200) return whole;
  const int units = (V + kTiled256Unit - 1) / kTiled256Unit;
  return 256 * rounds < units ? 256 * rounds : units;
}

// Up to 256 rows: eight wavefronts (two per SIMD: the kernel is short of memory parallelism there, not of LDS rate).  More: four, or
// eight in a cross-entropy call where they are ahead (loss_takes_eight_wavefronts).  In a verify step a partial there spans 128
// tokens, which only four wavefronts hold in one: eight would save 7 % at 512 rows of d = 512.
hipError_t launch_head_tiled256(const HeadArgs& a) {
  if (a.labels && a.nT == 256 && loss_wide_serves(a.nrows, a.V)) return launch_head_loss_wide(a);
  const int m_tiles = (a.nrows + 255) / 256;
  // A launch of 2^32 threads or more runs only in part, without an error.  A cross-entropy call, whose logits need no
  // memory, gets there within its documented rows (2^22 rows of V = 131072): several launches then.
  const long most = ((1L << 32) - 1) / (8L * ((a.nT + 7) / 8) * 512);  // row tiles per launch
  if (m_tiles > most && most > 0) {
    const int rows = (int)most * 256;
    for (int r = 0; r < a.nrows; r += rows) {
      HeadArgs part = a;
      part.row0 += r;
      part.nrows = a.nrows - r < rows ? a.nrows - r : rows;
      if (a.logits) part.logits += (size_t)r * a.ldl;
      part.partials += (size_t)r * a.nT;
      if (a.labels) {
        part.labels += r;
        part.label_logit += r;
      }
      part.ev_begin = r == 0 ? a.ev_begin : nullptr;
      part.ev_end = r + rows >= a.nrows ? a.ev_end : nullptr;
      const hipError_t e = launch_head_tiled256(part);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  if (a.labels && m_tiles == 1 && a.nT != (a.V + BN - 1) / BN) return launch_rows<4, kLossShares>(a, 1);
  if (m_tiles == 1) {
    const int m = row_tiles(a.nrows, a.nT, a.d, 64, 256);
    return a.labels ? launch_rows<4, kLossTiles>(a, m) : launch_rows<4, kTiles>(a, m);
  }
  const int m = row_tiles(a.nrows, a.nT, a.d, 96, 256);
  if (!a.labels) return launch_rows<2, kTiles>(a, m);
  return loss_takes_eight_wavefronts(a.nrows, m, a.d) ? launch_rows<4, kLossTiles>(a, m) : launch_rows<2, kLossTiles>(a, m);
}

// Workgroups of a launch of runs = partials per row: one per CU, fewer where the vocabulary is short.  The first stages of a
// workgroup's next tile are requested before the epilogue of the one in work.
int runs_grid(int V, int unit) {
  const int units = (V + unit - 1) / unit, per = unit == 64 ? 4 : 8;
  const int want = (units + per - 1) / per;
  return want < 256 ? want : 256;
}
hipError_t launch_head_runs(const HeadArgs& a, int unit) {
  const int m = row_tiles(a.nrows, a.nT, a.d, 64, 128);
  const long units = (a.V + unit - 1) / unit, longest = (units + a.nT - 1) / a.nT * unit;
  if (short_runs_serve(unit, longest, a.d) && !short_runs_lag(a.nrows, a.nT, a.d)) return launch_head_short_runs(a, m);
  if (double_runs_serve((a.nrows + m - 1) / m, longest, a.d)) return launch_head_double_runs(a, unit, m);
  return unit == 64 ? launch_rows<4, kRuns64>(a, m) : launch_rows<4, kRuns16>(a, m);
}

}  // namespace fef
