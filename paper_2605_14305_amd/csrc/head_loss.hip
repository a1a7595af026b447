// Vocabulary-head kernel of a cross-entropy call of 257 to 320 rows over a vocabulary that one round of workgroups covers: all rows in one
// row tile, an equal share of the tokens per CU.
//
// What bounds it: multiplies and the operands on their way.  In two row tiles of 160 rows and whole tiles of 256 tokens 300 rows of V = 50257
// were 394 workgroups, two rounds for 1.54, and a CU took in (160 + 256) rows of operands twice; here it takes (300 + 197) once.
// 300 rows of d = 2048, V = 50257: head 77.8 -> 68.4 us (0.9 PFLOP/s), 59.8 with W in the Infinity Cache; a k-step takes 2 us, 1.3 of them
// multiplies.  The fragments of a half step read under the multiplies of the one before: 71 -> 68 us.  Relative error against 64 bits, inputs of the
// performance cases, twelve seeds each, two row tiles -> one: 300 rows of d = 2048, V = 50257 2.49e-7 -> 2.37e-7, 290 of d = 4096, V = 47000
// 3.38e-7 -> 3.43e-7, 270 of d = 1024, V = 55000 1.90e-7 -> 1.88e-7; over seven sizes of random labels 5.80e-8 -> 5.80e-8 in the mean.
// W by ordinary loads at every size: non-temporal ones, which two row tiles want from 288 MiB on, are 1 to 9 % slower here (300 rows of d = 4096,
// V = 50257 121.7 -> 129.7 us per call, of d = 8192 235.6 -> 254.2, of d = 3072 92.4 -> 96.7; with one W the same).
//
// Eight wavefronts, 4 x 2, each 80 rows x 16 NT tokens; k-steps of 64 columns; W is requested two steps ahead, H one (it comes from L2).
// 304 rows of H and 224 tokens of W fill LDS to the byte; the 16 rows behind them are multiplied as whatever lies there and never used.
#include <type_traits>

#include "head_common.hpp"

namespace fef {
namespace {

constexpr int BK = 64, kThreads = 512, WM = 4, WN = 2, NR = 5, BM = 16 * NR * WM;
constexpr int kUnit = 16;  // tokens; shares are equal to a unit
constexpr float kLog2e = 1.4426950408889634f;

// ROWS: rows of H in LDS.
template <int NT, int ROWS>
__global__ __launch_bounds__(kThreads) void head_loss_wide_kernel(HeadArgs a) {
  constexpr int TOK = 16 * NT * WN, RW = 3, RH = 2;
  constexpr int kLoadsH = ROWS / 8, kLoadsW = TOK / 8, LH = 5, LW = 4;  // load instructions of eight rows: of a stage, per wavefront
  static_assert(8 * LH >= kLoadsH && 8 * LW >= kLoadsW && kLoadsH >= LH && kLoadsW >= LW, "");
  constexpr int kStageH = ROWS * 8, kStageW = TOK * 8;  // 16-byte chunks
  __shared__ bf16x8 ring[RH * kStageH + RW * kStageW];
  bf16x8* const ringH = ring;
  bf16x8* const ringW = ring + RH * kStageH;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int i16 = lane & 15, g = lane >> 4;
  const int M = a.nrows, nk = a.d / BK, nt = blockIdx.x;

  const int units = (a.V + kUnit - 1) / kUnit;
  const int share0 = (int)((long)nt * units / a.nT) * kUnit, share1 = min(a.V, (int)((long)(nt + 1) * units / a.nT) * kUnit);
  const int half = ((share1 - share0 + 1) / 2 + 15) / 16 * 16;  // tokens of the first column of wavefronts
  const int k0 = (int)((unsigned)(nt * 37) % (unsigned)nk);     // every share starts its walk over k elsewhere

  // Lane l owns LDS slot (row l / 8, position l % 8) of eight rows; chunk c of row r is kept at position c ^ (r / 2 % 8).  Every wavefront
  // issues as many loads as the others (the waits count them); the last ones repeat some.
  const int hi0 = min(wave * LH, kLoadsH - LH), wi0 = min(wave * LW, kLoadsW - LW);
  const __bf16* gh[LH];
  const __bf16* gw[LW];
#pragma unroll
  for (int q = 0; q < LH; ++q) {
    const int rl = (hi0 + q) * 8 + (lane >> 3);
    gh[q] = h_row(a, min(rl, M - 1)) + ((lane & 7) ^ ((rl >> 1) & 7)) * 8 + k0 * BK - q % 4 * 512;  // rows past M: the last, masked later
  }
#pragma unroll
  for (int q = 0; q < LW; ++q) {
    const int rl = (wi0 + q) * 8 + (lane >> 3);
    // rows 16 NT .. of a stage are the second column's tokens, which begin `half` behind the first's
    const int v = rl < 16 * NT ? min(share0 + rl, share0 + half - 1) : share0 + half + rl - 16 * NT;
    gw[q] = (const __bf16*)a.W + (size_t)min(v, share1 - 1) * a.d + ((lane & 7) ^ ((rl >> 1) & 7)) * 8 + k0 * BK - q * 512;
  }
  int h_left = nk - k0, w_left = nk - k0;  // steps until the walk is back at k = 0
  const uint32_t slotH = lds_offset(ringH + hi0 * 64), slotW = lds_offset(ringW + wi0 * 64);
  auto advance = [&](int& left) __attribute__((always_inline)) -> long { return --left == 0 ? (long)BK - a.d : (long)BK; };
  auto load_h = [&](int stage) __attribute__((always_inline)) {
    const __bf16* const four[4] = {gh[0], gh[1], gh[2], gh[3]};
    load_group_to_lds<false>(four, __builtin_amdgcn_readfirstlane(slotH + stage * kStageH * 16));
    load_to_lds_16(gh[4], __builtin_amdgcn_readfirstlane(slotH + stage * kStageH * 16 + 4096));
    const long move = advance(h_left);
#pragma unroll
    for (int q = 0; q < LH; ++q) gh[q] += move;
  };
  auto load_w = [&](int stage) __attribute__((always_inline)) {
    load_group_to_lds<false>(gw, __builtin_amdgcn_readfirstlane(slotW + stage * kStageW * 16));
    const long move = advance(w_left);
#pragma unroll
    for (int q = 0; q < LW; ++q) gw[q] += move;
  };
  load_w(0);
  load_h(0);
  if (nk > 1) load_w(1);

  floatx4 acc[NR][NT];  // acc[n][t]: tokens 16 t + 4 g .. + 3 of row 16 n + i16 of the wavefront's tile
#pragma unroll
  for (int n = 0; n < NR; ++n)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[n][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  int fo[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) fo[ks] = i16 * 8 + ((ks * 4 + g) ^ ((i16 >> 1) & 7));

  // A step's two halves of k: the fragments of one are read under the multiplies of the one before, the second half of a step is
  // multiplied behind the next step's barrier.
  bf16x8 wf[2][NT], hf[NR];
  auto phase = [&](auto ks_tag, auto mul_tag, const bf16x8* Hs, const bf16x8* Ws) __attribute__((always_inline)) {
    constexpr int KS = decltype(ks_tag)::value;
#pragma unroll
    for (int n = 0; n < NR; ++n) {
      if constexpr (decltype(mul_tag)::value)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[n][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[KS ^ 1][t], hf[n], acc[n][t], 0, 0, 0);
      hf[n] = Hs[n * 128 + fo[KS]];
#pragma unroll
      for (int t = n * NT / NR; t < (n + 1) * NT / NR; ++t) wf[KS][t] = Ws[t * 128 + fo[KS]];
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using First = std::integral_constant<int, 0>;
  using Second = std::integral_constant<int, 1>;
  int sw = 0;
  for (int k = 0; k < nk; ++k) {
    if (k + 1 < nk) wait_newer<LW>();  // W(k + 1) may stay on its way
    else wait_newer<0>();
    lds_barrier();
    if (k + 1 < nk) load_h((k + 1) & 1);
    if (k + 2 < nk) load_w(sw == 0 ? RW - 1 : sw - 1);
    const bf16x8* Hs = ringH + (k & 1) * kStageH + wm * NR * 128;
    const bf16x8* Ws = ringW + sw * kStageW + wn * NT * 128;
    if (k) phase(First{}, std::true_type{}, Hs, Ws);
    else phase(First{}, std::false_type{}, Hs, Ws);
    phase(Second{}, std::true_type{}, Hs, Ws);
    sw = sw == RW - 1 ? 0 : sw + 1;
  }
#pragma unroll
  for (int n = 0; n < NR; ++n)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[n][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[1][t], hf[n], acc[n][t], 0, 0, 0);
  lds_barrier();  // nobody reads the rings any more

  // Epilogue: nothing crosses lanes but the label's logit; the partial of each lane's own tokens goes to LDS, [slot][row].
  constexpr int kSlots = 4 * WN;  // 8
  static_assert((kSlots * BM * 8 + kThreads * NT * 16) <= (int)sizeof(ring), "");
  float2* part = reinterpret_cast<float2*>(ring);
  floatx4* own = reinterpret_cast<floatx4*>(part + kSlots * BM) + wave * (NT * kWave) + lane;
  const int vw = share0 + wn * half, v_end = wn == 0 ? min(share0 + half, share1) : share1, v0 = vw + 4 * g;
  const float sc = a.inv_tau;
#pragma unroll
  for (int n = 0; n < NR; ++n) {
    const int row = (wm * NR + n) * 16 + i16;
    floatx4 l[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) l[t] = acc[n][t] * sc;
    const int off = row < M ? a.labels[row] - vw : -1;
    const bool mine = (unsigned)off < (unsigned)(16 * NT) && ((off >> 2) & 3) == g && vw + off < v_end;
    if (__builtin_amdgcn_ballot_w64(mine) != 0) {  // wavefront-uniform
#pragma unroll
      for (int t = 0; t < NT; ++t) own[t * kWave] = l[t];
      if (mine) a.label_logit[row] = reinterpret_cast<const float*>(own + (off >> 4) * kWave)[off & 3];
    }
    float mx = kLowest;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (v0 + 16 * t + c >= v_end) l[t][c] = -INFINITY;
      mx = vmax3(vmax3(l[t][0], l[t][1], mx), l[t][2], l[t][3]);
    }
    const float mb = mx * -kLog2e;
    float e[8] = {};  // summed as trees, here and below: a chain over the tiles is 2 to 4 % further from the sum in 64 bits
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
      for (int c = 0; c < 4; ++c) l[t][c] = __builtin_amdgcn_exp2f(fmaf(l[t][c], kLog2e, mb));
      e[t] = (l[t][0] + l[t][1]) + (l[t][2] + l[t][3]);
    }
    part[(4 * wn + g) * BM + row] = make_float2(mx, ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7])));
  }
  lds_barrier();
  if (tid < M) {
    float2 p[kSlots];
    float mx = kLowest;
#pragma unroll
    for (int c = 0; c < kSlots; ++c) {
      p[c] = part[c * BM + tid];
      mx = fmaxf(mx, p[c].x);
    }
#pragma unroll
    for (int c = 0; c < kSlots; ++c) p[c].y *= exp2f((p[c].x - mx) * kLog2e);
    const float sum = ((p[0].y + p[1].y) + (p[2].y + p[3].y)) + ((p[4].y + p[5].y) + (p[6].y + p[7].y));
    a.partials[(size_t)tid * a.nT + nt] = make_float2(mx, sum);
  }
}

}  // namespace

// Shares of up to 192 tokens: 320 rows; of up to 224: 304.
hipError_t launch_head_loss_wide(const HeadArgs& a) {
  if ((a.V + 15) / 16 <= 192 / 16 * a.nT) {
    FEF_LAUNCH_HEAD((head_loss_wide_kernel<6, 320>), dim3(a.nT), dim3(kThreads), a, a);
  } else {
    FEF_LAUNCH_HEAD((head_loss_wide_kernel<7, 304>), dim3(a.nT), dim3(kThreads), a, a);
  }
  return hipGetLastError();
}

}  // namespace fef
