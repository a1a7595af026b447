// Vocabulary-head kernel for up to 128 rows whose workgroups walk k once over all their tokens.  It gives bit for bit what the runs of
// head_tiled256_kernel give, one tile of up to 256 tokens after another, and takes their place where those leave the CUs too little of W
// on its way: runs of up to 128 tokens, and many of 257 to 512 (short_runs_serve, double_runs_serve, with both sides measured).
// And where the runs, or up to 256 rows' tiles of 256 tokens, are too few for the CUs: a piece of one per workgroup, without partials
// (pieces_pay, piece_shape).
//
// What bounds it: the pass over W, at 4.8 to 5.3 TB/s with 110 rows of V = 100003 (4.5 to 4.8 in tiles), and for short vocabularies what
// a CU can have on its way at once: 63 workgroups of 128 tokens (V = 8000, d = 4096) get 33 KB of W each per us whether four,
// five, six or seven stages are requested ahead, k-steps of 128 columns are level, and so are fragments read in front of the
// loads' issue.
#include <type_traits>
#include <utility>

#include "head_common.hpp"
#include "head_swaps.hpp"

namespace fef {
namespace {

constexpr int BK = 64, kThreads = 512;  // columns of a k-step: 128 bytes, one line
constexpr int kLds = 160 * 1024;
constexpr float kLog2e = 1.4426950408889634f;

// Order of the sums, as in head_gemm_tiled256.hip: STREAM, ROWSTREAM, TILED256 (a run is a tile of 256 tokens).
enum Form { kRuns64, kRuns16, kTiles };
constexpr int form_unit(Form f) { return f == kRuns16 ? 16 : 64; }

template <class F, int... I>
__device__ __forceinline__ void for_each(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// Stages of W (one per k-step and piece of TOK tokens) and of H (one per k-step): W is requested rw - 1 steps ahead, H rh - 1 k-steps,
// which has to be as early as the W that its step asks for together with it.
struct Rings {
  int rw, rh;
};
constexpr Rings rings(int rows, int tok, int pieces) {
  Rings best{0, 0};
  for (int rh = 2; rh <= 8; ++rh) {
    int rw = (kLds - rh * rows * BK * 2) / (tok * BK * 2);
    if (rw > (rh - 1) * pieces + 2) rw = (rh - 1) * pieces + 2;
    if (rw > best.rw) best = Rings{rw, rh};
  }
  return best;
}

// A workgroup's tokens in NS pieces of up to TOK, walked side by side: at every k-step one piece after another.  Eight wavefronts, WM x 8 / WM,
// each 16 NR rows x 16 NT tokens of a piece.
// PIECES: the run is cut into `pieces` parts, a workgroup each, and partials are left to the next kernel (row_sums_draft_kernel).
template <int WM, int NR, int TOK, int NS, Form F, bool PIECES, bool STREAM_W>
__global__ __launch_bounds__(kThreads) void head_runs_kernel(HeadArgs a, int m_tiles, int pieces) {
  static_assert(PIECES ? NS == 1 : F != kTiles, "");
  constexpr int WN = 8 / WM, NT = TOK / (16 * WN), BM = 16 * NR * WM, WROWS = 16 * NR;
  static_assert(NT >= 2 && (PIECES || F != kRuns64 || NT == 4), "a partial in one wavefront");
  constexpr int LW = TOK / 64, LH = (2 * NR * WM + 7) / 8;  // loads per wavefront and stage, of eight rows each
  constexpr Rings R = rings(BM, TOK, NS);
  constexpr int RW = R.rw, RH = R.rh;
  static_assert(RW >= 3 && RH >= 2 && (RH - 1) * NS >= RW - 2, "H comes no later than the W it is multiplied with");
  constexpr int kStageH = BM * 8, kStageW = TOK * 8;  // 16-byte chunks
  __shared__ bf16x8 ring[RH * kStageH + RW * kStageW];
  bf16x8* const ringH = ring;
  bf16x8* const ringW = ring + RH * kStageH;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int i16 = lane & 15, g = lane >> 4;
  const int M = a.nrows, nk = a.d / BK;

  // row tiles of one run follow one another on one XCD, which shares W through its L2
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int per_run = PIECES ? m_tiles * pieces : m_tiles;
  const int nt = xcd + 8 * (seq / per_run), m0 = seq % m_tiles * BM;
  if (nt >= a.nT) return;
  constexpr int UNIT = form_unit(F);
  const int n_units = (a.V + UNIT - 1) / UNIT;
  int unit0 = F == kTiles ? 4 * nt : (int)((long)nt * n_units / a.nT);
  int units = F == kTiles ? min(4, n_units - unit0) : (int)((long)(nt + 1) * n_units / a.nT) - unit0;
  if constexpr (PIECES) {
    const int p = seq % per_run / m_tiles, begin = units * p / pieces;
    units = units * (p + 1) / pieces - begin;
    unit0 += begin;
    if (units == 0) return;
  }
  const int run0 = unit0 * UNIT, run1 = min(a.V, (unit0 + units) * UNIT);
  auto piece_at = [&](int s) { return min(run1, run0 + (int)(units * s / NS) * UNIT); };

  // every run starts its walk over k elsewhere; of a start in the middle of a k-step, the step's first half comes last of all
  constexpr int kStart = F == kRuns64 ? 32 : F == kRuns16 ? 128 : BK;
  const int start = (int)((unsigned)(nt * 37) % (unsigned)(a.d / kStart)) * kStart;
  const bool half = F == kRuns64 && start % BK != 0;
  const int k0 = start / BK, nsteps = nk + (half ? 1 : 0), total = nsteps * NS;

  // Loads: lane l owns LDS slot (row l / 8, position l % 8) of eight rows; chunk c of row r is kept at position c ^ (r / 2 % 8), so
  // that fragment reads touch every bank once.  Every wavefront issues as many loads as the others (the waits count them).
  const int hrow0 = 8 * min(wave * LH, max(0, 2 * NR * WM - LH));
  const __bf16* gh[LH];
  const __bf16* gw[NS][LW];
  int h_left = nk - k0, w_left[NS];  // steps until the walk is back at k = 0
#pragma unroll
  for (int q = 0; q < LH; ++q) {
    const int rl = hrow0 + q * 8 + (lane >> 3);
    gh[q] = h_row(a, min(m0 + rl, M - 1)) + ((lane & 7) ^ ((rl >> 1) & 7)) * 8 + k0 * BK - q * 512;  // rows past M: the last, masked later
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    w_left[s] = nk - k0;
#pragma unroll
    for (int q = 0; q < LW; ++q) {
      const int rl = wave * (8 * LW) + q * 8 + (lane >> 3);
      const int row = max(0, min(piece_at(s) + rl, piece_at(s + 1) - 1));  // past the piece: its last row, masked later
      gw[s][q] = (const __bf16*)a.W + (size_t)row * a.d + ((lane & 7) ^ ((rl >> 1) & 7)) * 8 + k0 * BK - q * 512;
    }
  }
  const uint32_t slotH = lds_offset(ringH + hrow0 * 8), slotW = lds_offset(ringW + wave * LW * 64);
  constexpr uint32_t kBytesH = kStageH * 16, kBytesW = kStageW * 16;
  auto advance = [&](int& left) __attribute__((always_inline)) -> long { return --left == 0 ? (long)BK - a.d : (long)BK; };
  auto load_h = [&](int stage) __attribute__((always_inline)) {
    load_group_to_lds<false>(gh, __builtin_amdgcn_readfirstlane(slotH + stage * kBytesH));
    const long move = advance(h_left);
#pragma unroll
    for (int q = 0; q < LH; ++q) gh[q] += move;
  };
  auto load_w = [&](int s, int stage) __attribute__((always_inline)) {
    load_group_to_lds<STREAM_W>(gw[s], __builtin_amdgcn_readfirstlane(slotW + stage * kBytesW));
    const long move = advance(w_left[s]);
#pragma unroll
    for (int q = 0; q < LW; ++q) gw[s][q] += move;
  };
  // Step j = k NS + s multiplies W(j) and H(k).  It requests H(k + RH - 1) if s = 0, then W(j + RW - 1).  Here: what the steps
  // before the first would have requested, in that order.
  constexpr int kAhead = RW - 1 > (RH - 1) * NS ? RW - 1 : (RH - 1) * NS;
  for_each(std::make_integer_sequence<int, kAhead>{}, [&](auto i_tag) __attribute__((always_inline)) {
    constexpr int j = decltype(i_tag)::value - kAhead, h = j % NS == 0 ? j / NS + RH - 1 : -1, w = j + RW - 1;
    if constexpr (h >= 0) {
      if (h < nsteps) load_h(h % RH);
    }
    if constexpr (w >= 0) {
      if (w < total) load_w(w % NS, w % RW);
    }
  });

  floatx4 acc[NS][NT][NR];  // acc[s][t][n]: tokens 16 t + 4 g .. + 3 of row 16 n + i16 of the wavefront's part of piece s
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int n = 0; n < NR; ++n) acc[s][t][n] = floatx4{0.f, 0.f, 0.f, 0.f};
  int fo[2];  // chunk of this lane's fragment of k-half ks within 16 rows of a stage
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) fo[ks] = i16 * 8 + ((ks * 4 + g) ^ ((i16 >> 1) & 7));
  const bool rows_live = __builtin_amdgcn_readfirstlane((int)(m0 + wm * WROWS < M)) != 0;

  int sw = 0, sh = 0;
  for (int k = 0; k < nsteps; ++k) {
    bf16x8 hf[2][NR];
    for_each(std::make_integer_sequence<int, NS>{}, [&](auto s_tag) __attribute__((always_inline)) {
      constexpr int s = decltype(s_tag)::value;
      // loads that may stay in flight: those younger than W(j) and, in the first step of a k, than H(k)
      constexpr auto issued_since = [](int from) constexpr {  // in the steps j + from .. j - 1
        int n = 0;
        for (int i = from; i < 0; ++i) n += LW + ((s + i + 64 * NS) % NS == 0 ? LH : 0);
        return n;
      };
      constexpr int kW = issued_since(2 - RW), kH = s == 0 ? LW + issued_since(1 - (RH - 1) * NS) : kW;
      const int j = k * NS + s;
      if (j + RW - 2 < total && k + RH - 1 < nsteps) {
        wait_newer<(kW < kH ? kW : kH)>();
      } else {  // the last steps: no more than the W of the steps that are left
        const int rest = min(total - 1 - j, RW - 2);
        if (rest >= 4) wait_newer<(RW >= 6 ? 4 * LW : 0)>();
        else if (rest >= 2) wait_newer<(RW >= 4 ? 2 * LW : 0)>();
        else if (rest == 1) wait_newer<LW>();
        else wait_newer<0>();
      }
      lds_barrier();
      if (s == 0 && k + RH - 1 < nsteps) load_h(sh == 0 ? RH - 1 : sh - 1);
      if (j + RW - 1 < total) load_w((s + RW - 1) % NS, sw == 0 ? RW - 1 : sw - 1);
      if (rows_live) {
        const bf16x8* Ws = ringW + sw * kStageW + wn * NT * 128;
        if constexpr (s == 0)
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int n = 0; n < NR; ++n) hf[ks][n] = ringH[sh * kStageH + (wm * NR + n) * 128 + fo[ks]];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          if (F == kRuns64 && half && k == (ks ? nsteps - 1 : 0)) continue;
          bf16x8 wf[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) wf[t] = Ws[t * 128 + fo[ks]];
#pragma unroll
          for (int n = 0; n < NR; ++n)
#pragma unroll
            for (int t = 0; t < NT; ++t)
              acc[s][t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[t], hf[ks][n], acc[s][t][n], 0, 0, 0);
        }
      }
      sw = sw == RW - 1 ? 0 : sw + 1;
    });
    sh = sh == RH - 1 ? 0 : sh + 1;
  }
  lds_barrier();  // nobody reads the rings any more

  // Epilogue: partials of all pieces in the place of the rings, [slot][row].
  constexpr int kSlots = F == kRuns64 ? TOK / 64 : TOK / 16;  // of a piece
  static_assert(NS * kSlots * BM * sizeof(float2) <= sizeof(ring), "");
  float2* part = reinterpret_cast<float2*>(ring);
  const float sc = a.inv_tau;
  for_each(std::make_integer_sequence<int, NS>{}, [&](auto s_tag) __attribute__((always_inline)) {
    constexpr int s = decltype(s_tag)::value;
    const int p_end = piece_at(s + 1), vw = piece_at(s) + wn * (16 * NT), v0 = vw + 4 * g;
    // slot of the wavefront's first partial; the units of 64 are counted from the start of the run, whatever piece they are in
    const int slot = F == kRuns64 ? (piece_at(s) - run0) / 64 + wn : s * kSlots + NT * wn;
    if (rows_live && vw < p_end) {
      auto rows = [&](auto edge) __attribute__((always_inline)) {
        constexpr bool EDGE = decltype(edge)::value;  // some of the wavefront's tokens do not exist
#pragma unroll
        for (int n = 0; n < NR; ++n) {
          const int rl = wm * WROWS + 16 * n + i16, row = m0 + rl;
          floatx4 l[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) l[t] = acc[s][t][n] * sc;
          // Neighbouring lanes (rows 2j, 2j + 1) trade one of every two 16-token tiles, so that a store instruction writes 128 bytes
          // of a row; non-temporal, past the W and H lines in L2.
          const bool odd = i16 & 1;
          const int row2 = row & ~1;
          const int pairs = EDGE ? (p_end - vw) / 32 : NT / 2;  // whole pairs of tiles, wavefront-uniform
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
          if constexpr (EDGE) {  // what does not fill a pair
            float* one = a.logits + (size_t)row * a.ldl + v0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              if (t / 2 < pairs || vw + 16 * t >= p_end || row >= M) continue;
              if (v0 + 16 * t + 3 < p_end) {
                __builtin_nontemporal_store(l[t], reinterpret_cast<floatx4*>(one + 16 * t));
              } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                  if (v0 + 16 * t + c < p_end) one[16 * t + c] = l[t][c];
              }
            }
          }
          if constexpr (PIECES) continue;
          if constexpr (EDGE)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if (v0 + 16 * t + c >= p_end) l[t][c] = -INFINITY;
          auto max_of = [&](float mx, int t) __attribute__((always_inline)) -> float {
            return vmax3(vmax3(l[t][0], l[t][1], mx), l[t][2], l[t][3]);
          };
          // l[t] becomes exp(l[t] - mx)
          auto exps = [&](int t, float mx) __attribute__((always_inline)) {
            const float mb = mx * -kLog2e;
#pragma unroll
            for (int c = 0; c < 4; ++c) l[t][c] = __builtin_amdgcn_exp2f(fmaf(l[t][c], kLog2e, mb));
          };
          if constexpr (F == kRuns16) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              float m = max_of(kLowest, t), o = m;
              swap_quarters(m, o);
              m = o = vmax(m, o);
              swap_halves(m, o);
              m = vmax(m, o);
              exps(t, m);
              float e = ((l[t][0] + l[t][1]) + l[t][2]) + l[t][3];
              o = e;
              swap_quarters(e, o);
              e = o = e + o;
              swap_halves(e, o);
              if (g == 0) part[(slot + t) * BM + rl] = make_float2(m, e + o);
            }
          } else if constexpr (F == kRuns64) {
            float mx = kLowest;
#pragma unroll
            for (int t = 0; t < 4; ++t) mx = max_of(mx, t);
            float o = mx;
            group_max(mx, o);
            float e0[4], e1[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) exps(t, mx);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              e0[c] = l[0][c] + l[2][c];
              e1[c] = l[1][c] + l[3][c];
            }
            float x = group_sum(e0, e1), y = x;
            swap_halves(x, y);
            if (g == 0) part[slot * BM + rl] = make_float2(mx, x + y);
          }
        }
      };
      if (vw + 16 * NT <= p_end) rows(std::false_type{});
      else rows(std::true_type{});
    }
  });
  if constexpr (PIECES) return;
  lds_barrier();
  // One (max, sum exp) partial per (row, run), merged in a fixed order by the thread that owns the row.
  if (tid < BM && m0 + tid < M) {
    float mx = -INFINITY, sum = 0.f;
    if constexpr (F == kRuns64) {  // four units at a time, counted from the start of the run
      for (int u = 0; u < units; u += 4) {
        float2 p[4];
        const float before = mx;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          p[c] = u + c < units ? part[(u + c) * BM + tid] : make_float2(kLowest, 0.f);
          mx = fmaxf(mx, p[c].x);
        }
        sum *= exp2f((before - mx) * kLog2e);
#pragma unroll
        for (int c = 0; c < 4; ++c) sum += p[c].y * exp2f((p[c].x - mx) * kLog2e);
      }
    } else {  // eight chains, every eighth 16-token tile of the run each
      float run_m[8], run_s[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        run_m[c] = -INFINITY;
        run_s[c] = 0.f;
      }
      for (int u = 0; u < units; u += 8)
#pragma unroll
        for (int c = 0; c < 8; ++c)
          if (u + c < units) {
            const int first = NS == 1 ? 0 : units / NS;  // units of the first piece
            const int at = u + c < first || NS == 1 ? u + c : kSlots + u + c - first;
            const float2 p = part[at * BM + tid];
            if (p.x > run_m[c]) {
              run_s[c] = run_s[c] * exp2f((run_m[c] - p.x) * kLog2e) + p.y;
              run_m[c] = p.x;
            } else {
              run_s[c] += p.y * exp2f((p.x - run_m[c]) * kLog2e);
            }
          }
      mx = run_m[0];
#pragma unroll
      for (int c = 0; c < 8; ++c) mx = fmaxf(mx, run_m[c]);
#pragma unroll
      for (int c = 0; c < 8; ++c) sum += run_s[c] * exp2f((run_m[c] - mx) * kLog2e);
    }
    a.partials[(size_t)(m0 + tid) * a.nT + nt] = make_float2(mx, sum);
  }
}

template <int WM, int NR, int TOK, int NS, Form F, bool PIECES = false>
hipError_t launch_form(const HeadArgs& a, int m_tiles, int pieces = 1) {
  const dim3 grid((unsigned)(8L * ((a.nT + 7) / 8) * m_tiles * pieces)), block(kThreads);
  if (!PIECES && streams_w(a.V, a.d, 2, m_tiles, false)) {
    FEF_LAUNCH_HEAD((head_runs_kernel<WM, NR, TOK, NS, F, PIECES, !PIECES>), grid, block, a, a, m_tiles, pieces);
  } else {
    FEF_LAUNCH_HEAD((head_runs_kernel<WM, NR, TOK, NS, F, PIECES, false>), grid, block, a, a, m_tiles, pieces);
  }
  return hipGetLastError();
}

// Runs of up to 128 tokens; of 257 to 512.
template <Form F>
hipError_t launch_short(const HeadArgs& a, int m) {
  const int nr = ((a.nrows + m - 1) / m + 31) / 32;
  return nr == 1 ? launch_form<2, 1, 128, 1, F>(a, m) : nr == 2 ? launch_form<4, 1, 128, 1, F>(a, m)
       : nr == 3 ? launch_form<2, 3, 128, 1, F>(a, m) : launch_form<4, 2, 128, 1, F>(a, m);
}
template <Form F>
hipError_t launch_double(const HeadArgs& a, int m) {
  const int nr = ((a.nrows + m - 1) / m + 31) / 32;
  return nr == 1 ? launch_form<2, 1, 256, 2, F>(a, m) : nr == 2 ? launch_form<2, 2, 256, 2, F>(a, m)
       : nr == 3 ? launch_form<2, 3, 256, 2, F>(a, m) : launch_form<2, 4, 256, 2, F>(a, m);
}
// Pieces of up to 64 tokens, of whole tiles also 128 (up to 128 rows piece_shape gives 64 everywhere), row tiles of 64 or 128 rows.
template <Form F>
hipError_t launch_pieces(const HeadArgs& a, const PieceShape& p) {
  if (p.tokens == 64)
    return p.rows == 64 ? launch_form<4, 1, 64, 1, F, true>(a, p.row_tiles, p.pieces) : launch_form<4, 2, 64, 1, F, true>(a, p.row_tiles, p.pieces);
  if constexpr (F == kTiles)
    return p.rows == 64 ? launch_form<4, 1, 128, 1, F, true>(a, p.row_tiles, p.pieces) : launch_form<4, 2, 128, 1, F, true>(a, p.row_tiles, p.pieces);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_head_short_runs(const HeadArgs& a, int row_tiles) { return launch_short<kRuns16>(a, row_tiles); }
hipError_t launch_head_double_runs(const HeadArgs& a, int unit, int row_tiles) {
  return unit == 64 ? launch_double<kRuns64>(a, row_tiles) : launch_double<kRuns16>(a, row_tiles);
}
hipError_t launch_head_pieces(const HeadArgs& a, int unit, const PieceShape& p) {
  return unit == 64 ? launch_pieces<kRuns64>(a, p) : unit == 16 ? launch_pieces<kRuns16>(a, p) : launch_pieces<kTiles>(a, p);
}

}  // namespace fef
