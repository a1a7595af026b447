// Vocabulary-head kernel for up to 32 rows and a long vocabulary.  It gives bit for bit what head_skinny_kernel gives (the SKINNY
// variant's order of sums) and takes its place where a workgroup's run of tokens is longer than 128 (slices_serve; slices_lag: exceptions).
//
// The order of the sums.  A logit is eight sums over d / 8 columns each (the slices), each ascending from zero, added in the
// order of the slices; a workgroup's tokens are a contiguous run of 16-token tiles; a tile's (max, sum exp) adds four
// neighbouring tokens in order and then the four groups pairwise; the tiles of a run are merged in four chains, every fourth tile each.
//
// What bounds it: the pass over W.  head_skinny_kernel keeps H in registers, eight wavefronts take a slice each and W goes
// straight to registers, 16 rows x 64 bytes a load; as much of W is on its way as a tile has bytes, which is little at hidden
// sizes below 4096, and all logits leave at the end.  Here the workgroup walks k over up to 256 tokens, W and H go to LDS three
// and two k-steps ahead, and the stages of the next tile are requested in front of the epilogue.  (Whole 128-byte lines in the
// loads of head_skinny_kernel, by trading halves between lanes, measured nothing.)  Head alone, us, head_skinny_kernel -> this
// kernel, W in non-temporal loads from 288 MiB on as elsewhere, 16 and 32 rows:
//   d, V           16 rows         32 rows          d, V           16 rows         32 rows
//   512, 50257     16.7 -> 14.3    19.5 -> 15.8     3072, 126464   136 -> 123      142 -> 127
//   512, 151936    37.1 -> 35.6    47.9 -> 39.5     3584, 50257    67.7 -> 59.4    70.8 -> 60.7
//   2048, 50257    43.9 -> 40.8    43.7 -> 42.6     3584, 151936   188 -> 169      192 -> 172
//   2048, 126464   90.8 -> 85.3    93.7 -> 89.9     4096, 50257    73.3 -> 70.1    76.5 -> 72.3
//   2560, 100003   94.5 -> 89.2    97.9 -> 92.5     4096, 126464   171 -> 166      175 -> 168
//   3072, 50257    65.1 -> 55.3    67.3 -> 55.1     4096, 151936   204 -> 198      208 -> 202
//
// Where the walk starts.  Rows of 4 or 8 KB put the same column of all rows on few memory channels, and workgroups that
// walk k in step then wait for those: 32 rows of d = 4096, V = 126464 186 us, of d = 2048, V = 126464 102.  So at these hidden
// sizes (ROTATE) a workgroup starts with a slice of its own, and since the slices are added in order from the first, their
// sums wait in registers.  Neighbours on an XCD start apart (169 and 91 us); one start per XCD is 3 % behind.  At the other hidden sizes
// everybody starts at the first slice and adds as it goes, which saves the registers and 1 to 6 %.
#include <type_traits>

#include "head_common.hpp"
#include "head_swaps.hpp"

namespace fef {
namespace {

constexpr int BK = 64, kTile = 256;  // columns of a k-step: 128 bytes, one line; tokens of a tile, at most
constexpr int kThreads = 512, kSlices = 8, kChains = 4;

// WM: groups of 16 rows.  Eight wavefronts, WM x 8 / WM, each 16 rows x 32 WM tokens.
template <int WM, bool ROTATE, bool STREAM_W>
__global__ __launch_bounds__(kThreads) void head_slices_kernel(HeadArgs a, int tiles_total) {
  constexpr int WN = 8 / WM, NT = kTile / (16 * WN), BM = 16 * WM;
  constexpr int LW = 4;                                 // loads of W per wavefront and step, of eight rows each; one of H
  constexpr int RW = 4, RH = 3;                         // stages in LDS: W is requested three steps ahead, H two
  constexpr int kStageH = BM * 8, kStageW = kTile * 8;  // 16-byte chunks
  __shared__ bf16x8 ringH[RH * kStageH];
  __shared__ bf16x8 ringW[RW * kStageW];
  __shared__ float2 part[kTile / 16][BM];               // (max, sum exp) of each 16-token tile and row
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int i16 = lane & 15, g = lane >> 4;
  const int M = a.nrows, nk = a.d / BK;

  // 16-token tiles [run0, run1) of this workgroup, taken up to 256 tokens at a time in tiles as equal as they can be
  const int run0 = (int)((long)blockIdx.x * tiles_total / gridDim.x), run1 = (int)((long)(blockIdx.x + 1) * tiles_total / gridDim.x);
  const int tiles = (run1 - run0 + kTile / 16 - 1) / (kTile / 16);
  auto tile_begin = [&](int i) { return run0 + (int)((long)i * (run1 - run0) / tiles); };
  const int slice0 = ROTATE ? (blockIdx.x >> 3) & (kSlices - 1) : 0;
  const int per_slice = nk / kSlices, k0 = slice0 * per_slice;

  // Loads: wavefront w fills rows [32 w, + 32) of a W stage and eight rows of an H stage (those beyond the last repeat it, since
  // every wavefront issues as many loads as the others: the waits count them).  Lane l owns LDS slot (row l / 8, position l % 8);
  // chunk c of row r is kept at position c ^ (r / 2 % 8) so that fragment reads touch every bank once.
  const int hrow0 = 8 * min(wave, 2 * WM - 1);
  const __bf16* gh;
  const __bf16* gw[LW];
  int h_left, w_left;  // steps until the walk is back at k = 0
  auto aim = [&](int begin, int end) __attribute__((always_inline)) {
    h_left = w_left = nk - k0;
    const int rh = hrow0 + (lane >> 3);
    gh = h_row(a, min(rh, M - 1)) + ((lane & 7) ^ ((rh >> 1) & 7)) * 8 + k0 * BK;  // rows past M re-read the last row; masked later
    const int last = min(a.V, 16 * end) - 1;
#pragma unroll
    for (int q = 0; q < LW; ++q) {
      const int rl = wave * (8 * LW) + q * 8 + (lane >> 3);
      gw[q] = (const __bf16*)a.W + (size_t)min(16 * begin + rl, last) * a.d + ((lane & 7) ^ ((rl >> 1) & 7)) * 8 + k0 * BK - q * 512;
    }
  };
  const uint32_t slotH = lds_offset(ringH + hrow0 * 8), slotW = lds_offset(ringW + wave * LW * 64);
  constexpr uint32_t kBytesH = kStageH * 16, kBytesW = kStageW * 16;
  auto advance = [&](int& left) __attribute__((always_inline)) -> long { return --left == 0 ? (long)BK - a.d : (long)BK; };
  auto load_h = [&](int stage) __attribute__((always_inline)) {
    load_to_lds_16(gh, __builtin_amdgcn_readfirstlane(slotH + stage * kBytesH));
    gh += advance(h_left);
  };
  auto load_w = [&](int stage) __attribute__((always_inline)) {
    load_group_to_lds<STREAM_W>(gw, __builtin_amdgcn_readfirstlane(slotW + stage * kBytesW));
    const long move = advance(w_left);
#pragma unroll
    for (int q = 0; q < LW; ++q) gw[q] += move;
  };
  // What the steps before the first would have requested, in their order: W(0), [H(0), W(1)], [H(1), W(2)].  (nk is at least eight.)
  auto prologue = [&]() __attribute__((always_inline)) {
    load_w(0);
    load_h(0);
    load_w(1);
    load_h(1);
    load_w(2);
  };

  floatx4 acc[NT], sum[ROTATE ? kSlices : 1][NT];  // acc[t]: tokens 16 t + 4 g .. + 3 of row i16 of the wavefront's tile
  int fo[2];  // chunk of this lane's fragment of k-half ks within 16 rows of a stage
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) fo[ks] = i16 * 8 + ((ks * 4 + g) ^ ((i16 >> 1) & 7));

  // The chains of the row that thread tid merges; chain c stands in run_m[(c - turned) % 4], since the first 16-token tile of a
  // tile may belong to any.
  float run_m[kChains], run_s[kChains];
#pragma unroll
  for (int c = 0; c < kChains; ++c) {
    run_m[c] = -INFINITY;
    run_s[c] = 0.f;
  }
  int turned = 0;
  auto turn = [&](int to) __attribute__((always_inline)) {
    const int by = (to - turned) & (kChains - 1);
    turned = to;
#pragma unroll
    for (int bit = 1; bit < kChains; bit *= 2) {
      if (!(by & bit)) continue;
      float m[kChains], s[kChains];
#pragma unroll
      for (int c = 0; c < kChains; ++c) {
        m[c] = run_m[(c + bit) & (kChains - 1)];
        s[c] = run_s[(c + bit) & (kChains - 1)];
      }
#pragma unroll
      for (int c = 0; c < kChains; ++c) {
        run_m[c] = m[c];
        run_s[c] = s[c];
      }
    }
  };

  const bool rows_live = __builtin_amdgcn_readfirstlane((int)(16 * wm < M)) != 0;
  int begin = run0, end = tile_begin(1);
  aim(begin, end);
  prologue();
  for (int tile = 0; tile < tiles; ++tile) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
      if constexpr (!ROTATE) sum[0][t] = floatx4{-0.f, -0.f, -0.f, -0.f};  // -0 + x is x
    }
    int slice = slice0, left = per_slice, sw = 0, sh = 0;
    for (int k = 0; k < nk; ++k) {
      // Younger than H(k), the later of the two that this step needs: W(k+1), H(k+1), W(k+2).
      if (k + 2 < nk) wait_newer<2 * LW + 1>();
      else if (k + 1 < nk) wait_newer<LW>();
      else wait_newer<0>();
      lds_barrier();
      if (k + 2 < nk) load_h(sh == 0 ? RH - 1 : sh - 1);
      if (k + 3 < nk) load_w(sw == 0 ? RW - 1 : sw - 1);
      if (rows_live) {
        const bf16x8* Hs = ringH + sh * kStageH + wm * 128;
        const bf16x8* Ws = ringW + sw * kStageW + wn * NT * 128;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const bf16x8 h = Hs[fo[ks]];
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ws[t * 128 + fo[ks]], h, acc[t], 0, 0, 0);
        }
      }
      sw = sw == RW - 1 ? 0 : sw + 1;
      sh = sh == RH - 1 ? 0 : sh + 1;
      if (--left == 0) {  // the slice is complete
        left = per_slice;
        if constexpr (ROTATE) {
          // (The empty statements keep the eight branches apart: merged into one store through an index, the sums would live in
          // scratch memory.  Selects in place of the branches cost 0.4 us per slice.)
          auto keep = [&](auto c_tag) __attribute__((always_inline)) {
            constexpr int c = decltype(c_tag)::value;
            if (slice == c)
#pragma unroll
              for (int t = 0; t < NT; ++t) {
                sum[c][t] = acc[t];
                asm volatile("; slice %1" : "+v"(sum[c][t]) : "n"(c));
              }
          };
          keep(std::integral_constant<int, 0>{});
          keep(std::integral_constant<int, 1>{});
          keep(std::integral_constant<int, 2>{});
          keep(std::integral_constant<int, 3>{});
          keep(std::integral_constant<int, 4>{});
          keep(std::integral_constant<int, 5>{});
          keep(std::integral_constant<int, 6>{});
          keep(std::integral_constant<int, 7>{});
          slice = (slice + 1) & (kSlices - 1);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if constexpr (!ROTATE) sum[0][t] += acc[t];
          acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
    if constexpr (ROTATE)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int c = 1; c < kSlices; ++c) sum[0][t] += sum[c][t];
    lds_barrier();  // nobody reads the rings any more: the first stages of the next tile are on their way during the epilogue
    const int v_tile = 16 * begin, v_end = min(a.V, 16 * end), first = begin - run0;
    if (tile + 1 < tiles) {
      begin = end;
      end = tile_begin(tile + 2);
      aim(begin, end);
      prologue();
    }

    const float sc = a.inv_tau;
    const int vw = v_tile + wn * (16 * NT), v0 = vw + 4 * g;  // first token of the wavefront, of the lane's piece of its first 16-token tile
    if (rows_live && vw < v_end) {
      auto rows = [&](auto edge) __attribute__((always_inline)) {
        constexpr bool EDGE = decltype(edge)::value;  // some of the wavefront's tokens do not exist
        const int rl = 16 * wm + i16;
        floatx4 l[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) l[t] = sum[0][t] * sc;
        // Neighbouring lanes (rows 2j, 2j + 1) trade one of every two 16-token tiles, so that a store instruction writes 128
        // bytes of a row; non-temporal, past the W and H lines in L2.
        const bool odd = i16 & 1;
        const int row2 = rl & ~1;
        const int pairs = EDGE ? (v_end - vw) / 32 : NT / 2;  // whole pairs of 16-token tiles, wavefront-uniform
        float* dst = a.logits + (size_t)row2 * a.ldl + v0 + (odd ? 16 : 0);
#pragma unroll
        for (int t = 0; t < NT; t += 2) {
          floatx4 x, y;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float near = swap_pair(l[t][c]), far = swap_pair(l[t + 1][c]);
            x[c] = odd ? far : l[t][c];
            y[c] = odd ? l[t + 1][c] : near;
          }
          if (EDGE && t / 2 >= pairs) continue;
          if (row2 < M) __builtin_nontemporal_store(x, reinterpret_cast<floatx4*>(dst + 16 * t));
          if (row2 + 1 < M) __builtin_nontemporal_store(y, reinterpret_cast<floatx4*>(dst + a.ldl + 16 * t));
        }
        if constexpr (EDGE) {  // what does not fill a pair
          float* one = a.logits + (size_t)rl * a.ldl + v0;
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if (t / 2 >= pairs && rl < M && v0 + 16 * t + c < v_end) one[16 * t + c] = l[t][c];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if constexpr (EDGE)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if (v0 + 16 * t + c >= v_end) l[t][c] = -INFINITY;
          // maximum of the 16-token tile in every lane, then its sum
          float m = vmax3(vmax3(l[t][0], l[t][1], kLowest), l[t][2], l[t][3]), o = m;
          swap_quarters(m, o);
          m = o = vmax(m, o);
          swap_halves(m, o);
          m = vmax(m, o);
          float e[4];
#pragma unroll
          for (int c = 0; c < 4; ++c)  // one rounding for the scaled logit minus the maximum, as in head_skinny_kernel
            e[c] = EDGE && v0 + 16 * t + c >= v_end ? 0.f : __expf(fmaf(sum[0][t][c], sc, -m));
          float s = ((e[0] + e[1]) + e[2]) + e[3];
          o = s;
          swap_quarters(s, o);
          s = o = s + o;
          swap_halves(s, o);
          if (g == 0) part[NT * wn + t][rl] = make_float2(m, s + o);
        }
      };
      if (vw + 16 * NT <= v_end) rows(std::false_type{});
      else rows(std::true_type{});
    }
    lds_barrier();
    // the thread that owns a row merges its 16-token tiles; the barriers of the next walk stand in front of the next writes
    if (tid < M) {
      turn(first);
#pragma unroll
      for (int t = 0; t < kTile / 16; ++t) {
        if (v_tile + 16 * t >= v_end) break;
        const float2 p = part[t][tid];
        float &rm = run_m[t & (kChains - 1)], &rs = run_s[t & (kChains - 1)];
        if (p.x > rm) {
          rs = rs * __expf(rm - p.x) + p.y;
          rm = p.x;
        } else {
          rs += p.y * __expf(p.x - rm);
        }
      }
    }
  }
  if (tid < M) {
    turn(0);
    float mx = run_m[0], s = 0.f;
#pragma unroll
    for (int c = 1; c < kChains; ++c) mx = fmaxf(mx, run_m[c]);
#pragma unroll
    for (int c = 0; c < kChains; ++c)
      if (run_m[c] > -INFINITY) s += run_s[c] * __expf(run_m[c] - mx);
    a.partials[(size_t)tid * a.nT + blockIdx.x] = make_float2(mx, s);
  }
}

template <int WM, bool ROTATE>
hipError_t launch_form(const HeadArgs& a, int tiles) {
  if (streams_w(a.V, a.d, 2, 1, false)) {
    FEF_LAUNCH_HEAD((head_slices_kernel<WM, ROTATE, true>), dim3(a.nT), dim3(kThreads), a, a, tiles);
  } else {
    FEF_LAUNCH_HEAD((head_slices_kernel<WM, ROTATE, false>), dim3(a.nT), dim3(kThreads), a, a, tiles);
  }
  return hipGetLastError();
}

}  // namespace

// At most 32 rows, d a multiple of 512.
hipError_t launch_head_slices(const HeadArgs& a) {
  const int tiles = (a.V + kSkinnyUnit - 1) / kSkinnyUnit;
  const bool rotate = a.d % 2048 == 0;
  if (a.nrows <= 16) return rotate ? launch_form<1, true>(a, tiles) : launch_form<1, false>(a, tiles);
  return rotate ? launch_form<2, true>(a, tiles) : launch_form<2, false>(a, tiles);
}

}  // namespace fef
