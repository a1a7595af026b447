// Rules that shape the launches of the head kernels: plain host code on sizes, without HIP, so that a program for the CPU can
// check them over all sizes.
#pragma once
#include <stddef.h>

namespace fef {

// W past the caches: non-temporal loads.  A W longer than the Infinity Cache (256 MB) comes from HBM in every call, and as
// ordinary loads it pushes what else is in use, H above all, out of the caches: of the requests to L2 that are not for W 72 % hit at 64
// rows of d = 4096, V = 126464 and 87 % with non-temporal loads, 69 and 87 % at 256 rows (reads from memory 8.6 -> 8.2 and 10.2 -> 8.3
// million lines, W being 8.1).  Per round of 64 rows 203 -> 179 us, of 256 rows 259 -> 252, of 48 rows of d = 4096, V = 40960
// 79 -> 69; 16 fp32 rows of d = 2048, V = 40960 90 -> 83.  At 64 rows that is more than the lines saved account for.
// A shorter W is another matter.  Whether it still lies in the Infinity Cache depends on what the program does between two
// calls, and non-temporal loads neither find it there nor leave it there.  45 bf16 and 20 fp32 calls of 80 to 256 MiB: where nothing
// runs between the calls ordinary loads are up to 1.5 times as fast (16 rows of d = 4864, V = 17354 44.5 against 62.6 us, 190 rows of
// d = 2560, V = 40000 60 against 77), and so is the second half of a split round (8 rows of d = 5056, V = 10577 111 against 129 us
// per round); where the cache is swept in between, non-temporal ones are 0 to 4 % ahead.  Some of a W a little longer than the cache
// stays too: at 258 MiB ordinary loads are up to 1.25 times as fast (16 fp32 rows of d = 2048), at 285 level, from 300 on behind by
// 4 to 10 % (37 rows of a cross-entropy call of d = 1024, V = 151936, 297 MiB, 65 against 59 us).  Hence the line.
// Rows of W that are not whole 128-byte lines (fp32, d not a multiple of 32): the two k-steps that share a line then fetch it twice, at
// any size of W (16 fp32 rows of d = 1046, V = 150369 164 -> 191 us with non-temporal loads, 30 of d = 2548, V = 47390 129 -> 152).
// Two row tiles share W through L2 as far as they keep in step, and non-temporal loads cost a round that (144 rows of d = 7168, V = 22000
// 124 -> 144 us where nothing runs between the calls and 127 -> 150 where the cache is swept, 160 of d = 4608, V = 30000 95 -> 102
// and level, 256 of d = 5120 to 8192 level to 4 % ahead); a cross-entropy call, which writes no logits, loses up to 2 % (300 rows of
// d = 2048, V = 81920) and gains up to 5 (300 rows of d = 4096, V = 126464 315 -> 303 us).  (Losses that loss_wide_serves: ordinary loads, see head_loss.hip.)
inline bool streams_w(size_t V, size_t d, size_t element_bytes, int row_tiles, bool loss) {
  return row_tiles <= (loss ? 2 : 1) && d * element_bytes % 128 == 0 && V * d * element_bytes > (size_t)288 << 20;
}

constexpr int kXcds = 8, kCusPerXcd = 32;

// Rounds of one workgroup per CU that a launch of row_tiles x n_tiles workgroups takes.  Workgroups go to the XCDs in turn and the row
// tiles of a token tile stay on one XCD, so the XCD with the most token tiles decides: 18 token tiles x 14 row tiles are 252
// workgroups, but 42 on two XCDs and 28 on the others.
inline long tile_rounds(long n_tiles, long row_tiles) {
  return ((n_tiles + kXcds - 1) / kXcds * row_tiles + kCusPerXcd - 1) / kCusPerXcd;
}

// Row tiles of a launch over M rows in n_tiles token tiles or runs: equal heights, a multiple of 32, at most `most` rows, and more of them
// than that takes only of `least` rows or more.  ceil(M / most) of them multiply the fewest rows that do not exist and read W the fewest
// times; but a short vocabulary leaves CUs idle then (V = 8437: 33 tiles), or fills a last round badly (V = 20000: 79 tiles x 4
// row tiles).  So the number is taken that makes rounds x (height + 64) smallest; 64 stands for what a k-step and a tile cost whatever
// their height.  More of them read W more often, so where a row is long the gain has to be more than 10 % of that unless they take no
// more rounds (1596 rows of d = 1984, V = 7989 67 us in seven, 63 in eight; 1422 of d = 1088, V = 17824 72 us in six, 67 in seven), and up
// to 256 rows (one row tile, whose W comes at the rate of the caches) the height has to fall below 0.6 of that of one.
// Fitted to the times of 640 calls in every number of row tiles that they allow, with W still in the Infinity Cache and with that cache
// swept: against ceil(M / most) 0.84 and 0.87 of the time in the mean, none slower but for one (4 % with the cache swept, 4 % faster
// without).  Rounds counted over the whole chip instead: 32 of the 640 slower by more than 3 %, up to 1.45 times (2310 rows of d = 4608,
// V = 4491 113 us in 10 row tiles, 152 in 14).  Without the 10 %: 384 rows of d = 3584, V = 44081 142 us in two, 166 in four; with it
// also at short rows: 450 of d = 896, V = 71400 18 % slower.  Without the 0.6: 144 rows of d = 3968, V = 29869 64 us in one tile of 160,
// 83 in two of 96.
inline int row_tiles(int M, int n_tiles, int d, int least, int most) {
  const int fewest = (M + most - 1) / most;
  if ((long)n_tiles * fewest > 8 * 256) return fewest;  // many rounds: the last one matters little
  const auto height_of = [=](int m) { return ((M + m - 1) / m + 31) / 32 * 32; };
  const auto cost_of = [=](int m) { return tile_rounds(n_tiles, m) * (height_of(m) + 64); };
  const bool runs = most == 128;
  int best = fewest;
  for (int height = height_of(fewest) - 32; height >= least; height -= 32) {  // the fewest tiles of each height
    const int m = (M + height - 1) / height;
    if ((long)n_tiles * m > 16 * 256 || height_of(m) < least) break;
    if (!runs && fewest == 1 && 5 * height_of(m) >= 3 * height_of(1)) continue;
    const int enough = runs || d <= 1024 || tile_rounds(n_tiles, m) == tile_rounds(n_tiles, fewest) ? 100 : 90;
    if (100 * cost_of(m) < enough * cost_of(fewest) && cost_of(m) < cost_of(best)) best = m;
  }
  return best;
}

// Cross-entropy of more than 256 rows in row_tiles row tiles: eight wavefronts, or four as a verify step.  Two wavefronts per SIMD overlap
// prologue and epilogue better, one asks LDS for fewer fragments.  Up to d = 1024 eight are ahead by 3 to 5 % (500 rows of
// V = 126464 126 -> 121 us), but for 1 us behind in low tiles of a short vocabulary; beyond, in two row tiles, by up to 10 % (300 rows
// of V = 50257, before loss_wide_serves took them, 84 -> 79 at d = 2048, 147 -> 139 at d = 4096) as long as the tile is low or the walk over k short: 512 rows of d = 3072 2
// to 5 % ahead or level, of d = 3584 up to 3 behind, of d = 4352 10 (V = 151936 522 -> 572); 384 rows of d = 4096 4 % ahead, of
// d = 5120 level.  In more row tiles 1 to 8 % behind.  Their error against 64 bits is the same (nine sizes of 257 to 1000 rows, six
// seeds each: 1.8e-7 to 3.7e-7 with four and 1.8e-7 to 3.4e-7 with eight, now one ahead and now the other).
inline bool loss_takes_eight_wavefronts(int M, int row_tiles, int d) {
  const int height = ((M + row_tiles - 1) / row_tiles + 31) / 32 * 32;
  return d <= 1024 || (row_tiles == 2 && d <= (height <= 192 ? 4096 : 3072));
}

// Up to 32 rows, H in registers or in LDS beside W (head_slices.hip): the latter where a workgroup's run, of one in 256, is longer than 128
// tokens.  Head alone, 322 calls of 2 to 32 rows in the seven hidden sizes and 23 vocabularies of 12000 to 151936, three Ws in turn: above the
// line 0.94 of the time in the mean, at V = 32000 1.00, at 28700 1.02, at 16400 1.24, at 12000 1.48 (short runs leave the CUs too little of W
// on its way).  d = 1024 is ahead up to V = 65536 and again where W is read past the caches, and 3 to 8 % behind in between (16 rows of
// V = 80000 33.7 -> 35.9 us, of V = 126464 49.9 -> 52.6).
inline bool slices_serve(int V, int d) {
  return V > 256 * 128 && (d != 1024 || V <= 65536 || streams_w((size_t)V, (size_t)d, 2, 1, false));
}
// ... but for calls of short rows where the kernel with H in LDS falls behind nevertheless: its runs have just become two tiles of half the
// length (V > 65536), which leaves the CUs less W on its way, and non-temporal loads do not make up for it yet.  Per call, with H in registers ->
// in LDS, three Ws in turn and one W: 8, 16 and 32 rows of d = 512, V = 65600 1.05, 1.03 and 1.04 times either way, from V = 82000 on level or ahead;
// of d = 2048, V = 67000 1.06, 1.04 and 1.09 and 1.07, 1.04 and 1.10, V = 72000 1.01, 1.00 and 1.05 and 1.01, 1.00 and 1.06, V = 73000 1.02, 1.01 and
// 1.04 and 1.04, 1.03 and 1.07, from the line of streams_w on 0.91 to 0.99 with three Ws.  d = 1024, V = 65300 to 65536: (almost) all runs start a multiple of
// 512 KB apart, 16 rows 39.7 -> 44 us with three Ws (V = 65100, where H in registers meets the same: 45 -> 41) and level with one.
inline bool slices_lag(int V, int d) {
  if (d == 512) return V > 256 * 256 && V <= 256 * 320;
  if (d == 1024) return V > 16 * 4072 && V <= 256 * 256;
  return d == 2048 && V > 256 * 256 && !streams_w((size_t)V, (size_t)d, 2, 1, false);
}

// Runs (STREAM, ROWSTREAM: units of 64 and 16 tokens) whose longest has that many tokens: by head_runs_kernel, which walks k once over all of
// them, or by head_tiled256_kernel, one tile of up to 256 tokens after another.  Head alone in us, three Ws in turn.
// Runs of up to 128 tokens (V <= 32768; up to 16384 mostly in pieces, see pieces_pay) fill half a tile of 256, and half its stages: 48 rows of
// d = 4096, V = 24000 49.0 -> 42.8, 96 rows of d = 2560, V = 32000 46.6 -> 43.9, 80 calls 0.94 of the time in the mean.  At d = 512 eight steps are too few
// for it to matter and longer runs fall 3 % behind.
inline bool short_runs_serve(int unit, long longest, int d) { return unit == 16 && longest <= 128 && (d > 512 || longest <= 96); }
// ... but sixteen steps are too few up to 64 rows once most CUs have a run: 16 rows of d = 1024, V = 21504 (168 runs) 23.5 -> 24.2 us per call, 32 of
// V = 27000 26.0 -> 26.9, 64 of V = 24000 and 32768 1.02 times, with three Ws and with one; 2 to 64 rows of V = 18000 0.95 to 1.01, of V = 19000 to 20352 (159
// runs) 0.95 to 1.04, 66 rows 0.93 to 1.01, 128 0.90 to 0.97.
inline bool short_runs_lag(int rows, long n_runs, int d) { return d == 1024 && rows <= 64 && n_runs >= 160; }
// Runs of 257 to 512 tokens are a tile of 256 and a narrow one, whose k-steps cost the load latency however few tokens it has: 110 rows of
// d = 2560, V = 100003 111.9 -> 101.4, 64 rows of d = 2048, V = 66000 71.7 -> 59.9, 128 rows of d = 512, V = 126464 43.9 -> 38.4.  Two full
// tiles do better one after the other (40 rows of d = 4096, V = 115000 149 -> 162 on one machine, level on another), and with more than
// 96 rows and long rows so do shorter ones (128 rows of d = 3584, V = 75000 122 -> 134).  240 calls of 40 to 128 rows: where this says
// yes 0.91 of the time in the mean; 312 of 2 to 32 rows 0.90, and 0.91 with one W, 3 and 5 % behind at most.  Between d = 2560 and 3584 with more than
// 96 rows the line is drawn on the careful side: 120 calls of 98 to 128 rows of d = 2688 to 3584, V = 66000 to 106496 take 0.90 to 1.02 of the
// time in one walk, 0.93 to 1.05 with one W.
inline bool double_runs_serve(int rows, long longest, int d) {
  if (longest <= 256) return false;
  if (d <= 1024) return longest <= (rows <= 48 ? 384 : 512);
  return rows > 96 ? d <= 2560 && longest <= 448 : longest <= 320;
}

// Verify steps of a short vocabulary: the runs (or tiles) that carry a partial each are too few for 256 CUs, and a CU takes in no more than some
// 48 KB per us of W and H however many stages it asks for.  So a run is cut into pieces, a workgroup each (head_runs.hip), and the partials are
// made from the logits by the kernel that merges them (row_sums_draft_kernel), which costs 1 to 2 us more than reading them.
struct PieceShape {
  int pieces, tokens, rows, row_tiles;  // per run, of up to `tokens` tokens (64 or 128), in row tiles of `rows` rows (64 or 128); pieces 0: none
};
// Where that pays, per call in us, three Ws in turn and with W still in the Infinity Cache: 64 rows of d = 4096, V = 8000 64.1 -> 42.3 and 45.5 -> 39.7;
// 256 rows of d = 4096, V = 8000 74.2 -> 48.1 and 56.8 -> 43.8, V = 16384 78.0 -> 64.5 and 61.0 -> 59.3; 128 rows of d = 2560, V = 12000 52.9 -> 41.4 and
// 38.1 -> 35.7; 96 rows of d = 1024, V = 3000 25.5 -> 21.8 and 26.1 -> 22.4.  780 calls of 12 to 256 rows, d = 512 to 4096, V = 3000 to 16384, half of them
// either way: where this says yes 0.87 of the time in the mean, none more than 5 % behind both ways; 297 of 2 to 10
// rows 0.82 and 0.89, none behind by more than 2 % either way; 1030 of 34 to 256 rows 0.83 and 0.85, 1 % of them behind by 2 to 4 % (200 to 224 rows of
// d = 2560, V = 10000 by 3 to 5).  Where it says no: the second row tile of 128 multiplies rows that one of 224 does not have (194 to 224 rows of d = 1792 to 2304,
// V = 8193 to 12288 1.05 to 1.08 of the time both ways, 226 to 256 0.98 to 1.01), steps are few (256 rows of d = 512, V = 4608 1.03, V = 5120 1.05, but V = 4000
// 0.96), a walk is short and the sums
// cost what it gains (256 rows of d = 512, V = 13000 1.22 and 1.25 of the time), a second row tile is half empty (192 rows of d = 4096, V = 16384
// 0.80 and 1.13), and beyond V = 16384 up to 64 rows gain 9 to 19 % one way and lose 8 to 15 the other.
constexpr int kPieceTokens = 16384;  // the longest vocabulary: a thread of that kernel takes 16 tokens
inline bool pieces_pay(int M, int V, int d) {
  if (M > 256 || d < 512 || V > kPieceTokens || streams_w((size_t)V, (size_t)d, 2, 1, false)) return false;
  if (V <= 5120) return M > 8 && (M <= 192 || d >= 1024 || V <= 4096);
  if (M <= 16 && d < 1280) return false;
  if (M <= 128) return V <= (d >= 1280 ? kPieceTokens : M <= 64 ? 12288 : 8192);
  if (V <= 8192) return d >= 1280;
  if (M > 192 && M <= 224 && d < 2560) return false;
  return d >= 1792 && V <= (d >= 2560 ? M > 192 ? kPieceTokens : 12288 : M > 192 ? 12288 : 10240);
}
// Equal pieces of 64 or 128 tokens and row tiles of 64 or 128 rows: the shape that makes (rounds of the busiest XCD) x (rows + tokens + 64)
// smallest, for the bytes of a k-step are those of its rows and its tokens.
inline PieceShape piece_shape(int M, int V, int d, int n_runs, int unit) {
  PieceShape best{0, 0, 0, 0};
  if (!pieces_pay(M, V, d)) return best;
  const int run = unit == 16 ? 128 : 256;
  long least = 0;
  for (int tokens = 64; tokens <= 128; tokens *= 2)
    for (int rows = 64; rows <= (M <= 64 ? 64 : 128); rows *= 2) {
      const int pieces = run / tokens, m = (M + rows - 1) / rows;
      const long cost = tile_rounds(n_runs, (long)pieces * m) * (rows + tokens + 64);
      if (!best.pieces || cost < least) {
        best = PieceShape{pieces, tokens, rows, m};
        least = cost;
      }
    }
  return best;
}

// Cross-entropy of a little more than 256 rows whose vocabulary is one round of shares of 177 to 224 tokens (320 rows: 192): all rows in one row tile
// (head_loss.hip).  Two row tiles of whole token tiles are one round and a half there, and read W twice.  Head alone in us, 300 rows, three Ws in turn
// and one W: d = 512, V = 50257 28.8 -> 25.6 and 26.4 -> 23.3, d = 2048 77.8 -> 68.4 and 67.4 -> 59.8, d = 4096 137.5 -> 123.6 and 137.1 -> 126.7;
// d = 3072, V = 47000 111.7 -> 90.7 and 103.5 -> 78.4.  Narrower shares gain 8 to 17 % one way (d = 2048, V = 40000 68.8 -> 58.4) and lose up to 10 the
// other (260 rows of d = 3072, V = 40000 67.7 -> 74.5): the second round of the two tiles is short then.
inline bool loss_wide_serves(int M, int V) { return M > 256 && M <= 320 && V > 256 * 176 && V <= 256 * (M <= 304 ? 224 : 192); }

// Token tiles of an fp32 launch below which they are dealt out one by one instead of by XCD: 2048 sequences x 16 rows of V = 256 80 -> 53 us
// per call.
constexpr int kF32FewTiles = 64;

// Row tiles of an fp32 launch: equal heights of 16 to 64 rows.  As few as possible, for every one reads W again, but more where that leaves
// CUs idle or gives some of them more than others: the number that makes (workgroups of the busiest CU) x (height + 16) smallest,
// more of them only for 3 % of it.  (Several workgroups share a CU, so a CU's work counts and not its rounds.)  A workgroup of 48 or 64 rows
// that has its CU to itself counts 24 more: one wavefront per SIMD overlaps with nothing (60 rows of d = 1848, V = 9284 60.4 us in one
// tile, 55.9 in two).  Fitted to 160 calls in every number of row tiles that they allow: 0.89 of the time in as few as possible, 0.9 %
// behind the best, none slower than 1 %.  "More of them up to 240 workgroups", whatever their height, was slower than as few as possible for
// one call in twenty: 113 rows of d = 3976, V = 7478 109 us in two, 134 in three (101 in four, as now).
inline int f32_row_tiles(int M, int n_tiles) {
  const int fewest = (M + 63) / 64;
  const auto cost_of = [=](int m) -> long {
    const long height = ((M + m - 1) / m + 15) / 16 * 16;
    const long cus = kXcds * kCusPerXcd, busiest = n_tiles < kF32FewTiles ? ((long)n_tiles * m + cus - 1) / cus : tile_rounds(n_tiles, m);
    return busiest * (height + 16) + (busiest == 1 && height >= 48 ? 24 : 0);
  };
  int best = fewest;
  if (cost_of(fewest) > 8L * (64 + 16)) return best;  // many workgroups per CU: the last ones matter little
  for (int height = 48; height >= 16; height -= 16) {  // the fewest tiles of each height
    const int m = (M + height - 1) / height;
    if (m > fewest && 100 * cost_of(m) < 97 * cost_of(best)) best = m;
  }
  return best;
}

}  // namespace fef
