// Sampling and verification kernels that follow the vocabulary head (Algorithm 2 of the
// paper, lines "Sample draft tokens" to "break", and the LowConf re-corruption):
//
//   row_lse_draft_kernel     one wavefront per logits row: merge the head kernel's per-tile
//                            (max, sum exp) partials into the row's log-sum-exp; draft rows
//                            also locate their window slot and draw x~ ~ rho by a two-level
//                            inverse CDF (tiles, then tokens inside the tile).
//   accept_resid_kernel      per sequence: accept tests u <= min{1, pi(x~)/rho(x~)}, first
//                            rejection by ballot; per 256-token chunk the residual mass
//                            sum [pi - rho]_+ of the rejected slot.
//   slot_mass_kernel         in its place where the masses of every slot are wanted: residual and
//                            overlap mass (sum min{pi, rho}) per slot and chunk.
//   finalize_kernel          per sequence: inverse CDF over the residual chunks and inside
//                            the selected chunk, commit of tokens and confidences, block-mask
//                            update and LowConf.  (A separate launch on purpose: handing the
//                            chunk masses to a last-arriving workgroup inside one kernel needs
//                            device-scope fences, which write back and invalidate a whole
//                            XCD's L2 each time; measured 300 us at B = 64 against 13 us.)
//
// Every floating-point reduction uses a fixed tree (no float atomics), so results are
// reproducible bit for bit.
#include <limits.h>
#include <math.h>

#include <type_traits>

#include "fef_device.hpp"
#include "head_f32.hpp"
#include "wave_ops.hpp"

namespace fef {
namespace {

constexpr int NT = 256;          // threads per workgroup of every kernel in this file
constexpr int NW = NT / kWave;   // wavefronts per workgroup

struct BlockTmp {
  float f[NW];
  int i[NW];
  float bcast_f, bcast_u;
  int bcast_i;
};

__device__ inline float block_sum(float x, BlockTmp& t) {
  x = wave_sum(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) t.f[threadIdx.x >> 6] = x;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) s += t.f[w];
  return s;
}
__device__ inline float block_max(float x, BlockTmp& t) {
  x = wave_max(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) t.f[threadIdx.x >> 6] = x;
  __syncthreads();
  float s = t.f[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) s = fmaxf(s, t.f[w]);
  return s;
}
__device__ inline int block_min_int(int x, BlockTmp& t) {
  x = wave_min_int(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) t.i[threadIdx.x >> 6] = x;
  __syncthreads();
  int s = t.i[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) s = min(s, t.i[w]);
  return s;
}
__device__ inline int block_max_int(int x, BlockTmp& t) {
  x = wave_max_int(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) t.i[threadIdx.x >> 6] = x;
  __syncthreads();
  int s = t.i[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) s = max(s, t.i[w]);
  return s;
}

// Exclusive prefix sum of one value per thread in thread order; `total` gets the sum.
__device__ inline float block_exclusive_scan(float x, BlockTmp& t, float& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const float inc = wave_scan_add(x);
  float exc = __shfl_up(inc, 1, 64);
  if (lane == 0) exc = 0.f;
  __syncthreads();
  if (lane == 63) t.f[w] = inc;
  __syncthreads();
  float base = 0.f, tot = 0.f;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    if (i == w) base = tot;
    tot += t.f[i];
  }
  total = tot;
  return base + exc;
}

struct Found {
  int idx;       // first index whose inclusive prefix sum reaches the target
  float before;  // prefix sum of everything before idx
  float total;   // sum of all masses
};

// min{i in [0,n) : sum_{j<=i} mass(j) >= target} over non-negative masses, ascending i.
// Thread t owns the contiguous segment [t*per, (t+1)*per).  If rounding leaves every prefix
// below the target, the last index with positive mass is returned (index 0 if there is none).
template <class F>
__device__ inline Found block_find_first(int n, F mass, float target, BlockTmp& t) {
  const int per = (n + NT - 1) / NT;
  const int begin = min(n, (int)threadIdx.x * per), end = min(n, begin + per);
  float local = 0.f;
  for (int i = begin; i < end; ++i) local += mass(i);
  float total;
  const float exc = block_exclusive_scan(local, t, total);
  float run = exc, before = 0.f, before_pos = 0.f;
  int cand = INT_MAX, last_pos = -1;
  for (int i = begin; i < end; ++i) {
    const float mi = mass(i);
    const float nxt = run + mi;
    if (mi > 0.f) { last_pos = i; before_pos = run; }
    if (cand == INT_MAX && nxt >= target) { cand = i; before = run; }
    run = nxt;
  }
  int win = block_min_int(cand, t);
  bool mine = cand != INT_MAX && cand == win;
  if (win == INT_MAX) {  // target not reached: fall back to the last positive mass
    const int lp = block_max_int(last_pos, t);
    if (lp < 0) { win = 0; mine = threadIdx.x == 0; before = 0.f; }
    else { win = lp; mine = last_pos == lp; before = before_pos; }
  }
  __syncthreads();
  if (mine) t.bcast_f = before;
  __syncthreads();
  Found f;
  f.idx = win;
  f.before = t.bcast_f;
  f.total = total;
  return f;
}

// Token range of partial tile i: [unit * floor(i T / G), unit * floor((i+1) T / G)) within [0, V).
__device__ inline int tile_start(const VerifyArgs& a, int i) {
  return (int)((long)i * a.tile_T / a.tile_G) * a.tile_unit;
}

// Wavefront version of block_find_first: lane l owns the contiguous segment [l*per, (l+1)*per).
template <class F>
__device__ inline Found wave_find_first(int n, F mass, float target) {
  const int lane = threadIdx.x & 63;
  const int per = (n + kWave - 1) / kWave;
  const int begin = min(n, lane * per), end = min(n, begin + per);
  float local = 0.f;
  for (int i = begin; i < end; ++i) local += mass(i);
  const float inc = wave_scan_add(local);
  float exc = __shfl_up(inc, 1, 64);
  if (lane == 0) exc = 0.f;
  float run = exc, before = 0.f, before_pos = 0.f;
  int cand = INT_MAX, last_pos = -1;
  for (int i = begin; i < end; ++i) {
    const float mi = mass(i);
    const float nxt = run + mi;
    if (mi > 0.f) { last_pos = i; before_pos = run; }
    if (cand == INT_MAX && nxt >= target) { cand = i; before = run; }
    run = nxt;
  }
  int win = wave_min_int(cand);
  bool mine = cand != INT_MAX && cand == win;
  if (win == INT_MAX) {  // target not reached: fall back to the last positive mass
    const int lp = wave_max_int(last_pos);
    if (lp < 0) { win = 0; mine = lane == 0; before = 0.f; }
    else { win = lp; mine = last_pos == lp; before = before_pos; }
  }
  const unsigned long long owner = __ballot(mine);
  Found f;
  f.idx = win;
  f.before = __shfl(before, __ffsll((long long)owner) - 1, 64);
  f.total = __shfl(inc, 63, 64);
  return f;
}

// Register-resident variant of wave_find_first: lane l holds the masses of elements
// l*PER .. l*PER + PER-1 (zero beyond the end).
// REL: the target is a fraction of the total mass.
template <int PER, bool REL = false>
__device__ inline Found wave_find_first_reg(const float (&m)[PER], float target) {
  const int lane = threadIdx.x & 63;
  float local = 0.f;
#pragma unroll
  for (int j = 0; j < PER; ++j) local += m[j];
  const float inc = wave_scan_add(local);
  if (REL) target *= __shfl(inc, 63, 64);
  float exc = __shfl_up(inc, 1, 64);
  if (lane == 0) exc = 0.f;
  float run = exc, before = 0.f, before_pos = 0.f;
  int cand = -1, last_pos = -1;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const float nxt = run + m[j];
    if (m[j] > 0.f) { last_pos = j; before_pos = run; }
    if (cand < 0 && nxt >= target) { cand = j; before = run; }
    run = nxt;
  }
  // segments ascend with the lane id: the lowest lane that reached the target holds the answer
  unsigned long long hit = __ballot(cand >= 0);
  int owner;
  if (hit) {
    owner = __ffsll((long long)hit) - 1;
  } else {  // target not reached: fall back to the last positive mass
    hit = __ballot(last_pos >= 0);
    owner = hit ? 63 - __clzll((long long)hit) : 0;
    cand = last_pos < 0 ? 0 : last_pos;
    before = before_pos;
  }
  Found f;
  f.idx = owner * PER + __shfl(cand, owner, 64);
  f.before = __shfl(before, owner, 64);
  f.total = __shfl(inc, 63, 64);
  return f;
}

// window slot m = (m+1)-th unresolved position of block b in ascending order; also counts the
// unresolved positions.  Whole wavefront.
__device__ inline int window_slot(const VerifyArgs& a, int b, int m, int& unresolved) {
  const int lane = threadIdx.x & 63;
  int cnt = 0, pos = -1;
  for (int base = 0; base < a.block; base += kWave) {
    const int i = base + lane;
    const bool bit = i < a.block && (a.mask_in ? a.mask_in[(size_t)b * a.block + i] != 0 : true);
    const unsigned long long bal = __ballot(bit);
    const int rank = cnt + __popcll(bal & ((1ull << lane) - 1ull));
    if (bit && rank == m) pos = i;
    cnt += __popcll(bal);
  }
  unresolved = cnt;
  return wave_max_int(pos);
}

// Greedy variant: arg max of a logits row (lowest token id on a tie) from the head kernel's
// partials.  Every partial maximum is the exact maximum of the stored logits of its tile, so the
// first tile whose maximum equals the row maximum holds the answer, and the first token of that
// tile whose stored logit equals it is the arg max.  Whole wavefront.
__device__ inline int row_argmax(const VerifyArgs& a, const float2* P, const float* L, float row_max) {
  const int lane = threadIdx.x & 63;
  int cand = INT_MAX;
  for (int t = lane; t < a.nT && cand == INT_MAX; t += kWave)
    if (P[t].x == row_max) cand = t;
  const int tile = wave_min_int(cand);
  if (tile == INT_MAX) return 0;  // only if the row holds NaN
  const int v0 = tile_start(a, tile);
  const int nv = min(tile_start(a, tile + 1), a.V) - v0;
  cand = INT_MAX;
  for (int i = lane; i < nv && cand == INT_MAX; i += kWave)
    if (L[v0 + i] == row_max) cand = i;
  const int idx = wave_min_int(cand);
  return idx == INT_MAX ? v0 : v0 + idx;
}

constexpr int kChunkPer = 16;  // residual chunks per lane in the one-wavefront final phase
constexpr int kTilePer = 10;  // tokens per lane inside one partial tile: up to 640 tokens (a 151936-token vocabulary over
                              // 256 workgroups: 576 to 640 tokens each); longer ones are re-read

// ---------------------------------------------------------------------------------------------
// Kernel 1: per-row log-sum-exp, window slot, draft sample.  One wavefront per row.
// PER > 0: the row's partials (at most 64*PER) and the tokens of the selected tile live in
// registers, so every global value is loaded once and every exponential evaluated once.
// PER == 0: any number of partials, re-read from memory.
// ---------------------------------------------------------------------------------------------
constexpr int exchange_floats(int per) { return per > 10 ? kWave * (per + 1) : 0; }

// One row by one wavefront from its partials P; ex: its slice of LDS for the tokens of a tile, exchange: for the partials (PER > 10).
template <int PER>
__device__ __forceinline__ void row_lse_draft(const VerifyArgs& a, int r, const float2* P, float* ex, float* exchange) {
  const int lane = threadIdx.x & 63;
  const int BK = a.B * a.K;
  const bool is_draft = r < BK;
  const int s = is_draft ? r : r - BK;
  const int b = s / a.K, m = s % a.K;

  // log-sum-exp of the row from the head kernel's per-tile partials; the window slot and a given draft token are asked
  // for in the same breath (each trip to memory that waits for another costs about 1 us)
  int pos = -1, window = 0, given = -1;
  float u = 0.f;  // the slot's draft uniform
  auto window_and_token = [&]() {
    if (!is_draft) return;
    int unresolved;
    if (a.draft_tokens_in) given = a.draft_tokens_in[s];
    // The generator's ten rounds are a chain of about 0.4 us.  In a block of up to 64 positions every lane draws for one
    // position while the mask is on its way, and the slot's position picks the lane.
    float u_lane = 0.f;
    if (a.block <= kWave)
      u_lane = philox_uniform(a.seed, a.pos_base + (uint32_t)lane, a.step, a.seq_base + (uint32_t)b, kStreamDraft);
    pos = window_slot(a, b, m, unresolved);
    window = min(a.K, unresolved);
    u = a.block <= kWave ? __shfl(u_lane, max(pos, 0), kWave)
                         : philox_uniform(a.seed, a.pos_base + (uint32_t)pos, a.step, a.seq_base + (uint32_t)b, kStreamDraft);
  };
  float mass[PER > 0 ? PER : 1];  // exp-sums of this lane's tiles relative to the row maximum
  float mx = -INFINITY, sm = 0.f;
  if constexpr (PER > 0) {
    // Lane l owns the consecutive tiles l*PER .. l*PER + PER-1 (the ordered search below needs
    // that).  With few partials per lane it loads them as they lie (PER * 8 contiguous bytes per
    // lane); with many it loads tile j*64 + l, 512 contiguous bytes per instruction, and hands
    // each exp-sum to its owner through this wavefront's slice of LDS (rows of PER + 1 floats,
    // an odd stride, so both directions are conflict-free).
    constexpr bool EXCHANGE = exchange_floats(PER) > 0;
    float2 p[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int t = EXCHANGE ? j * kWave + lane : lane * PER + j;
      p[j] = t < a.nT ? P[t] : make_float2(-INFINITY, 0.f);
    }
    window_and_token();
#pragma unroll
    for (int j = 0; j < PER; ++j) mx = fmaxf(mx, p[j].x);
    mx = wave_max(mx);
#pragma unroll
    for (int j = 0; j < PER; ++j) mass[j] = p[j].y > 0.f ? p[j].y * expf(p[j].x - mx) : 0.f;
    if constexpr (EXCHANGE) {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int t = j * kWave + lane;
        exchange[(t / PER) * (PER + 1) + t % PER] = mass[j];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // same wavefront on both sides: order only
#pragma unroll
      for (int j = 0; j < PER; ++j) mass[j] = exchange[lane * (PER + 1) + j];
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) sm += mass[j];
  } else {
    window_and_token();
    for (int t = lane; t < a.nT; t += kWave) mx = fmaxf(mx, P[t].x);
    mx = wave_max(mx);
    for (int t = lane; t < a.nT; t += kWave) {
      const float2 p = P[t];
      sm += p.y * expf(p.x - mx);
    }
  }
  sm = wave_sum(sm);
  const float lse = mx + logf(sm);
  if (lane == 0) {
    a.lse[r] = lse;
    if (a.diag_lse) a.diag_lse[r] = lse;
  }
  if (!is_draft) {
    if (a.greedy) {  // point mass of the target law
      const int xt = row_argmax(a, P, a.logits + (size_t)r * a.ldl, mx);
      if (lane == 0) a.xtarget[s] = xt;
    }
    return;
  }

  if (lane == 0) {
    a.slot_pos[s] = pos;
    if (m == 0) a.window[b] = window;
  }
  int x = -1;
  if (m < window) {
    if (a.draft_tokens_in) {
      x = min(max(given, 0), a.V - 1);  // keep the gathers in bounds
    } else if (a.greedy) {
      x = row_argmax(a, P, a.logits + (size_t)r * a.ldl, mx);  // point mass of the draft law
    } else {
      // x~ = min{v : sum_{w<=v} rho_w >= u}: first over vocabulary tiles, then inside the tile
      Found tile;
      if constexpr (PER > 0) {
        const float inv = 1.f / sm;  // tile probability = exp-sum / row exp-sum
#pragma unroll
        for (int j = 0; j < PER; ++j) mass[j] *= inv;
        tile = wave_find_first_reg(mass, u);
      } else {
        tile = wave_find_first(
            a.nT, [&](int t) { const float2 p = P[t]; return p.y * expf(p.x - lse); }, u);
      }
      const float* L = a.logits + (size_t)r * a.ldl;
      const int v0 = tile_start(a, tile.idx);
      const int nv = min(tile_start(a, tile.idx + 1), a.V) - v0;
      Found in;
      if (nv <= kWave * kTilePer) {
        // The prefix sums run over kTilePer tokens per lane whatever the tile's length: they decide the token, and another
        // grouping rounds otherwise.  In a short tile that would leave most lanes idle, so there every lane evaluates one
        // or four exponentials and hands them over (50.2 -> 48.8 us per fp32 call of 32 rows of V = 32000 with diagnostics and
        // logits, 14.5 -> 13.1 at a toy vocabulary; 25.9 -> 24.6 per round of 80 rows of d = 512, V = 9000).
        float q[kTilePer];
        if (nv <= kWave) {
          const float e = lane < nv ? expf(L[v0 + lane] - lse) : 0.f;
#pragma unroll
          for (int j = 0; j < kTilePer; ++j) {
            const int i = lane * kTilePer + j;
            const float ei = __shfl(e, i & (kWave - 1), kWave);
            q[j] = i < kWave ? ei : 0.f;
          }
        } else if (nv <= 4 * kWave) {
          const int i0 = 4 * lane;
          float4 e;
          e.x = i0 < nv ? expf(L[v0 + i0] - lse) : 0.f;
          e.y = i0 + 1 < nv ? expf(L[v0 + i0 + 1] - lse) : 0.f;
          e.z = i0 + 2 < nv ? expf(L[v0 + i0 + 2] - lse) : 0.f;
          e.w = i0 + 3 < nv ? expf(L[v0 + i0 + 3] - lse) : 0.f;
          *reinterpret_cast<float4*>(ex + i0) = e;
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // same wavefront on both sides: order only
#pragma unroll
          for (int j = 0; j < kTilePer; j += 2) {
            const int i = lane * kTilePer + j;
            const float2 pair = *reinterpret_cast<const float2*>(ex + min(i, 4 * kWave - 2));
            q[j] = i < 4 * kWave ? pair.x : 0.f;
            q[j + 1] = i < 4 * kWave ? pair.y : 0.f;
          }
        } else {
#pragma unroll
          for (int j = 0; j < kTilePer; ++j) {
            const int i = lane * kTilePer + j;
            q[j] = i < nv ? expf(L[v0 + i] - lse) : 0.f;
          }
        }
        in = wave_find_first_reg(q, u - tile.before);
      } else {
        in = wave_find_first(nv, [&](int i) { return expf(L[v0 + i] - lse); }, u - tile.before);
      }
      x = v0 + in.idx;
    }
  }
  if (lane == 0) {
    a.xdraft[s] = x;
    if (a.diag_draft_tokens) a.diag_draft_tokens[s] = x;
    if (a.phase == 1) a.out_tokens[s] = x;  // draft-only call: the caller gets the draft tokens
  }
}

template <int PER>
__global__ __launch_bounds__(NT) void row_lse_draft_kernel(VerifyArgs a) {
  __shared__ __attribute__((aligned(16))) float tile_mass[NW][4 * kWave];
  __shared__ float exchange[NW][exchange_floats(PER) + 1];
  const int wave = threadIdx.x >> 6;
  const int r = a.row0 + blockIdx.x * NW + wave;
  if (r < a.row0 + a.nrows) row_lse_draft<PER>(a, r, a.partials + (size_t)r * a.nT, tile_mass[wave], exchange[wave]);
}

// ---------------------------------------------------------------------------------------------
// Kernel 1 of a call whose head left no partials (head_rules.hpp: pieces_pay): one workgroup per row makes them from the logits, with the
// sums of the head kernels to the bit (head_gemm_tiled256.hip, "The order of the sums"), and one of its wavefronts goes on as above.
// BLOCK = 64: (max, sum exp) of 64 tokens, merged per run of up to four; 16: of 16 tokens, up to eight.
// Four threads per 64 tokens, 16 tokens each straight from memory: bound by the chain load, exponentials, two hand-overs through LDS (1 to
// 2 us on top of kernel 1).  A token per lane and reductions over the wavefront instead: +12 us at V = 32000; a block of 64 per thread
// through LDS: +4, with 20 KB of code that arrive from a cold instruction cache.
// ---------------------------------------------------------------------------------------------
constexpr int kSumThreads = kPieceTokens / 16;

template <int BLOCK>
__global__ __launch_bounds__(kSumThreads) void row_sums_draft_kernel(VerifyArgs a) {
  constexpr float kLog2e = 1.4426950408889634f;
  __shared__ float2 blocks[kPieceTokens / BLOCK];
  __shared__ float2 runs[256];
  __shared__ __attribute__((aligned(16))) float tile_mass[4 * kWave];
  const int tid = threadIdx.x;
  const int r = a.row0 + blockIdx.x;
  // This thread's tokens.  BLOCK = 64: v .. v + 7 and v + 32 .. v + 39, v's bits 4 and 3 from the thread; 16: v .. v + 15.
  const int v = BLOCK == 64 ? tid / 4 * 64 + tid % 4 * 8 : tid * 16;
  constexpr int kFar = BLOCK == 64 ? 32 : 8;
  auto token = [&](int j) { return v + (j < 8 ? j : j - 8 + kFar); };
  if (tid / 4 * 64 < a.V) {  // (the four threads of 64 tokens together: they trade)
    const float* L = a.logits + (size_t)r * a.ldl + v;  // rows are padded to 64 tokens
    float l[16];
#pragma unroll
    for (int j = 0; j < 16; j += 4) {
      const floatx4 x = *reinterpret_cast<const floatx4*>(L + (j < 8 ? j : j - 8 + kFar));
#pragma unroll
      for (int c = 0; c < 4; ++c) l[j + c] = x[c];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (token(j) >= a.V) l[j] = -INFINITY;
    auto other = [](float x, auto ctrl) {  // the value of another thread of the four
      return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    using Bit0 = std::integral_constant<int, 0xB1>;  // quad_perm [1, 0, 3, 2]
    using Bit1 = std::integral_constant<int, 0x4E>;  // quad_perm [2, 3, 0, 1]
    float mx = kLowest;
#pragma unroll
    for (int j = 0; j < 16; j += 2) mx = vmax3(mx, l[j], l[j + 1]);
    if constexpr (BLOCK == 64) {
      mx = vmax(mx, other(mx, Bit0{}));
      mx = vmax(mx, other(mx, Bit1{}));
    }
    const float mb = mx * -kLog2e;
#pragma unroll
    for (int j = 0; j < 16; ++j) l[j] = __builtin_amdgcn_exp2f(fmaf(l[j], kLog2e, mb));
    float e;
    if constexpr (BLOCK == 64) {
      // tokens j and j + 32, then bits 3 (the neighbouring thread), 2, 1, 0 of j, then bit 4
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        l[j] += l[j + 8];
        l[j] += other(l[j], Bit0{});
      }
#pragma unroll
      for (int bit = 4; bit >= 1; bit /= 2)
#pragma unroll
        for (int j = 0; j < bit; ++j) l[j] += l[j + bit];
      e = l[0] + other(l[0], Bit1{});
    } else {
      // four neighbours in order, then the groups of four pairwise
#pragma unroll
      for (int j = 0; j < 16; j += 4) l[j] = ((l[j] + l[j + 1]) + l[j + 2]) + l[j + 3];
      e = (l[0] + l[4]) + (l[8] + l[12]);
    }
    if (BLOCK == 16 || tid % 4 == 0) blocks[v / BLOCK] = make_float2(mx, e);
  }
  __syncthreads();
  if (tid < a.nT) {
    const int b0 = tile_start(a, tid) / BLOCK, b1 = (min(tile_start(a, tid + 1), a.V) + BLOCK - 1) / BLOCK;
    float mx = kLowest, sum = 0.f;
    for (int b = b0; b < b1; ++b) mx = fmaxf(mx, blocks[b].x);
    for (int b = b0; b < b1; ++b) sum += blocks[b].y * exp2f((blocks[b].x - mx) * kLog2e);
    runs[tid] = make_float2(mx, sum);
  }
  __syncthreads();
  if (tid < kWave) row_lse_draft<4>(a, r, runs, tile_mass, nullptr);
}

// ---------------------------------------------------------------------------------------------
// Final phase for one sequence (one workgroup): residual sample, commit, mask update, LowConf.
// ---------------------------------------------------------------------------------------------

// rm_pre: (wavefront 0 only) the residual chunk masses of this sequence, 16 per lane, loaded by the
// caller before the accept-phase results were known; valid if have_pre.  s_conf, s_mask, s_cand: the
// block state before the round, my_pos: slot_pos of slot tid, pass: seq_pass of the sequence, likewise;
// my_u: the residual uniform of slot tid (threads below K).
__device__ void finalize_sequence(const VerifyArgs& a, int b, const SeqState& st, BlockTmp& tmp,
                                  float* s_conf, uint8_t* s_mask, uint8_t* s_cand, const float (&rm_pre)[16],
                                  bool have_pre, int my_pos, int pass, float my_u) {
  const int tid = threadIdx.x;
  const int BK = a.B * a.K;
  const int window = st.window, acc_len = st.acc_len;

  // Diagnostics: overlap and residual mass of every slot, one wavefront per slot, eight loads of each in flight (27 -> 13 us
  // at 64 sequences x 16 slots of 494 chunks against a workgroup sum per slot).  A residual mass that is the small difference
  // of two laws shows the order of its terms: 256 chains over the chunks, 64 of them added at a time, four such sums in
  // order, as a workgroup adds them.
  if (a.all_slots) {
    const int lane = tid & 63;
    for (int m = tid >> 6; m < a.K; m += NW) {
      float al = 0.f, rm = 0.f;
      if (m < window) {
        const float* A = a.amass + (size_t)(b * a.K + m) * a.nRC;
        const float* R = a.rmass + (size_t)(b * a.K + m) * a.nRC;
        float as[4] = {0.f, 0.f, 0.f, 0.f}, rs[4] = {0.f, 0.f, 0.f, 0.f};
        for (int c0 = lane; c0 < a.nRC; c0 += 8 * kWave) {
          float x[8], y[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int c = c0 + j * kWave;
            x[j] = c < a.nRC ? A[c] : 0.f;
            y[j] = c < a.nRC ? R[c] : 0.f;
          }
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            as[j & 3] += x[j];
            rs[j & 3] += y[j];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          al += wave_sum(as[j]);
          rm += wave_sum(rs[j]);
        }
      }
      if (lane == 0) {
        if (a.diag_alpha) a.diag_alpha[b * a.K + m] = al;
        if (a.diag_resid_mass) a.diag_resid_mass[b * a.K + m] = rm;
      }
    }
  }

  // corrected token at the first rejection
  int z = -1;
  float z_conf = 0.f;
  if (acc_len < window) {
    const int s = b * a.K + acc_len;
    const float* Lq = a.logits + (size_t)s * a.ldl;
    const float* Lp = a.logits + (size_t)(BK + s) * a.ldl;
    // log-sum-exps, position and target arg max of the rejected slot travel with the accept-phase
    // results, so nothing here waits for a load whose address depends on acc_len except the logits
    const float lse_q = st.rej_lse_q, lse_p = st.rej_lse_p;
    const float* rm = a.rmass + (size_t)(a.all_slots ? s : b) * a.nRC;
    if (tid == acc_len) tmp.bcast_u = my_u;
    __syncthreads();
    const float u = tmp.bcast_u;
    if (a.greedy) {
      z = st.rej_xtarget;  // residual of two point masses: the target's
      z_conf = expf(Lp[z] - lse_p);
    } else if (a.nRC <= kWave * kChunkPer) {
      // one wavefront, everything in registers
      if (tid < kWave) {
        float rmv[kChunkPer];
#pragma unroll
        for (int j = 0; j < kChunkPer; ++j) {
          const int c = tid * kChunkPer + j;
          rmv[j] = have_pre ? rm_pre[j] : (c < a.nRC ? rm[c] : 0.f);
        }
        const Found chunk = wave_find_first_reg<kChunkPer, true>(rmv, u);
        int zz;
        float zc;
        if (chunk.total > 0.f) {
          const int v0 = chunk.idx * kResidChunk + tid * 4;
          float qv[4] = {0.f, 0.f, 0.f, 0.f}, pv[4] = {0.f, 0.f, 0.f, 0.f};
          if (v0 + 3 < a.V) {
            const float4 q4 = *reinterpret_cast<const float4*>(Lq + v0);
            const float4 p4 = *reinterpret_cast<const float4*>(Lp + v0);
            qv[0] = q4.x; qv[1] = q4.y; qv[2] = q4.z; qv[3] = q4.w;
            pv[0] = p4.x; pv[1] = p4.y; pv[2] = p4.z; pv[3] = p4.w;
          } else {
            for (int j = 0; j < 4; ++j)
              if (v0 + j < a.V) { qv[j] = Lq[v0 + j]; pv[j] = Lp[v0 + j]; }
          }
          float rv[4], pe[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            pe[j] = expf(pv[j] - lse_p);
            rv[j] = v0 + j < a.V ? fmaxf(pe[j] - expf(qv[j] - lse_q), 0.f) : 0.f;
          }
          const Found in = wave_find_first_reg<4>(rv, u * chunk.total - chunk.before);
          zz = chunk.idx * kResidChunk + in.idx;
          // pi(z) from the lane that holds token z: no second trip to memory
          const int j = in.idx & 3;
          const float mine = j == 0 ? pe[0] : j == 1 ? pe[1] : j == 2 ? pe[2] : pe[3];
          zc = __shfl(mine, in.idx >> 2, 64);
        } else {
          // residual mass vanished in rounding although a rejection occurred: commit argmax pi
          float best = -INFINITY;
          int bi = INT_MAX;
          for (int v = tid; v < a.V; v += kWave) {
            const float l = Lp[v];
            if (l > best) { best = l; bi = v; }
          }
          const float gbest = wave_max(best);
          zz = wave_min_int(best == gbest ? bi : INT_MAX);
          zc = expf(Lp[zz] - lse_p);
        }
        if (tid == 0) { tmp.bcast_i = zz; tmp.bcast_f = zc; }
      }
      __syncthreads();
      z = tmp.bcast_i;
      z_conf = tmp.bcast_f;
    } else {
    float Z = 0.f;
    {
      const int per = (a.nRC + NT - 1) / NT;
      const int begin = min(a.nRC, tid * per), end = min(a.nRC, begin + per);
      float local = 0.f;
      for (int c = begin; c < end; ++c) local += rm[c];
      block_exclusive_scan(local, tmp, Z);
    }
    if (Z > 0.f) {
      const float target = u * Z;
      const Found chunk = block_find_first(a.nRC, [&](int c) { return rm[c]; }, target, tmp);
      const int v0 = chunk.idx * kResidChunk;
      const int nv = min(kResidChunk, a.V - v0);
      const Found in = block_find_first(
          nv,
          [&](int i) {
            return fmaxf(expf(Lp[v0 + i] - lse_p) - expf(Lq[v0 + i] - lse_q), 0.f);
          },
          target - chunk.before, tmp);
      z = v0 + in.idx;
    } else {
      // residual mass vanished in rounding although a rejection occurred: commit argmax pi
      float best = -INFINITY;
      int bi = INT_MAX;
      for (int v = tid; v < a.V; v += NT) {
        const float l = Lp[v];
        if (l > best) { best = l; bi = v; }
      }
      const float gbest = block_max(best, tmp);
      z = block_min_int(best == gbest ? bi : INT_MAX, tmp);
    }
    z_conf = expf(Lp[z] - lse_p);
    }
  }

  // commit tokens and confidences
  const int committed = min(acc_len + 1, window);
  if (tid < a.K) {
    const int s = b * a.K + tid;
    int tok = -1;
    float c = 0.f;
    if (tid < acc_len) { tok = st.x[tid]; c = st.ptok[tid]; }
    else if (tid == acc_len && acc_len < window) { tok = z; c = z_conf; }
    a.out_tokens[s] = tok;
    if (a.diag_conf_tok) a.diag_conf_tok[s] = c;
  }
  if (tid == 0) a.out_accept_len[b] = acc_len;

  // block state: mask, pass set, confidences
  const size_t row = (size_t)b * a.block;
  if (tid < committed) {
    s_mask[my_pos] = 0;
    s_cand[my_pos] = 1;
    s_conf[my_pos] = (tid < acc_len) ? st.ptok[tid] : z_conf;
  }
  __syncthreads();
  int unresolved = 0;
  for (int i = tid; i < a.block; i += NT) unresolved |= s_mask[i];
  unresolved = block_max_int(unresolved, tmp);

  const bool final = a.seq_pass ? pass >= a.n_pass - 1 : a.final_pass != 0;
  const bool fire = !unresolved && !final;
  int remasked = 0;
  if (fire) {
    // LowConf: rank every candidate by (confidence, position); the n_rm lowest are re-masked
    const int n_rm = a.n_rm < 0 ? a.block / 2 : a.n_rm;
    for (int i = tid; i < a.block; i += NT) {
      const bool cand_i = a.lowconf_scope ? true : (s_cand[i] != 0);
      if (!cand_i) continue;
      const float ci = s_conf[i];
      int rank = 0;
      for (int j = 0; j < a.block; ++j) {
        const bool cand_j = a.lowconf_scope ? true : (s_cand[j] != 0);
        const float cj = s_conf[j];
        rank += (cand_j && (cj < ci || (cj == ci && j < i))) ? 1 : 0;
      }
      if (rank < n_rm) {
        // absorbing forward kernel: back to MASK with probability recorrupt_prob, else the
        // position keeps its token (both sides of u < prob are exact binary32 numbers)
        bool to_mask = true;
        if (a.recorrupt_prob < 1.f)
          to_mask = philox_uniform(a.seed, a.pos_base + (uint32_t)i, a.step, a.seq_base + (uint32_t)b,
                                   kStreamRecorrupt) < a.recorrupt_prob;
        if (to_mask) s_mask[i] = 1;
      }
    }
    __syncthreads();
    for (int i = tid; i < a.block; i += NT) remasked |= s_mask[i];
    remasked = block_max_int(remasked, tmp);
  }
  if (a.tokens_state && tid < committed)
    a.tokens_state[row + my_pos] = tid < acc_len ? st.x[tid] : z;
  __syncthreads();  // the token writes precede the -1s
  for (int i = tid; i < a.block; i += NT) {
    a.out_remask[row + i] = s_mask[i];
    if (a.pass_mask) a.pass_mask[row + i] = fire ? 0 : s_cand[i];
    if (a.conf) a.conf[row + i] = s_conf[i];
    if (a.tokens_state && fire && s_mask[i]) a.tokens_state[row + i] = -1;
  }
  if (tid == 0) {
    if (a.seq_pass) {
      if (fire && remasked) a.seq_pass[b] = pass + 1;
      else if (!unresolved) a.seq_pass[b] = a.n_pass;  // final pass resolved, or nothing left to redo
    }
    if (a.seq_rounds && window > 0) a.seq_rounds[b] += 1;
  }
}

// ---------------------------------------------------------------------------------------------
// Accept tests and first rejection of sequence b, by one whole wavefront; results in st (LDS).
// ---------------------------------------------------------------------------------------------
__device__ inline void accept_tests(const VerifyArgs& a, int b, SeqState& st) {
  const int lane = threadIdx.x & 63;
  const int BK = a.B * a.K;
  // everything whose address is known up front is requested together (slots beyond the window
  // hold x = -1 and are not used); only the two gathers at x~ wait for a previous load
  const int window = a.window[b];
  const int sl = b * a.K + min(lane, a.K - 1);
  const int x = a.xdraft[sl], pos = a.slot_pos[sl];
  const float lse_q = a.lse[sl], lse_p = a.lse[BK + sl];
  const int xt = a.greedy ? a.xtarget[sl] : -1;
  bool rejected = false;
  if (lane < window) {
    const float lq = a.logits[(size_t)sl * a.ldl + x] - lse_q;
    const float lp = a.logits[(size_t)(BK + sl) * a.ldl + x] - lse_p;
    const float ratio = fminf(1.f, expf(lp - lq));
    const float u = philox_uniform(a.seed, a.pos_base + (uint32_t)pos, a.step,
                                   a.seq_base + (uint32_t)b, kStreamAccept);
    // greedy: the ratio of the two point masses is 1 if the arg maxes agree, else 0
    rejected = a.greedy ? x != xt : !(u <= ratio);
    st.x[lane] = x;
    st.ptok[lane] = expf(lp);
  }
  const unsigned long long rej = __ballot(rejected);
  const int acc = rej ? __ffsll((long long)rej) - 1 : window;
  if (lane == 0) {
    st.window = window;
    st.acc_len = acc;
  }
  if (lane == acc && acc < window) {  // the rejected slot's own values, for the final phase
    st.rej_lse_q = lse_q;
    st.rej_lse_p = lse_p;
    st.rej_pos = pos;
    st.rej_xtarget = xt;
  }
}

// Four logits of each of the two rows of a slot, from token v on (zero past V).  ONCE: in non-temporal loads.
struct Quad {
  float q[4], p[4];
};
template <bool ONCE = false>
__device__ inline Quad load_quad(const VerifyArgs& a, const float* Lq, const float* Lp, int v) {
  Quad r;
  if (v + 3 < a.V) {
    const auto load = [](const float* p) {
      const floatx4* at = reinterpret_cast<const floatx4*>(p);
      return ONCE ? __builtin_nontemporal_load(at) : *at;
    };
    const floatx4 q4 = load(Lq + v), p4 = load(Lp + v);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      r.q[j] = q4[j];
      r.p[j] = p4[j];
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      r.q[j] = v + j < a.V ? Lq[v + j] : 0.f;
      r.p[j] = v + j < a.V ? Lp[v + j] : 0.f;
    }
  }
  return r;
}
// Residual mass (and, if asked for, overlap mass) of a chunk whose four tokens from v on this lane holds.
__device__ inline float chunk_mass(const VerifyArgs& a, const Quad& x, int v, float lse_q, float lse_p, float* overlap) {
  float rs = 0.f, as = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (v + j < a.V) {
      const float q = expf(x.q[j] - lse_q), p = expf(x.p[j] - lse_p);
      rs += fmaxf(p - q, 0.f);
      as += fminf(p, q);
    }
  }
  if (overlap) *overlap = wave_sum(as);
  return wave_sum(rs);
}

// ---------------------------------------------------------------------------------------------
// Kernel 2: accept tests, first rejection, residual mass per chunk of the rejected slot.
// grid = (B, ceil(nRC / NW)).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(NT) void accept_resid_kernel(VerifyArgs a) {
  __shared__ SeqState st;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x;   // sequence
  const int cg = blockIdx.y;  // chunk group
  if (wave == 0) accept_tests(a, b, st);
  __syncthreads();
  if (cg == 0 && tid < (int)(sizeof(SeqState) / 4))
    reinterpret_cast<int*>(a.seqstate + b)[tid] = reinterpret_cast<const int*>(&st)[tid];
  const int c = cg * NW + wave;
  // not needed when nothing was rejected, or in the greedy variant (the corrected token is the target arg max)
  if (st.acc_len < st.window && c < a.nRC && !a.greedy) {
    const size_t s = (size_t)b * a.K + st.acc_len;
    const int v = c * kResidChunk + lane * 4;
    const Quad x = load_quad(a, a.logits + s * a.ldl, a.logits + (s + (size_t)a.B * a.K) * a.ldl, v);
    const float rs = chunk_mass(a, x, v, st.rej_lse_q, st.rej_lse_p, nullptr);
    if (lane == 0) a.rmass[(size_t)b * a.nRC + c] = rs;
  }
}

// ---------------------------------------------------------------------------------------------
// Kernel 2 of a call that wants the masses of every slot: residual and overlap mass per chunk.
// grid = (B*K, ceil(nRC / (NW * kMassPer))), both capped; a wavefront takes kMassPer neighbouring chunks and asks
// for all of them before it uses the first.  Bound: the two passes' worth of exponentials and one read of all logits
// (1.04 GB at 64 x 16 slots, V = 126464).  Which slot was rejected does not matter here, so nothing waits for the
// accept tests (the final kernel does them); with them repeated in front of every chunk this took 260 us, without them 191, and
// 167 (6.2 TB/s) with non-temporal loads: the logits are read once (per call 411 -> 393 us at 540 slots of V = 151936, 148 -> 134 at 512 of
// V = 50257).  Two chunks per wavefront; four leave a small call short of wavefronts (50.4 -> 49.1 us at 32 slots of V = 100003), one
// or two per mille behind at the large ones.  COPY: a call that wants the logits too gets them from here, where they are in
// registers: 122 -> 112 us per call of 128 rows of d = 1024, V = 126464 against a kernel that reads them once more, 106 -> 101 at
// V = 100003, and a launch less (51.2 -> 50.0 at 32 fp32 rows of V = 32000).
// ---------------------------------------------------------------------------------------------
constexpr int kMassPer = 2;
template <bool COPY>
__device__ __forceinline__ void slot_masses(const VerifyArgs& a, int s, int c0) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, BK = a.B * a.K;
  const float* Lq = a.logits + (size_t)s * a.ldl;
  const float* Lp = a.logits + (size_t)(BK + s) * a.ldl;
  const int window = a.window[s / a.K];
  const float lse_q = a.lse[s], lse_p = a.lse[BK + s];
  Quad x[kMassPer];
#pragma unroll
  for (int j = 0; j < kMassPer; ++j) x[j] = load_quad<true>(a, Lq, Lp, (c0 + j) * kResidChunk + lane * 4);
  if constexpr (COPY) {
    // diagnostic logits: these rows without the padding, while they are in registers; of the target half of a split round
    // its own rows only
    float* Dq = a.diag_logits + (size_t)s * a.V;
    float* Dp = a.diag_logits + (size_t)(BK + s) * a.V;
    const bool quads = a.V % 4 == 0 && (reinterpret_cast<uintptr_t>(a.diag_logits) & 15) == 0, draft = a.row0 == 0;
#pragma unroll
    for (int j = 0; j < kMassPer; ++j) {
      const int v = (c0 + j) * kResidChunk + lane * 4;
      if (quads) {
        if (v < a.V) {
          if (draft) *reinterpret_cast<float4*>(Dq + v) = make_float4(x[j].q[0], x[j].q[1], x[j].q[2], x[j].q[3]);
          *reinterpret_cast<float4*>(Dp + v) = make_float4(x[j].p[0], x[j].p[1], x[j].p[2], x[j].p[3]);
        }
      } else {  // 256 neighbouring bytes per store instruction, through this wavefront's slice of LDS
        __shared__ __attribute__((aligned(16))) float turn[COPY ? NW : 1][2][kResidChunk];
        float(&t)[2][kResidChunk] = turn[wave];
        *reinterpret_cast<float4*>(&t[0][lane * 4]) = make_float4(x[j].q[0], x[j].q[1], x[j].q[2], x[j].q[3]);
        *reinterpret_cast<float4*>(&t[1][lane * 4]) = make_float4(x[j].p[0], x[j].p[1], x[j].p[2], x[j].p[3]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // same wavefront on both sides: order only
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int w = (c0 + j) * kResidChunk + i * kWave + lane;
          if (w < a.V) {
            if (draft) Dq[w] = t[0][i * kWave + lane];
            Dp[w] = t[1][i * kWave + lane];
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
      }
    }
  }
  if (s % a.K >= window) return;
#pragma unroll
  for (int j = 0; j < kMassPer; ++j) {
    if (c0 + j >= a.nRC) break;
    float as;
    const float rs = chunk_mass(a, x[j], (c0 + j) * kResidChunk + lane * 4, lse_q, lse_p, &as);
    if (lane == 0) {
      a.rmass[(size_t)s * a.nRC + c0 + j] = rs;
      a.amass[(size_t)s * a.nRC + c0 + j] = as;
    }
  }
}

// MANY: slots that would be 2^32 threads, of which a launch runs only a part, or more groups of chunks than a grid is high.  (The loops cost
// the ordinary call 2 us of 167.)
constexpr int kMassSlots = 1 << 23, kMassGroups = 65535;
template <bool COPY, bool MANY>
__global__ __launch_bounds__(NT) void slot_mass_kernel(VerifyArgs a) {
  const int c = (blockIdx.y * NW + (threadIdx.x >> 6)) * kMassPer;
  if constexpr (MANY) {
    for (int s = blockIdx.x; s < a.B * a.K; s += kMassSlots)
      for (int c0 = c; c0 < a.nRC; c0 += kMassGroups * NW * kMassPer) slot_masses<COPY>(a, s, c0);
  } else if (c < a.nRC) {
    slot_masses<COPY>(a, blockIdx.x, c);
  }
}

template <bool COPY>
void launch_slot_masses(const VerifyArgs& a) {
  const int slots = a.B * a.K, groups = (a.nRC + NW * kMassPer - 1) / (NW * kMassPer);
  const dim3 grid(slots < kMassSlots ? slots : kMassSlots, groups < kMassGroups ? groups : kMassGroups);
  if (slots > kMassSlots || groups > kMassGroups) hipLaunchKernelGGL((slot_mass_kernel<COPY, true>), grid, dim3(NT), 0, a.stream, a);
  else hipLaunchKernelGGL((slot_mass_kernel<COPY, false>), grid, dim3(NT), 0, a.stream, a);
}

// ---------------------------------------------------------------------------------------------
// Kernel 3: residual sample, commit, mask update, LowConf.  One workgroup per sequence.
//   kHandoff  the accept tests and the chunk masses come from kernel 2
//   kSlots    the chunk masses of every slot come from kernel 2, the accept tests are done here
//   kAlone    both are done here: a vocabulary of at most kAloneChunks chunks is not worth a launch
//             of its own (tiny vocabulary, 1 sequence: 2.6 + 5.2 us in two kernels, 5.5 in one), and
//             the greedy variant needs no masses at all
// ---------------------------------------------------------------------------------------------
enum FinalMode { kHandoff, kSlots, kAlone };
constexpr int kAloneChunks = 16;

template <FinalMode MODE>
__device__ __forceinline__ void finalize_round(const VerifyArgs& a, int b) {
  __shared__ BlockTmp tmp;
  __shared__ SeqState st;
  __shared__ float s_conf[kMaxBlock];
  __shared__ uint8_t s_mask[kMaxBlock], s_cand[kMaxBlock];
  __shared__ float s_mass[MODE == kAlone ? kAloneChunks : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  int word = 0;
  if (MODE == kHandoff && tid < (int)(sizeof(SeqState) / 4)) word = reinterpret_cast<const int*>(a.seqstate + b)[tid];
  // Without the diagnostics the chunk masses of a sequence sit at an address that does not depend
  // on which slot was rejected: wavefront 0 asks for them in the same breath as the accept-phase
  // results (when nothing was rejected they are stale and unused).  So does everybody for the block state.
  float rm_pre[kChunkPer];
  const bool have_pre = MODE == kAlone || (MODE == kHandoff && !a.greedy && a.nRC <= kWave * kChunkPer);
#pragma unroll
  for (int j = 0; j < kChunkPer; ++j) {
    const int c = tid * kChunkPer + j;
    rm_pre[j] = (MODE == kHandoff && have_pre && tid < kWave && c < a.nRC) ? a.rmass[(size_t)b * a.nRC + c] : 0.f;
  }
  const int my_pos = tid < a.K ? a.slot_pos[b * a.K + tid] : 0;
  const int pass = a.seq_pass ? a.seq_pass[b] : 0;
  const size_t row = (size_t)b * a.block;
  for (int i = tid; i < a.block; i += NT) {
    const uint8_t mask = a.mask_in ? (a.mask_in[row + i] != 0) : 1;
    const uint8_t cand = a.pass_mask ? (a.pass_mask[row + i] != 0) : 0;
    const float conf = a.conf ? a.conf[row + i] : 0.f;
    s_mask[i] = mask;
    s_cand[i] = cand;
    s_conf[i] = conf;
  }
  // drawn for every slot while the loads above are on their way
  const float my_u = tid < kWave ? philox_uniform(a.seed, a.pos_base + (uint32_t)my_pos, a.step, a.seq_base + (uint32_t)b,
                                                  kStreamResidual)
                                 : 0.f;
  if (MODE == kHandoff) {
    if (tid < (int)(sizeof(SeqState) / 4)) reinterpret_cast<int*>(&st)[tid] = word;
  } else if (tid < kWave) {
    accept_tests(a, b, st);
  }
  __syncthreads();
  if (MODE == kAlone && st.acc_len < st.window && !a.greedy) {
    const size_t s = (size_t)b * a.K + st.acc_len;
    for (int c = tid >> 6; c < a.nRC; c += NW) {
      const int v = c * kResidChunk + lane * 4;
      const Quad x = load_quad(a, a.logits + s * a.ldl, a.logits + (s + (size_t)a.B * a.K) * a.ldl, v);
      const float rs = chunk_mass(a, x, v, st.rej_lse_q, st.rej_lse_p, nullptr);
      if (lane == 0) s_mass[c] = rs;
    }
    __syncthreads();  // uniform: st is the workgroup's
#pragma unroll
    for (int j = 0; j < kChunkPer; ++j) {
      const int c = tid * kChunkPer + j;
      if (c < a.nRC) rm_pre[j] = s_mass[c];
    }
  }
  finalize_sequence(a, b, st, tmp, s_conf, s_mask, s_cand, rm_pre, have_pre, my_pos, pass, my_u);
}

template <FinalMode MODE>
__global__ __launch_bounds__(NT) void finalize_kernel(VerifyArgs a) {
  finalize_round<MODE>(a, blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// A whole round of a toy model in one launch: one workgroup per sequence takes its 2 K <= 16 rows through the fp32 head, a wavefront
// per row, and the final phase.  Bound: start-up, code that arrives from a cold instruction cache, and trips to memory that wait for one
// another; with three kernels each has its own, and what they hand on goes through memory.  Here logits, partials, log-sum-exps and
// draft tokens stay in LDS: the sequence is a batch of one whose workspace is this workgroup's LDS.  Per call, calls queued one
// behind another, three machines: 4 tokens of a toy model (d = 64, V = 32) 13.4 to 16.0 -> 9.7 to 11.3 us (the host's 8 are next),
// 8 tokens of d = 128, V = 256 16.0 -> 12.7 to 14.5, 64 sequences of d = 64, V = 256 17.6 -> 12.6 to 13.3.  Four or eight wavefronts are
// slower (12.4, 12.8 at V = 32, still through memory, against 10.8), and so is handing on through memory (11.7).
// ---------------------------------------------------------------------------------------------
constexpr int kToyWaves = 16, kToyTokens = 16 * kToyWaves;

template <int VEC>
__global__ __launch_bounds__(kToyWaves * kWave) void toy_round_kernel(HeadArgs h, VerifyArgs a) {
  __shared__ __attribute__((aligned(16))) float ring[f32_ring_floats<kToyWaves, 16, VEC, 32>()];
  __shared__ __attribute__((aligned(16))) float logits[16][kToyTokens];
  __shared__ float tile_max[16][kToyWaves];
  __shared__ float2 partials[16 * (kToyTokens / kTiledTn)];
  __shared__ float lse[16];
  __shared__ int32_t xdraft[8], xtarget[8], slot_pos[8], window;
  const int b = blockIdx.x, K = a.K, wave = threadIdx.x >> 6;
  const size_t slot = (size_t)b * K, position = (size_t)b * a.block;

  const float* hd = (const float*)h.h_draft + slot * h.d;
  const float* ht = (const float*)h.h_target + slot * h.d - (size_t)K * h.d;
  const auto h_of = [=](int m) { return (m < K ? hd : ht) + (size_t)m * h.d; };
  f32_tile<kToyWaves, 16, VEC, 32, false, false>(h, 0, 0, 2 * K, h_of, &logits[0][0], kToyTokens, partials, ring, tile_max);

  float* diag_lse = a.diag_lse;
  const int BK = a.B * K;
  auto move = [](auto*& p, size_t by) __attribute__((always_inline)) { if (p) p += by; };
  a.B = 1;
  a.nrows = 2 * K;
  a.seq_base += (uint32_t)b;
  a.logits = &logits[0][0];
  a.ldl = kToyTokens;
  a.partials = partials;
  a.lse = lse;
  a.xdraft = xdraft;
  a.xtarget = xtarget;
  a.slot_pos = slot_pos;
  a.window = &window;
  a.diag_lse = nullptr;
  move(a.mask_in, position);
  move(a.pass_mask, position);
  move(a.conf, position);
  move(a.tokens_state, position);
  a.out_remask += position;
  move(a.draft_tokens_in, slot);
  a.out_tokens += slot;
  move(a.diag_draft_tokens, slot);
  move(a.diag_conf_tok, slot);
  a.out_accept_len += b;
  move(a.seq_pass, b);
  move(a.seq_rounds, b);
  if (wave < 2 * K) {
    row_lse_draft<4>(a, wave, partials + wave * a.nT, ring + wave * (4 * kWave), nullptr);
    if (diag_lse && (threadIdx.x & 63) == 0) diag_lse[wave < K ? slot + wave : BK + slot + wave - K] = lse[wave];
  }
  __syncthreads();
  if (wave < NW) finalize_round<kAlone>(a, 0);  // the other wavefronts end; barriers count the ones that are left
}

// ---------------------------------------------------------------------------------------------
// Baseline step (parallel prediction with top-n confidence transfer): after kernel 1 has drawn a
// token for every window slot, one wavefront per sequence takes the confidences p(x) and commits
// the n most confident slots (equal confidences: the lower position first).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kWave) void topn_kernel(VerifyArgs a) {
  // everything whose address is known up front is requested together; only the gather at x waits for a load
  const int b = blockIdx.x, lane = threadIdx.x;
  const int s = b * a.K + lane, sl = b * a.K + min(lane, a.K - 1);
  const int window = a.window[b];
  int x = a.xdraft[sl], pos = a.slot_pos[sl];
  const float lse = a.lse[sl];
  const size_t row = (size_t)b * a.block;
  for (int i = lane; i < a.block; i += kWave) a.out_remask[row + i] = a.mask_in ? (a.mask_in[row + i] != 0) : 1;
  const bool live = lane < window;
  float c = -1.f;
  if (live) {
    c = expf(a.logits[(size_t)s * a.ldl + x] - lse);
  } else {
    x = -1;
    pos = INT_MAX;
  }
  int rank = 0;
  for (int j = 0; j < window; ++j) {  // j is the same in every lane: v_readlane, no trip through the LDS crossbar
    const float cj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, c), j));
    const int pj = __builtin_amdgcn_readlane(pos, j);
    rank += (cj > c || (cj == c && pj < pos)) ? 1 : 0;
  }
  const bool commit = live && rank < a.n_transfer;
  if (lane < a.K) {
    a.out_tokens[s] = commit ? x : -1;
    if (a.diag_conf_tok) a.diag_conf_tok[s] = live ? c : 0.f;
  }
  if (lane == 0) a.out_accept_len[b] = min(a.n_transfer, window);
  __syncthreads();  // one wavefront: orders the mask copy before the committed positions are cleared
  if (commit) {
    a.out_remask[row + pos] = 0;
    if (a.conf) a.conf[row + pos] = c;
    if (a.tokens_state) a.tokens_state[row + pos] = x;
  }
}

// Logits without the padding of the workspace rows, for calls without slot_mass_kernel.  grid = (rows, pieces of kCopyPer tokens),
// the rows capped (a launch has less than 2^32 threads, a call up to 2^25 rows); a thread asks for all of its eight elements before
// it stores the first.  (One flat index divided by V per element before: 131 -> 122 us per call of 128 rows of V = 126464, d = 1024,
// that keeps its logits.)
constexpr int kCopyPer = 8 * NT;
__global__ __launch_bounds__(NT) void copy_logits_kernel(const float* __restrict__ src, long ldl, float* __restrict__ dst, int V, int rows) {
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    const float* s = src + (size_t)r * ldl;
    float* d = dst + (size_t)r * V;
    for (long v0 = (long)blockIdx.y * kCopyPer + threadIdx.x; v0 < V; v0 += (long)gridDim.y * kCopyPer) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = v0 + j * NT < V ? s[v0 + j * NT] : 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (v0 + j * NT < V) d[v0 + j * NT] = x[j];
    }
  }
}

// Diagnostic logits of a call without slot_mass_kernel.
hipError_t launch_copy(const VerifyArgs& a) {
  if (a.diag_logits && (!a.all_slots || a.phase == 1 || a.phase == 3)) {
    const long pieces = (a.V + (long)kCopyPer - 1) / kCopyPer;
    hipLaunchKernelGGL(copy_logits_kernel, dim3(a.nrows < 1 << 20 ? a.nrows : 1 << 20, pieces < 65535 ? pieces : 65535), dim3(NT), 0,
                       a.stream, a.logits + (size_t)a.row0 * a.ldl, a.ldl, a.diag_logits + (size_t)a.row0 * a.V, a.V, a.nrows);
  }
  return hipGetLastError();
}

}  // namespace

// Up to 16 rows per sequence and 256 tokens, which is one pass of the workgroup's wavefronts; up to one sequence per CU (at 512 sequences of
// d = 64, V = 128 18 us in three kernels, 24 in one); and hidden sizes up to which one CU's matrix units are not what it costs (V = 256:
// 16.0 against 14.5 us at d = 192, 16.1 against 16.3 at d = 256).
bool toy_round_serves(int B, int K, int d, int V) { return B <= 256 && 2 * K <= 16 && V <= kToyTokens && d <= 192; }

hipError_t launch_toy_round(const HeadArgs& h, const VerifyArgs& a) {
  if (h.d % 4 == 0) hipLaunchKernelGGL(toy_round_kernel<4>, dim3(a.B), dim3(kToyWaves * kWave), 0, a.stream, h, a);
  else hipLaunchKernelGGL(toy_round_kernel<1>, dim3(a.B), dim3(kToyWaves * kWave), 0, a.stream, h, a);
  return hipGetLastError();
}

hipError_t launch_verify(const VerifyArgs& a) {
  const dim3 g1((a.nrows + NW - 1) / NW);
  if (a.row_sums == 64) hipLaunchKernelGGL(row_sums_draft_kernel<64>, dim3(a.nrows), dim3(kSumThreads), 0, a.stream, a);
  else if (a.row_sums) hipLaunchKernelGGL(row_sums_draft_kernel<16>, dim3(a.nrows), dim3(kSumThreads), 0, a.stream, a);
  else if (a.nT <= 64 * 4) hipLaunchKernelGGL(row_lse_draft_kernel<4>, g1, dim3(NT), 0, a.stream, a);
  else if (a.nT <= 64 * 8) hipLaunchKernelGGL(row_lse_draft_kernel<8>, g1, dim3(NT), 0, a.stream, a);
  else if (a.nT <= 64 * 10) hipLaunchKernelGGL(row_lse_draft_kernel<10>, g1, dim3(NT), 0, a.stream, a);  // V = 151936: 594 tiles
  else if (a.nT <= 64 * 40) hipLaunchKernelGGL(row_lse_draft_kernel<40>, g1, dim3(NT), 0, a.stream, a);
  else hipLaunchKernelGGL(row_lse_draft_kernel<0>, g1, dim3(NT), 0, a.stream, a);
  if (a.phase == 3) {
    hipLaunchKernelGGL(topn_kernel, dim3(a.B), dim3(kWave), 0, a.stream, a);
  } else if (a.phase != 1) {  // everything after the draft sample needs the target laws
    if (a.all_slots) {
      if (a.diag_logits) launch_slot_masses<true>(a);
      else launch_slot_masses<false>(a);
      hipLaunchKernelGGL(finalize_kernel<kSlots>, dim3(a.B), dim3(NT), 0, a.stream, a);
    } else if (a.nRC <= kAloneChunks || a.greedy) {
      hipLaunchKernelGGL(finalize_kernel<kAlone>, dim3(a.B), dim3(NT), 0, a.stream, a);
    } else {
      hipLaunchKernelGGL(accept_resid_kernel, dim3(a.B, (a.nRC + NW - 1) / NW), dim3(NT), 0, a.stream, a);
      hipLaunchKernelGGL(finalize_kernel<kHandoff>, dim3(a.B), dim3(NT), 0, a.stream, a);
    }
  }
  return launch_copy(a);
}

}  // namespace fef
