// Observation-window token scoring (the attention-based selection policy that the ablation of
// Sec. 4.4 runs under the LKV-H budgets; O(W T) in the complexity table of Sec. 4.5): a prefix
// token's score is the attention mass it receives from the last W queries of the prompt, summed
// over the window, averaged over the query heads of its GQA group and smoothed by a short 1-D
// pooling; the window tokens themselves score +inf.
//
// The work is one [G W x 128] x [128 x T] product per (layer, KV head) followed by a softmax over
// T, so the keys stream past the matrix cores exactly as they do for the MLP scorer: the G W
// window queries sit on the M side of v_mfma_f32_16x16x32_bf16 as register-resident A fragments,
// 16 keys at a time form the B operand, read once from HBM with coalesced 16-byte loads and
// staged in LDS.  A softmax needs its normaliser before any weight can be summed over the rows,
// so the keys are read twice:
//   pass 1  per window row, the log-sum-exp of its logits over one block's keys (causal inside
//           the window), written as a (reference, sum) pair per block;
//   merge   the pairs of all blocks of a head into each row's log-normaliser (a small kernel);
//   pass 2  recomputes the logits and adds exp(logit - normaliser) over the rows: the token's vote,
//           the two waves of a block adding their rows' shares in LDS; then the block takes the
//           group mean, smooths and writes the scores of its keys.  The pooling reaches into the
//           neighbouring blocks' keys, so a block also computes the votes of up to two tiles on
//           either side of its own (3 to 6 % more work, less than a pooling launch costs).
// Keeping the logits instead would cost as many bytes as reading the keys again (G W = 128
// logits per 128-element key).  A caller that still has the log-normalisers of the window rows
// (the prefill's attention kernel computes them for every query) passes them in: pass 1 and the
// merge are skipped and the keys are read once.
//
// Pass 1 takes its sums per (row, lane) relative to logits of the block's first 32 keys (that lane's own two, or the row's
// largest where some are not modest): any reference gives the same sum to fp32 rounding as long as nothing overflows, so nothing
// looks at a maximum.  A wave looks at its sums after 64 keys and then every 128; where some have grown their references
// follow by whole binary orders, and where one overflowed (a logit more than 2^7 binary orders above its reference) the keys
// since the last look are taken again with references that follow every key.  So the price of wide logits is bounded:
// 32 layers of 8 heads x 32768 keys, 128 window rows, logits of a deviation of 1, 8, 16 and 32: 867, 868, 921 and 1092 us with
// references that move tile by tile, 799, 818, 2045 and 2013 with whole blocks taken again beyond 2^100, 792, 804, 853 and
// 902 with this.
//
// A block is a pair of waves that share the staged keys (two tiles of 16 between barriers); the
// window rows are split between the two (at most 64 rows, 64 fragment registers, per wave).
// What bounds both passes: the keys' stream (341 us a pass of 2.1 GB at the 6.3 TB/s that a large read reaches here) and
// the issue of one exponential, a multiplication and an addition per logit next to the matrix work, in one power budget.  So what pays
// is work not done: references that stay put (no maximum and no vote on it), addresses from a scalar base, sums over
// the row blocks of both tiles at once.  32 layers of 8 heads x 32768 keys, 128 window rows, in turn with a kernel that moved its
// references: 908 -> 829 us on one machine, 852 -> 797 on another (given the normalisers 471 -> 439 and 434 -> 418); 4 x 7
// heads, 20001 keys, 8 layers 105 -> 99; one layer of 4097 28.2 -> 26.0.  Measured and dropped: keys straight from memory to LDS (a ring of four steps, 37 KB
// a block: too few bytes in flight, 433 -> 486 us a pass, 188 -> 216 with 8 window rows), temporal loads, and pass 2 from the
// last block backwards so that it finds the end of the keys in the memory-side cache (0 to 7 % slower).
#include "lkv_common.h"

namespace lkv {

constexpr int kWinThreads = 128;
constexpr int kWinTokTile = 16;                  // keys per MFMA N tile
constexpr int kWinRowStride = 256 + 32;          // bytes per staged key row in LDS
constexpr int kWinTileLds = kWinTokTile * kWinRowStride;
constexpr int kWinTilesPerStep = 2;     // tiles staged, multiplied and finished between two barriers
constexpr int kWinStep = kWinTilesPerStep * kWinTokTile;
constexpr int kWinStepLds = kWinTilesPerStep * kWinTileLds;
constexpr int kWinManyRounds = 1024;             // keys of a block where the blocks go round several times (see below)
constexpr int kWinMaxReach = 31;                // pooling widths up to 63
// pass 2: a block's keys, two tiles before, the reach after, rounded up to a tile
constexpr int win_vote_slots(int keys) { return keys + 32 + kWinMaxReach + 17; }
constexpr float kWinMoveSum = 4294967296.f;      // 2^32: sum over a lane's rows from which pass 1 moves its references
constexpr float kWinModest = 24.f;               // first logits (log2 units) up to which a lane's own serve as its references
constexpr int kWinMostOrders = 100;              // by which one goes at once (what is left of a sum stays far from underflow)
constexpr float kWinNoRef = -1e30f;              // reference of a row that has seen no key yet

// row / window, for the rows of a block, as row * win_turns(window) >> 16.  A step around the window asks for the place of every
// row in its head's window; as integer remainders those were some 2 us of a call: one layer of 8 heads, 128 window rows, 6001
// keys 33.0 -> 28.8 us, 12001 37.5 -> 33.7; 2 heads, 12001 keys 31.8 -> 27.3.
constexpr uint32_t win_turns(int window) { return (65535u + (uint32_t)window) / (uint32_t)window; }
constexpr bool win_turns_exact() {
  for (int w = 1; w <= 128; ++w)
    for (uint32_t row = 0; row < 128; ++row)
      if ((row * win_turns(w) >> 16) != row / (uint32_t)w) return false;
  return true;
}
static_assert(win_turns_exact(), "a quotient by multiplication");

__device__ __forceinline__ int win_seq_of_unit(const WinTable& tab, int unit) {
  int s = 0;
  while (s + 1 < tab.n && unit >= tab.first[s + 1]) ++s;
  return s;
}

__device__ __forceinline__ float row16_allreduce_max(float x) {
  x = fmaxf(x, dpp_f32<kDppQuadXor1>(x));
  x = fmaxf(x, dpp_f32<kDppQuadXor2>(x));
  x = fmaxf(x, dpp_f32<kDppRowHalfMirror>(x));
  x = fmaxf(x, dpp_f32<kDppRowMirror>(x));
  return x;
}

// kPass 1: partial log-sum-exp pairs.  kPass 2: votes (the merged normalisers are read from the
// workspace).  MTW: 16-row M tiles per wave; the rows past n_rows = G W are padding (zero queries,
// never counted).
template <int MTW, int kPass>
__global__ void __launch_bounds__(kWinThreads, 2)
score_window_kernel(WinTable tab, int heads, int window, int n_rows, int rows_per_block, float log2_scale,
                    int reach /* pass 2: pooling reach c, width 2 c + 1 */, int pool_kind, float inv_group) {
  constexpr int RP = 32 * MTW;                      // padded rows of the block
  __shared__ __align__(16) unsigned char x_lds[2 * kWinStepLds];   // the staged keys of two steps
  // pass 2: the votes of the keys the block multiplies (win_vote_slots of rows_per_block); both waves add the shares of their rows
  extern __shared__ float v_lds[];

  const int seq = win_seq_of_unit(tab, blockIdx.x);
  const int local = blockIdx.x - tab.first[seq];
  const int T = tab.T[seq];
  const int chunks = (T + rows_per_block - 1) / rows_per_block;
  const int lh = local / chunks;
  const int chunk = local - lh * chunks;
  const int prefix = T - window;                    // tokens that are scored

  // The block's own keys, and the keys it multiplies: in pass 2 also those within the pooling's reach on either
  // side (whole tiles before, single keys after), as far as they lie inside the prefix.
  const int own_row0 = chunk * rows_per_block;
  const int own_end = min(T, own_row0 + rows_per_block);
  const int block_end_all = kPass == 1 ? T : prefix;    // pass 2 has no votes to compute inside the window
  float* out = tab.scores[seq] + (size_t)lh * T;
  if (own_row0 >= block_end_all) {
    if (kPass == 2)   // a block of window tokens
      for (int j = own_row0 + (int)threadIdx.x; j < own_end; j += kWinThreads) out[j] = INFINITY;
    return;
  }
  const int halo = kPass == 2 ? ((reach + 15) >> 4) << 4 : 0;
  const int block_row0 = max(0, own_row0 - halo);
  const int block_end = kPass == 1 ? own_end : min(prefix, own_end + reach);
  const int block_rows = block_end - block_row0;

  const int lane = threadIdx.x & 63;
  const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int r = lane >> 4;
  const int c = lane & 15;
  if (kPass == 2)
    for (int i = threadIdx.x; i < block_rows; i += kWinThreads) v_lds[i] = 0.f;   // ordered by the barriers below

  // A fragments: window row 16 (half MTW + mw) + c, features 32 ks + 8 r .. +7
  bf16x8_t qfrag[MTW][4];
  {
    const uint4* qb = reinterpret_cast<const uint4*>(tab.q[seq]) + (size_t)lh * n_rows * kChunksPerRow;
#pragma unroll
    for (int mw = 0; mw < MTW; ++mw) {
      const int row = 16 * (half * MTW + mw) + c;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row < n_rows) v = qb[(size_t)row * kChunksPerRow + ks * 4 + r];
        qfrag[mw][ks] = __builtin_bit_cast(bf16x8_t, v);
      }
    }
  }

  // per lane: rows 16 (half MTW + mw) + 4 r + e of token c of the current tile
  float ref[MTW][4], sum[MTW][4];   // pass 1: reference (log2 units) and sum; pass 2: ref = log-normaliser
#pragma unroll
  for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
    for (int e = 0; e < 4; ++e) ref[mw][e] = sum[mw][e] = 0.f;

  const size_t part_row0 = ((size_t)lh * chunks) * RP;
  if (kPass == 2) {
    if (tab.lse[seq] != nullptr) {
      // the caller's log-normalisers (natural logarithm, one per window row of the group: what the prefill's
      // attention kernel already returns for these queries); padding rows get +inf, i.e. weight zero
      const float* lse = tab.lse[seq] + (size_t)lh * n_rows;
#pragma unroll
      for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = 16 * (half * MTW + mw) + 4 * r + e;
          ref[mw][e] = row < n_rows ? lse[row] * 1.44269504088896340736f : INFINITY;
        }
    } else {
      // log-normaliser of every row, merged from the pairs of pass 1 by the kernel in between
      const float* lse = tab.partial[seq] + (size_t)heads * chunks * RP * 2 + (size_t)lh * RP;
#pragma unroll
      for (int mw = 0; mw < MTW; ++mw) {
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(lse + 16 * (half * MTW + mw) + 4 * r);
#pragma unroll
        for (int e = 0; e < 4; ++e) ref[mw][e] = v[e];
      }
    }
  }

  const unsigned char* Kh = reinterpret_cast<const unsigned char*>(tab.k[seq]) + ((size_t)lh * (size_t)T + block_row0) * 256;

  // Staging: thread (half, r, c) brings piece c of rows 16 nt + 8 half + r and 16 nt + 8 half + 4 + r of each step.
  // No branch encloses a load between its issue and the staging that waits for it: the compiler counts the loads
  // still in flight at a wait from the path on which the fewest were issued, so a conditional load makes every wait
  // drain the whole queue.  Steps past the block's rows are clamped instead of skipped.
  const int n_steps = (block_rows + kWinStep - 1) / kWinStep;
  uint4 xa[2 * kWinTilesPerStep], xb[2 * kWinTilesPerStep];
  auto load_step = [&](uint4 (&xx)[2 * kWinTilesPerStep], int i) __attribute__((always_inline)) {
    const int at = min(i * kWinStep, block_rows - 1);   // past the last step: the last row only
    const unsigned char* src = Kh + (size_t)at * 256;
#pragma unroll
    for (int j = 0; j < 2 * kWinTilesPerStep; ++j) {
      // past the block's rows: its last row again, masked below
      const uint32_t row = (uint32_t)min(16 * (j >> 1) + 8 * half + 4 * (j & 1) + r, block_rows - 1 - at);
      xx[j] = load_stream16(reinterpret_cast<const uint4*>(src + (row * 256u + (uint32_t)c * 16u)));
    }
  };
  const uint32_t stage_at = (uint32_t)((8 * half + r) * kWinRowStride + c * 16);
  auto stage_step = [&](const uint4 (&xx)[2 * kWinTilesPerStep], int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2 * kWinTilesPerStep; ++j)
      *reinterpret_cast<uint4*>(x_lds + buf * kWinStepLds + stage_at + (16 * (j >> 1) + 4 * (j & 1)) * kWinRowStride) = xx[j];
  };
  const uint32_t read_at = (uint32_t)(c * kWinRowStride + r * 16);
  auto products = [&](f32x4_t (&acc)[MTW], const unsigned char* xt) __attribute__((always_inline)) {
#pragma unroll
    for (int mw = 0; mw < MTW; ++mw) acc[mw] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const bf16x8_t xv = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(xt + read_at + ks * 64));
#pragma unroll
      for (int mw = 0; mw < MTW; ++mw)
        acc[mw] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qfrag[mw][ks], xv, acc[mw], 0, 0, 0);
    }
  };
  // The last key that window row `row` sees: row i of a head's window sees those up to its own, rows past n_rows none.
  const uint32_t turns = win_turns(window);
  auto last_seen = [&](int row) __attribute__((always_inline)) {
    uint32_t n = turns;
    asm volatile("" : "+s"(n));   // or the compiler keeps every row's place in the window in registers all the way
    return row < n_rows ? prefix + row - (int)((uint32_t)row * n >> 16) * window : -1;
  };
  // One step: products and arithmetic of its two tiles, staging of step i + 1 (fetching step i + 3 behind it).  Barrier i
  // makes the keys of step i visible and means both waves have finished reading those of step i - 1.
  auto step = [&](uint4 (&x_next)[2 * kWinTilesPerStep], int i, int buf) __attribute__((always_inline)) {
    const unsigned char* cur = x_lds + buf * kWinStepLds;
    f32x4_t acc[2][MTW];
    products(acc[0], cur);
    products(acc[1], cur + kWinTileLds);
    stage_step(x_next, buf ^ 1);               // past the last step: rows nobody reads
    load_step(x_next, i + 3);
    if (kPass == 1) {
      const bool causal = block_row0 + kWinStep * (i + 1) > prefix;   // uniform: the step touches the window or the ragged tail
      if (causal) {
        const int j = block_row0 + kWinStep * i + c;
#pragma unroll
        for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int last = last_seen(16 * (half * MTW + mw) + 4 * r + e);
            if (j > last) acc[0][mw][e] = -INFINITY;
            if (j + kWinTokTile > last) acc[1][mw][e] = -INFINITY;
          }
      }
      if (i == 0) {   // uniform: the first references
        float most = 0.f;
#pragma unroll
        for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            ref[mw][e] = fmaxf(fmaxf(acc[0][mw][e], acc[1][mw][e]) * log2_scale, kWinNoRef);
            most = fmaxf(most, fabsf(ref[mw][e]));
          }
        if (__ballot(most > kWinModest) != 0ull) {
#pragma unroll
          for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
            for (int e = 0; e < 4; ++e) ref[mw][e] = row16_allreduce_max(ref[mw][e]);
        }
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[mw][e] += __builtin_amdgcn_exp2f(fmaf(acc[t][mw][e], log2_scale, -ref[mw][e]));
    } else {
      float part[2] = {0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
          for (int e = 0; e < 4; ++e) part[t] += __builtin_amdgcn_exp2f(fmaf(acc[t][mw][e], log2_scale, -ref[mw][e]));
      // sums over the row blocks of both tiles at once: the first tile's in lanes r = 0, 1, the second's in r = 2, 3
      const u32x2_swap_t a = __builtin_amdgcn_permlane32_swap(__float_as_uint(part[0]), __float_as_uint(part[1]), false, false);
      const float x = __uint_as_float(a.x) + __uint_as_float(a.y);
      const u32x2_swap_t b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      const int key = kWinStep * i + kWinTokTile * (r >> 1) + c;
      // two additions to a zero: the same sum whichever wave comes first
      if ((r & 1) == 0 && key < block_rows) atomicAdd(&v_lds[key], __uint_as_float(b.x) + __uint_as_float(b.y));
    }
    __syncthreads();
  };
  // Pass 1: a look at the sums, `upto` steps done.  Where some have grown, the references of their lanes follow by whole
  // binary orders; where one overflowed, the keys since the last look are taken again, straight from memory and with
  // references that follow every one of them.
  float kept_sum[MTW][4];   // as the last look left them
#pragma unroll
  for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
    for (int e = 0; e < 4; ++e) kept_sum[mw][e] = 0.f;
  int looked = 0;
  auto look = [&](int upto) __attribute__((always_inline)) {
    float total = 0.f;
#pragma unroll
    for (int mw = 0; mw < MTW; ++mw) total += (sum[mw][0] + sum[mw][1]) + (sum[mw][2] + sum[mw][3]);
    if (__builtin_expect(__ballot(!(total < kWinMoveSum)) != 0ull, 0)) {
      bool lost = false;
#pragma unroll
      for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
        for (int e = 0; e < 4; ++e) lost |= !(sum[mw][e] < INFINITY);
      if (__ballot(lost) != 0ull) {
#pragma unroll
        for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sum[mw][e] = kept_sum[mw][e];
            // the first references may be infinite (those of padding rows, which see no key, are not)
            if (looked == 0 && 16 * (half * MTW + mw) + 4 * r + e < n_rows) ref[mw][e] = kWinNoRef;
          }
#pragma unroll 1
        for (int row0 = looked * kWinStep; row0 < min(upto * kWinStep, block_rows); row0 += kWinTokTile) {
          f32x4_t acc[MTW];
#pragma unroll
          for (int mw = 0; mw < MTW; ++mw) acc[mw] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          const uint4* key = reinterpret_cast<const uint4*>(Kh + (size_t)min(row0 + c, block_rows - 1) * 256);
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const bf16x8_t xv = __builtin_bit_cast(bf16x8_t, key[ks * 4 + r]);
#pragma unroll
            for (int mw = 0; mw < MTW; ++mw)
              acc[mw] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qfrag[mw][ks], xv, acc[mw], 0, 0, 0);
          }
#pragma unroll
          for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const bool seen = block_row0 + row0 + c <= last_seen(16 * (half * MTW + mw) + 4 * r + e);
              const float s = acc[mw][e] * log2_scale;
              const float moved = fmaxf(ref[mw][e], s);
              const float kept = sum[mw][e] * __builtin_amdgcn_exp2f(ref[mw][e] - moved) + __builtin_amdgcn_exp2f(s - moved);
              sum[mw][e] = seen ? kept : sum[mw][e];
              ref[mw][e] = seen ? moved : ref[mw][e];
            }
        }
      } else {
#pragma unroll
        for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int orders = sum[mw][e] >= 1.f ? min(__builtin_amdgcn_frexp_expf(sum[mw][e]), kWinMostOrders) : 0;
            const float moved = ref[mw][e] + (float)orders;
            sum[mw][e] *= __builtin_amdgcn_exp2f(ref[mw][e] - moved);
            ref[mw][e] = moved;
          }
      }
    }
#pragma unroll
    for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
      for (int e = 0; e < 4; ++e) kept_sum[mw][e] = sum[mw][e];
    looked = upto;
  };
  load_step(xa, 0);
  load_step(xb, 1);
  stage_step(xa, 0);
  load_step(xa, 2);
  __syncthreads();
#pragma unroll 1
  for (int i = 0; i < n_steps; i += 2) {   // (no break: one way out of the loop keeps one set of sums)
    step(xb, i, 0);                        // stages the odd step i + 1
    if (i + 1 < n_steps) step(xa, i + 1, 1);
    if (kPass == 1 && ((i & 2) == 0 || i + 2 >= n_steps)) look(min(i + 2, n_steps));
  }

  if (kPass == 2) {
    // Scores of the block's own keys: centred pooling over the votes inside the prefix (votes are non-negative and
    // the slots outside hold zeros, which change neither rule), group mean, +inf on window tokens.
    const float inv_width = 1.f / (float)(2 * reach + 1);
    for (int j = own_row0 + (int)threadIdx.x; j < own_end; j += kWinThreads) {
      float sc = INFINITY;
      if (j < prefix) {
        const int lo = j - reach - block_row0;   // may be negative at the start of the head
        sc = 0.f;
        if (pool_kind == 0) {
          for (int u = 0; u <= 2 * reach; ++u) {
            const int t = lo + u;
            sc = fmaxf(sc, t >= 0 && t < block_rows ? v_lds[t] : 0.f);
          }
          sc *= inv_group;
        } else {
          for (int u = 0; u <= 2 * reach; ++u) {
            const int t = lo + u;
            sc += t >= 0 && t < block_rows ? v_lds[t] : 0.f;
          }
          sc *= inv_width * inv_group;
        }
      }
      out[j] = sc;
    }
  }
  if (kPass == 1) {
    // one (reference, sum) pair per row: merge the 16 token lanes
    float* part = tab.partial[seq] + (part_row0 + (size_t)chunk * RP) * 2;
#pragma unroll
    for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 16 * (half * MTW + mw) + 4 * r + e;
        const float mine = row < n_rows ? ref[mw][e] : kWinNoRef;
        const float m = row16_allreduce_max(mine);
        const float l = row16_allreduce_sum(sum[mw][e] * __builtin_amdgcn_exp2f(mine - m));
        if (c == 0) {
          part[row * 2] = m;
          part[row * 2 + 1] = l;
        }
      }
  }
}

// Between the passes: the log-normaliser (log2 units) of every window row of every head, from the pairs
// the blocks of pass 1 left; +inf for the padding rows, whose weights then vanish.  One block per head.
__global__ void __launch_bounds__(128)
score_window_merge_kernel(WinTable tab, int heads, int n_rows, int rows_per_block, int padded_rows) {
  const int seq = blockIdx.x / heads;
  const int lh = blockIdx.x - seq * heads;
  const int chunks = (tab.T[seq] + rows_per_block - 1) / rows_per_block;
  const float* part = tab.partial[seq] + (size_t)lh * chunks * padded_rows * 2;
  float* lse = tab.partial[seq] + (size_t)heads * chunks * padded_rows * 2 + (size_t)lh * padded_rows;
  const int row = threadIdx.x;
  if (row >= padded_rows) return;
  float out = INFINITY;
  if (row < n_rows) {
    const float2* pairs = reinterpret_cast<const float2*>(part) + row;
    float m = kWinNoRef;
#pragma unroll 8
    for (int ch = 0; ch < chunks; ++ch) m = fmaxf(m, pairs[(size_t)ch * padded_rows].x);
    float l = 0.f;
#pragma unroll 8
    for (int ch = 0; ch < chunks; ++ch) {
      const float2 p = pairs[(size_t)ch * padded_rows];
      l += p.y * __builtin_amdgcn_exp2f(p.x - m);
    }
    out = m + __log2f(l);
  }
  lse[row] = out;
}

int score_window_max_rows() { return 128; }

// Keys of a block.  A block has a fixed price, its query fragments and the first loads (some 3 us before it streams), and a
// second round that is a small part of the first leaves the chip idle.  So, where blocks of up to 4096 keys (2048 with
// fewer than 97 window rows) get there: as few keys as leave one round of 1024 blocks, four on each of 256 compute units, or
// 5/8 of one while they have under 256 keys.  More keys than that go round several times, 1024 at a time: the rounds mix, and
// the votes of longer blocks take LDS that more of pass 2's would fit in (given the normalisers, 32 layers of 32768 keys:
// 2048 keys a block 419 -> 453 us).
// 8 heads, 128 window rows, both passes, against the power of two that gives 2048 blocks, 1024 keys at the most: 32768 keys of
// one layer 74 -> 53 us, 131071 169 -> 123, of 8 layers 232 -> 202, of 16 440 -> 408; 12001 of one 39.9 -> 37.4, 16384 42.5 ->
// 38.4, 9001 of 32 253 -> 222, 60001 of 8 405 -> 371.  With 64 window rows 32768 keys of 5 layers 125 -> 118; with 16, given
// the normalisers, of 8 layers 97 -> 93.  5/8 and not less: 8193 keys of one layer take 32.6 with 520 blocks of 128 keys, 35.4
// with 344 of 192.
int score_window_rows_per_block(const int32_t* seq_len, int n_seq, int64_t heads, int n_rows) {
  constexpr int64_t kRound = 1024;
  constexpr int kUnit = 64;
  const int mtw = (n_rows + 31) / 32;
  const int most = mtw == 4 ? 4096 : 2048;
  auto blocks = [&](int rows) {
    int64_t n = 0;
    for (int s = 0; s < n_seq; ++s) n += heads * (((int64_t)seq_len[s] + rows - 1) / rows);
    return n;
  };
  if (blocks(most) > kRound) return kWinManyRounds;
  int64_t keys = 0;
  for (int s = 0; s < n_seq; ++s) keys += heads * seq_len[s];
  int rows = 128;
  while (rows < 256 && blocks(rows) > kRound * 5 / 8) rows += kUnit;
  const int share = (int)(keys / kRound) / kUnit * kUnit;   // below this no split fits
  if (rows < share) rows = share;
  while (rows < most && blocks(rows) > kRound) rows += kUnit;
  return rows;
}

// Workspace of one sequence: pairs [heads, ceil(T / 128), 128, 2] (the largest the pairs can get: the smallest
// block and the most padded rows) followed by the merged normalisers [heads, 128]; 256-byte aligned.
size_t score_window_pairs_bytes(int64_t heads, int T) {
  return ((size_t)heads * (((T + 127) / 128) * 2 + 1) * 128 * sizeof(float) + 255) & ~(size_t)255;
}

template <int MTW>
static void launch_passes(const WinTable& tab, int heads, int window, int n_rows, int rows_per_block, float log2_scale,
                          int reach, int pool_kind, float inv_group, hipStream_t stream) {
  const int blocks = tab.first[tab.n];
  if (tab.lse[0] == nullptr) {   // all sequences of a call come with normalisers, or none does
    hipLaunchKernelGGL((score_window_kernel<MTW, 1>), dim3(blocks), dim3(kWinThreads), 0, stream, tab, heads, window,
                       n_rows, rows_per_block, log2_scale, 0, 0, 0.f);
    hipLaunchKernelGGL(score_window_merge_kernel, dim3(tab.n * heads), dim3(128), 0, stream, tab, heads, n_rows,
                       rows_per_block, 32 * MTW);
  }
  hipLaunchKernelGGL((score_window_kernel<MTW, 2>), dim3(blocks), dim3(kWinThreads),
                     win_vote_slots(rows_per_block) * sizeof(float), stream, tab, heads, window, n_rows, rows_per_block,
                     log2_scale, reach, pool_kind, inv_group);
}

// `tab.first` counts the blocks of the passes (the same grid for both).
void launch_score_window(const WinTable& tab, int heads, int window, int group, int pool_width, int pool_kind,
                         int rows_per_block, float scale, hipStream_t stream) {
  if (tab.n <= 0) return;
  const int n_rows = group * window;
  const float log2_scale = scale * 1.44269504088896340736f;
  const float inv_group = 1.f / (float)group;
  const int reach = (pool_width - 1) / 2;
  if (reach > kWinMaxReach) return;   // the host checks the width before
  switch ((n_rows + 31) / 32) {
    case 1: launch_passes<1>(tab, heads, window, n_rows, rows_per_block, log2_scale, reach, pool_kind, inv_group, stream); break;
    case 2: launch_passes<2>(tab, heads, window, n_rows, rows_per_block, log2_scale, reach, pool_kind, inv_group, stream); break;
    case 3: launch_passes<3>(tab, heads, window, n_rows, rows_per_block, log2_scale, reach, pool_kind, inv_group, stream); break;
    case 4: launch_passes<4>(tab, heads, window, n_rows, rows_per_block, log2_scale, reach, pool_kind, inv_group, stream); break;
    default: return;
  }
}

}  // namespace lkv
