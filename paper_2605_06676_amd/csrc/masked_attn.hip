// Training-time causal attention with the multiplicative soft mask of App. B of the paper,
// forward pass, at prefill shape (every token of a sequence is a query):
//
//   p_ij = e^{s_ij} m_j / sum_{k <= i} e^{s_ik} m_k,   s_ij = scale q_i . k_j,   o_i = sum_j p_ij v_j
//
// m is one weight in [0, 1] per KV head and key; the heads of a GQA group share their KV head's
// weights (Sec. 3.1).  As App. B.2 describes, the mask multiplies the exponentials inside the
// softmax (the references of the exponentials are raw scores), so no logarithm of m is ever
// taken.  Next to the output the kernel returns log sum_k e^{s_ik} m_k per query, which the
// backward pass uses to rebuild p from s.
//
// Tiling (flash-attention style, for 64-wide waves and the 16x16x32 bf16 matrix instruction).  A block of four
// waves owns one query head and 128 consecutive queries, 32 per wave; it walks the keys up to its diagonal in tiles
// of 64, staged once per block in LDS, double buffered with one barrier per tile, and read back as operands by all
// four waves.  Per wave and step of 32 keys:
//   S^T[key, query] = K[key, :] . Q[query, :]^T      (A = K rows from LDS, B = Q^T held in registers)
//   O[query, ch]   += P[query, key] V[key, ch]       (A = P, B = V rows by the transposing LDS read)
// The accumulator layout of S^T (lane (rb, query) holds keys 4 rb .. 4 rb + 3 of a 16-key half) is the
// A-operand layout of P for one K-step over the 32 keys, so probabilities go from the first product to the
// second without leaving their lanes.  Each K and V operand read is shared by the two query blocks of the wave.
// The denominator that divides the output is one more output column of the second product (P times a column of
// ones), see acc_l below.
//
// What bounds it: instruction issue, at the clock that the power allows.  At 16384 tokens the matrix pipe is busy for 58 %
// of the cycles and the vector pipe for 60 %, 21 % of them together: 97 % in all, no LDS conflicts (counters), while the
// chip holds 1.7 to 1.9 of its 2.4 GHz.  So what pays is work not done: references that stay put (no maximum, no
// rescaling: 8 %), rows that go from memory to LDS without passing registers (which also frees the 32 registers that the
// pipeline needs), sums kept from being postponed into the next step (6 %).  The steps are pipelined inside a wave (value
// products of step s - 1, weights of step s, logits of step s + 1, in fenced pieces): vector work runs beside 36 % of the
// matrix time, and ran beside 15 to 17 % in kernels that did one thing after the other.  32 query heads, 8 KV heads, in turn with the
// kernel of running maxima and staging through registers: 2.40 -> 2.02 ms at 16384 tokens (1090 TFLOP/s; a library product
// of 8192 x 8192 x 8192 reaches 1310 here), 649 -> 530 us at 8192, 182 -> 147 at 4096, 74 -> 62 at 2345; what the order of
// the blocks and the pieces of plain_step took off since then stands there.  18 registers are kept in scratch
// memory around the loops, none inside them.  Measured and dropped: 64 queries per wave
// at one wave per SIMD (half the LDS reads; 2.38 ms), a block of eight waves in two groups that split the keys (2.41
// ms; 86 us at 2345 tokens), different wave priorities on a SIMD (no change).
#include <type_traits>

#include "lkv_common.h"
#include "lkv_kernels.h"
#include "lkv_lds.h"
#include "lkv_order.h"

namespace lkv {

namespace {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
constexpr int kMaThreads = 256;
constexpr int kMaWaves = kMaThreads / 64;
constexpr int kMaStep = 32;                   // keys per pipeline step: one K-step of the P.V product
constexpr int kMaTile = 2 * kMaStep;          // keys staged per barrier
constexpr int kMaRow = 256;                   // LDS bytes per staged row: rows lie as in memory, their 16-byte pieces permuted
constexpr int kMaQB = 2;                      // 16-query column blocks per wave
constexpr int kMaWaveQ = 16 * kMaQB;
constexpr int kMaBlockQ = kMaWaves * kMaWaveQ;
constexpr int kMaTileLds = 2 * kMaTile * kMaRow + kMaTile * 4;   // K rows, V rows, mask weights
constexpr float kMaLog2e = 1.4426950408889634f;
constexpr double kMaLn2 = 0.69314718055994530942;
constexpr float kMaMoveSum = 1048576.f;       // 2^20: sum of weights at which a reference moves

__device__ __forceinline__ float ma_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ s16x4_t ma_read_tr16(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p));
}

}  // namespace

__global__ void __launch_bounds__(kMaThreads, 2)
masked_attn_fwd_kernel(const uint16_t* __restrict__ q, const uint4* __restrict__ k, const uint4* __restrict__ v,
                       const float* __restrict__ m, int T, int n_heads, int G, float scale, float* __restrict__ o,
                       float* __restrict__ lse) {
  // Two arrays and not one: the compiler then knows that reads of one do not touch the rows on their way to the other.
  __shared__ __align__(1024) unsigned char tile_a[kMaTileLds];
  __shared__ __align__(1024) unsigned char tile_b[kMaTileLds];
  const int n_qtiles = (T + kMaBlockQ - 1) / kMaBlockQ;
  const CausalBlock mine = causal_block(blockIdx.x, n_qtiles, n_heads);
  const int qtile = mine.tile;
  const int hq = mine.head;
  const int h = hq / G;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane >> 4;
  const int c = lane & 15;
  const int q0 = qtile * kMaBlockQ;
  const int qw0 = q0 + wave * kMaWaveQ;                // first query of this wave
  // steps of 32 keys: this wave's last one is the one on its diagonal; a wave past the end has none
  const int n_steps = qw0 < T ? (qw0 + kMaWaveQ) / kMaStep : 0;
  const float qscale = scale * kMaLog2e;
  bf16x8_t ones;
#pragma unroll
  for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;

  // B operand of the first product: Q^T, lane (query c of block qb, K-block r) holds q[query][32 ks + 8 r .. +7]
  bf16x8_t qfrag[kMaQB][4];
#pragma unroll
  for (int qb = 0; qb < kMaQB; ++qb) {
    const int query = min(qw0 + 16 * qb + c, T - 1);   // queries past the end repeat the last one; never stored
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      qfrag[qb][ks] = __builtin_bit_cast(
          bf16x8_t, reinterpret_cast<const uint4*>(q + ((size_t)hq * T + query) * kHeadDim)[ks * 4 + r]);
  }
  float ref[kMaQB];                 // per query c of block qb: reference of the exponentials (log2 domain)
  float l_run[kMaQB];               // this lane's share of the unrounded denominator (for the log-normaliser returned)
  f32x4_t acc_o[kMaQB][8];          // O[query 4 r + e of block qb][channel 16 ct + c]
  // Denominator the output is divided by, for query 4 r + e, the same in all 16 lanes of a row block: it is
  // accumulated by the matrix cores as one more output column, P times a column of ones, hence from the same
  // bf16-rounded weights as the output.  The output is then an exact convex combination of value rows, which keeps o (and the
  // D_i = dO_i . o_i of the backward pass) accurate where one key holds nearly all the weight.
  f32x4_t acc_l[kMaQB];
  bf16x8_t pfrag[kMaQB];            // weights of the step before, not yet multiplied with its value rows
  bf16x8_t plow[kMaQB];             // what their rounding left, where that is multiplied too (last_tile, below)

  const uint4* kh = k + (size_t)h * T * kChunksPerRow;
  const uint4* vh = v + (size_t)h * T * kChunksPerRow;
  const float* mh = m + (size_t)h * T;
  f32x4_t sacc[kMaQB][2];           // S^T of a step: lane (rb = r, query c) holds keys 16 sub + 4 r + e

  // Staging, straight from memory into LDS: a wave instruction fills 1 KB, four rows; lane (row slot, piece slot) fetches
  // piece `slot ^ f(row)` of its row, so that the straight reads of K (16 rows of one piece: f = row) and the transposing
  // reads of V (4 rows of 32 bytes: f = 2 row) both find their banks apart.  Tile t holds the K rows of steps 2 t + 1 and
  // 2 t + 2, the V rows of steps 2 t - 1 and 2 t and the weights of steps 2 t and 2 t + 1: what the pipeline multiplies
  // in its steps 2 t and 2 t + 1.  Rows outside the sequence repeat its first or last one.
  const int srow = tid >> 4, spiece = tid & 15;
  const uint32_t k_piece = (uint32_t)((spiece ^ srow) * 16), v_piece = (uint32_t)((spiece ^ (2 * srow & 15)) * 16);
  auto stage = [&](unsigned char* dst, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int krow = min(t * kMaTile + kMaStep + srow + 16 * j, T - 1);
      const int vrow = min(max(t * kMaTile - kMaStep + srow + 16 * j, 0), T - 1);
      lds_fill16(reinterpret_cast<const unsigned char*>(kh) + ((uint32_t)krow * 256u + k_piece),
                 dst + (16 * j + 4 * wave) * kMaRow);
      lds_fill16(reinterpret_cast<const unsigned char*>(vh) + ((uint32_t)vrow * 256u + v_piece),
                 dst + (kMaTile + 16 * j + 4 * wave) * kMaRow);
    }
    if (wave == 0) lds_fill4(mh + min(t * kMaTile + lane, T - 1), dst + 2 * kMaTile * kMaRow);
  };
  // The last tile has one K step less (no wave has a step after the fourth around the diagonal); the V rows of its second
  // step, whose products come last of all, take that place.
  const int n_full = q0 / kMaTile;   // tiles whose steps lie wholly below the diagonal of every wave of the block; even
  auto stage_last = [&](unsigned char* dst) __attribute__((always_inline)) {
    const int t = n_full + 1;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const int vrow = min(t * kMaTile - kMaStep + srow + 16 * j, T - 1);
      lds_fill16(reinterpret_cast<const unsigned char*>(vh) + ((uint32_t)vrow * 256u + v_piece),
                 dst + ((j < 4 ? kMaTile + 16 * j : 16 * (j - 2)) + 4 * wave) * kMaRow);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int krow = min(t * kMaTile + kMaStep + srow + 16 * j, T - 1);
      lds_fill16(reinterpret_cast<const unsigned char*>(kh) + ((uint32_t)krow * 256u + k_piece),
                 dst + (16 * j + 4 * wave) * kMaRow);
    }
    if (wave == 0) lds_fill4(mh + min(t * kMaTile + lane, T - 1), dst + 2 * kMaTile * kMaRow);
  };
  // where this lane reads: K rows 16 sub + c, pieces 4 ks + r; V rows 4 r + c / 4, channels 16 ct + 4 (c % 4)
  const uint32_t k_at = c * kMaRow + ((r ^ c) * 16);   // piece 4 ks + r is at k_at ^ 64 ks
  const int v_row = 4 * r + (c >> 2);
  const uint32_t v_at = v_row * kMaRow + ((((c >> 1) & 1) ^ (2 * v_row & 15)) * 16) + (c & 1) * 8;   // tile ct at v_at ^ 32 ct

  // O += P V of the step before: B operand lane (channel c of tile ct, K-block r) holds
  // V[keys 4r..4r+3 and 16+4r..16+4r+3][channel]
  auto value_products = [&](auto fine_tag, const unsigned char* v_lds) __attribute__((always_inline)) {
    constexpr bool kFine = decltype(fine_tag)::value;
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb) {
      acc_l[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pfrag[qb], ones, acc_l[qb], 0, 0, 0);
      if (kFine) acc_l[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plow[qb], ones, acc_l[qb], 0, 0, 0);
    }
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      const s16x4_t v0 = ma_read_tr16(v_lds + (v_at ^ (32 * ct)));
      const s16x4_t v1 = ma_read_tr16(v_lds + (v_at ^ (32 * ct)) + 16 * kMaRow);
      const s16x8_t vb = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
      for (int qb = 0; qb < kMaQB; ++qb) {
        acc_o[qb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pfrag[qb], __builtin_bit_cast(bf16x8_t, vb),
                                                                acc_o[qb][ct], 0, 0, 0);
        if (kFine)
          acc_o[qb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plow[qb], __builtin_bit_cast(bf16x8_t, vb),
                                                                  acc_o[qb][ct], 0, 0, 0);
      }
    }
  };
  // The reference of this lane's query of block qb goes up by `up`, what has been summed against it goes down by
  // alpha = 2^-up (queries 4 r + e in the output registers).
  auto lower_by = [&](int qb, float up, float alpha) __attribute__((always_inline)) {
    ref[qb] += up;
    l_run[qb] *= alpha;
    float al[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) al[e] = __shfl(alpha, 4 * r + e, 64);
#pragma unroll
    for (int ct = 0; ct < 8; ++ct)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc_o[qb][ct][e] *= al[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc_l[qb][e] *= al[e];
  };
  // One pipeline step: the value products of step s - 1, the weights of step s, the logits of step s + 1; nothing in
  // it waits for anything else in it, so matrix and vector instructions of one wave run side by side.
  // Some key of the step may lie above some query's diagonal.  kMoving: the references follow the running maxima; else they
  // stay and nothing looks at the maxima.
  auto step = [&](auto moving_tag, auto fine_tag, const unsigned char* tile, int s, int half) __attribute__((always_inline)) {
    constexpr bool kMoving = decltype(moving_tag)::value, kFine = decltype(fine_tag)::value;
    const unsigned char* k_lds = tile + half * kMaStep * kMaRow;
    const float* m_lds = reinterpret_cast<const float*>(tile + 2 * kMaTile * kMaRow) + half * kMaStep;
    value_products(fine_tag, k_lds + kMaTile * kMaRow);
    float top = -INFINITY;
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float x = fmaf(sacc[qb][i >> 2][i & 3], qscale, -ref[qb]);
        x = s * kMaStep + 16 * (i >> 2) + 4 * r + (i & 3) > qw0 + 16 * qb + c ? -INFINITY : x;
        if (kMoving) top = fmaxf(top, x);
        sacc[qb][i >> 2][i & 3] = x;
      }
    if (kMoving && __ballot(top > 0.f) != 0ull) {
#pragma unroll
      for (int qb = 0; qb < kMaQB; ++qb) {
        float up = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) up = fmaxf(up, sacc[qb][i >> 2][i & 3]);
        up = max_over_row_blocks(up);
#pragma unroll
        for (int i = 0; i < 8; ++i) sacc[qb][i >> 2][i & 3] -= up;
        lower_by(qb, up, ma_exp2(-up));
      }
    }
    float psum[kMaQB];   // the step's weights are added up by themselves: the running sum rounds once per step
    f32x4_t next[kMaQB][2];
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int qb = 0; qb < kMaQB; ++qb) next[qb][sub] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const uint4 kx = *reinterpret_cast<const uint4*>(k_lds + sub * 16 * kMaRow + (k_at ^ (64 * ks)));
#pragma unroll
        for (int qb = 0; qb < kMaQB; ++qb)
          next[qb][sub] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kx), qfrag[qb][ks],
                                                                  next[qb][sub], 0, 0, 0);
      }
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const float4 mw4 = *reinterpret_cast<const float4*>(m_lds + 16 * tt + 4 * r);
      const float mw[4] = {mw4.x, mw4.y, mw4.z, mw4.w};
#pragma unroll
      for (int qb = 0; qb < kMaQB; ++qb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p = ma_exp2(sacc[qb][tt][e]) * mw[e];   // the mask multiplies the exponential (App. B.2)
          psum[qb] = tt == 0 && e == 0 ? p : psum[qb] + p;
          pfrag[qb][tt * 4 + e] = (__bf16)p;
          if (kFine) plow[qb][tt * 4 + e] = (__bf16)(p - (float)pfrag[qb][tt * 4 + e]);
        }
    }
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb) l_run[qb] += psum[qb];
    // the weights and their sums are due here, beside the products above, and not where they are used
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb) asm volatile("" : "+v"(pfrag[qb]), "+v"(l_run[qb]));
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb)
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) sacc[qb][sub] = next[qb][sub];
  };
  // The same for the steps wholly below the diagonal, with references that stay put, in eight pieces that the compiler may
  // not mix: the operands of the next products, four or six products, an eighth of the weights.  K operands are read two
  // pieces ahead, V operands one (both one ahead: 2 to 3 % slower where a wave has a SIMD to itself, both two ahead or K three
  // up to 1 % slower).  Against the compiler's own order: 2170 -> 2140 us at 16384 tokens, 32 heads, 562 -> 555 at 8192, 63.2 ->
  // 62.5 at 2345; 8 heads of 4096 75.5 -> 73.3.
  auto plain_step = [&](const unsigned char* tile, int half) __attribute__((always_inline)) {
    const unsigned char* k_lds = tile + half * kMaStep * kMaRow;
    const unsigned char* v_lds = k_lds + kMaTile * kMaRow;
    const float* m_lds = reinterpret_cast<const float*>(tile + 2 * kMaTile * kMaRow) + half * kMaStep;
    f32x4_t next[kMaQB][2];
    uint32_t pw[kMaQB][4];
    float psum[kMaQB], mw[4];
    auto read_k = [&](int i) __attribute__((always_inline)) {
      return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(k_lds + (i >> 2) * 16 * kMaRow + (k_at ^ (64 * (i & 3)))));
    };
    bf16x8_t kx = read_k(0), k1 = read_k(1);
    auto read_v = [&](int ct) __attribute__((always_inline)) {
      const s16x4_t v0 = ma_read_tr16(v_lds + (v_at ^ (32 * ct)));
      const s16x4_t v1 = ma_read_tr16(v_lds + (v_at ^ (32 * ct)) + 16 * kMaRow);
      return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    bf16x8_t vx = read_v(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int sub = i >> 2, ks = i & 3, qp = (i >> 1) & 1, e0 = 2 * (i & 1);
      bf16x8_t kn, vn;
      if (i < 6) kn = read_k(i + 2);
      if (i < 7) vn = read_v(i + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (ks == 0) {
        const float4 mw4 = *reinterpret_cast<const float4*>(m_lds + 16 * sub + 4 * r);
        mw[0] = mw4.x; mw[1] = mw4.y; mw[2] = mw4.z; mw[3] = mw4.w;
      }
#pragma unroll
      for (int qb = 0; qb < kMaQB; ++qb) {
        if (ks == 0) next[qb][sub] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        next[qb][sub] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kx, qfrag[qb][ks], next[qb][sub], 0, 0, 0);
      }
      float ev[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) ev[j] = ma_exp2(fmaf(sacc[qp][sub][e0 + j], qscale, -ref[qp]));
#pragma unroll
      for (int qb = 0; qb < kMaQB; ++qb) {
        if (i == 0) acc_l[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pfrag[qb], ones, acc_l[qb], 0, 0, 0);
        acc_o[qb][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pfrag[qb], vx, acc_o[qb][i], 0, 0, 0);
      }
      bf16x2_t pair;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float p = ev[j] * mw[e0 + j];   // the mask multiplies the exponential (App. B.2)
        psum[qp] = sub == 0 && e0 + j == 0 ? p : psum[qp] + p;
        pair[j] = (__bf16)p;
      }
      uint32_t& word = pw[qp][2 * sub + (i & 1)];
      word = __builtin_bit_cast(uint32_t, pair);
      asm volatile("" : "+v"(word), "+v"(psum[qp]));   // due here, beside the products
      __builtin_amdgcn_sched_barrier(0);
      kx = k1;
      k1 = kn;
      vx = vn;
    }
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb) {
      l_run[qb] += psum[qb];
      asm volatile("" : "+v"(l_run[qb]));
      pfrag[qb] = __builtin_bit_cast(bf16x8_t, make_uint4(pw[qb][0], pw[qb][1], pw[qb][2], pw[qb][3]));
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) sacc[qb][sub] = next[qb][sub];
    }
  };
  // References that stay put save the maximum, the branch on it and the rescaling it guards, 8 % of the time.  Any
  // reference gives the same weights to a rounding as long as no sum overflows (logits far below a reference vanish next
  // to the key that set it, as below a maximum), so a wave looks at its sums every 128 keys, and where one has passed
  // 2^20 moves the references up by whole binary orders.  Where a logit ran away so far from one look to the next that
  // something overflowed all the same, it stays infinite or NaN to the end, and the block starts over with references that
  // follow the running maxima.  (Starting over wherever a sum passes 2^40, with no look in between, cost 1.3 to 1.9
  // times the time on logits of a deviation of 8 and 16.)
  auto move_references = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb) {
      const float sum = max_over_row_blocks(l_run[qb]);
      const int up = min(max((__float_as_int(sum) >> 23) - 127, 0), 120);
      const float alpha = __int_as_float((127 - up) << 23);
      lower_by(qb, (float)up, alpha);
#pragma unroll
      for (int i = 0; i < 8; ++i) pfrag[qb][i] = (__bf16)((float)pfrag[qb][i] * alpha);   // not yet multiplied
    }
  };
  auto start = [&]() __attribute__((always_inline)) {
    // S^T of the first step, its K rows straight from memory: lane (rb = r, query c) gets keys 16 sub + 4 r + e
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int qb = 0; qb < kMaQB; ++qb) sacc[qb][sub] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const uint4 kx = kh[(size_t)min(16 * sub + c, T - 1) * kChunksPerRow + ks * 4 + r];
#pragma unroll
        for (int qb = 0; qb < kMaQB; ++qb)
          sacc[qb][sub] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kx), qfrag[qb][ks],
                                                                  sacc[qb][sub], 0, 0, 0);
      }
    }
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb) {
      float top = -INFINITY;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float x = sacc[qb][i >> 2][i & 3] * qscale;
        top = fmaxf(top, 16 * (i >> 2) + 4 * r + (i & 3) > qw0 + 16 * qb + c ? -INFINITY : x);
      }
      top = max_over_row_blocks(top);
      ref[qb] = top > -INFINITY ? top : 0.f;   // key 0 is seen by every query: only a logit of -inf gets here
      l_run[qb] = 0.f;
      acc_l[qb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) acc_o[qb][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 8; ++i) pfrag[qb][i] = (__bf16)0.f;
    }
  };
  // The steps around the diagonal, where the waves of the block end one after the other.  fine: the weights are
  // multiplied to twice the digits, the rounded ones and then what the rounding left.  The first block of a head does
  // so: its queries see few keys, their outputs are the largest, and a third of the error of all outputs is theirs, while
  // the block is the shortest of all.  It more than makes up for the references that stay put, which round the weight of
  // the largest logit too (exactly 1 against a running maximum).  Error of o against 64 bits at 1024, 2345 and 16384
  // tokens: 1.33e-3, 1.38e-3 and 1.44e-3 with running maxima, 1.35e-3, 1.41e-3 and 1.48e-3 with references that stay put
  // alone, 1.04e-3, 1.16e-3 and 1.32e-3 with this; 128 tokens take 8.9 -> 9.8 us, 512 and more no longer.
  auto last_tile = [&](auto moving_tag, auto fine_tag, const unsigned char* tile, int t) __attribute__((always_inline)) {
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {   // wave-uniform branches
      const int s = 2 * t + half;
      if (s < n_steps) step(moving_tag, fine_tag, tile, s, half);
      else if (s == n_steps) value_products(fine_tag, tile + (kMaTile + half * kMaStep) * kMaRow);
    }
    if (t == n_full + 1 && n_steps == 2 * t + 2) value_products(fine_tag, tile + kMaStep * kMaRow);
  };

  // One barrier per tile: every wave waits for its transfers of the tile before it, so it makes the tile's rows visible,
  // and it means that every wave is done with the other array, which the next tile then fills.
  stage(tile_a, 0);
  if (n_full == 0) stage_last(tile_b);   // all there is: one wait for both
  start();
  if (n_full == 0) {
#pragma unroll
    for (int qb = 0; qb < kMaQB; ++qb)
#pragma unroll
      for (int i = 0; i < 8; ++i) plow[qb][i] = (__bf16)0.f;
    lds_fill_barrier();
#pragma unroll 1
    for (int t = 0; t < 2; ++t) last_tile(std::false_type{}, std::true_type{}, t == 0 ? tile_a : tile_b, t);
  } else {
#pragma unroll 1
    for (int t = 0; t < n_full; t += 2) {
      lds_fill_barrier();
      stage(tile_b, t + 1);
      if (__builtin_expect(__ballot(!(fmaxf(l_run[0], l_run[1]) < kMaMoveSum)) != 0ull, 0)) move_references();
      plain_step(tile_a, 0);
      plain_step(tile_a, 1);
      lds_fill_barrier();
      stage(tile_a, t + 2);
      plain_step(tile_b, 0);
      plain_step(tile_b, 1);
    }
    lds_fill_barrier();
    stage_last(tile_b);
    last_tile(std::false_type{}, std::false_type{}, tile_a, n_full);
    lds_fill_barrier();
    last_tile(std::false_type{}, std::false_type{}, tile_b, n_full + 1);
  }

  float finite = 0.f;   // NaN where anything is not
#pragma unroll
  for (int qb = 0; qb < kMaQB; ++qb) {
    finite = fmaf(l_run[qb], 0.f, finite);
#pragma unroll
    for (int ct = 0; ct < 8; ++ct)
#pragma unroll
      for (int e = 0; e < 4; ++e) finite = fmaf(acc_o[qb][ct][e], 0.f, finite);
  }
  if (__builtin_expect(__syncthreads_or(finite != 0.f), 0)) {
    stage(tile_a, 0);
    start();
#pragma unroll 1
    for (int t = 0; t < n_full + 2; ++t) {
      unsigned char* tile = t & 1 ? tile_b : tile_a;
      unsigned char* other = t & 1 ? tile_a : tile_b;
      lds_fill_barrier();
      if (t < n_full) stage(other, t + 1);
      else if (t == n_full) stage_last(other);
      last_tile(std::true_type{}, std::false_type{}, tile, t);
    }
  }

  // normalise and store: lane (r, c) holds O[query 4 r + e][channels 16 ct + c] and the (rounded) denominators of
  // those queries; the log-normaliser comes from the unrounded sum, held per query c
#pragma unroll
  for (int qb = 0; qb < kMaQB; ++qb) {
    float l = l_run[qb];
    l = sum_over_row_blocks(l);
    const int query = qw0 + 16 * qb + c;
    if (r == 0 && query < T) {
      // log2 of the mantissa is good to 2^-24 absolute; reference and exponent are exact beside it
      const double log2_sum = (double)ref[qb] + (double)__builtin_amdgcn_frexp_expf(l) +
                              (double)__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(l));
      lse[(size_t)hq * T + query] = l > 0.f ? (float)(log2_sum * kMaLn2) : -INFINITY;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lr = acc_l[qb][e];
      const float li = lr > 0.f ? 1.f / lr : 0.f;          // no weight in the whole prefix: zero output
      const int qrow = qw0 + 16 * qb + 4 * r + e;
      if (qrow < T) {
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) o[((size_t)hq * T + qrow) * kHeadDim + 16 * ct + c] = acc_o[qb][ct][e] * li;
      }
    }
  }
}

void launch_masked_attn_fwd(const void* q, const void* k, const void* v, const float* m, int n_q_heads, int n_kv_heads,
                            int T, float scale, float* o, float* lse, hipStream_t stream) {
  const int G = n_q_heads / n_kv_heads;
  hipLaunchKernelGGL(masked_attn_fwd_kernel, dim3((T + kMaBlockQ - 1) / kMaBlockQ * n_q_heads), dim3(kMaThreads),
                     0, stream, static_cast<const uint16_t*>(q), static_cast<const uint4*>(k),
                     static_cast<const uint4*>(v), m, T, n_q_heads, G, scale, o, lse);
}

}  // namespace lkv
