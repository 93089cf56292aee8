// Backward pass of the training-time causal attention with the multiplicative soft mask
// (App. B.3 of the paper).  With s_ij = scale q_i . k_j, L_i = log sum_{k <= i} e^{s_ik} m_k (kept by
// the forward pass) and the upstream gradient dO:
//
//   e_ij  = e^{s_ij - L_i}                 the weight before the mask (a raw softmax up to its normaliser)
//   p_ij  = e_ij m_j                       the attention weight
//   dP_ij = dO_i . v_j,   D_i = dO_i . o_i = sum_j p_ij dP_ij
//   dV_j  = sum_i p_ij dO_i
//   dm_j  = sum_i e_ij (dP_ij - D_i)       the factor towards the mask is e_ij, never 1 / m_j: finite at m_j = 0
//   dS_ij = p_ij (dP_ij - D_i),   dQ_i = scale sum_j dS_ij k_j,   dK_j = scale sum_i dS_ij q_i
//
// sums over the causal pairs j <= i, and for K, V and m also over the query heads of the GQA group.
// Queries whose prefix carries no weight (L_i = -inf) contribute nothing.
//
// Two kernels (three for short sequences), no atomics, every output element written once:
//   masked_attn_bwd_dq_kernel     one block per query head and 128 queries: Q and dO rows in registers,
//                                 K and V rows of all earlier keys stream through LDS; yields dQ, and D_i for the next.
//   masked_attn_bwd_dkv_kernel    one block (eight waves, 32 keys each) per KV head and 256 keys: the K rows of
//                                 the block stay in registers as matrix operands, its V rows in LDS, the Q and dO rows of
//                                 all later queries (and of every query head of the group) stream through LDS; yields
//                                 dK, dV and dm of its keys.  When that gives too few blocks the query heads of a group
//                                 are dealt to several and a reduce kernel adds the partial results in a fixed order.
//   masked_attn_bwd_dkv_narrow_kernel   the same with 16 keys per wave, for short sequences.
// Both recompute s and dP with the 16x16x32 bf16 matrix instruction.  As in the forward kernel the
// products whose result feeds another product are computed transposed, so that the accumulator
// layout of the first (lane (rb, col) holds rows 4 rb .. 4 rb + 3 of two 16-row halves) is the
// A-operand layout of the second over a K-step of 32, and the streamed tile is read once straight
// (A operand of the first products) and once through the transposing LDS read (B operand of the
// second ones).
#include <type_traits>

#include "lkv_common.h"
#include "lkv_kernels.h"
#include "lkv_lds.h"
#include "lkv_order.h"

namespace lkv {

namespace {

constexpr int kMbThreads = 256;
constexpr int kMbWaves = kMbThreads / 64;
constexpr int kMbStep = 32;                    // streamed rows per K-step of the second products
constexpr int kMbSteps = 2;                    // steps staged per barrier (64 rows)
constexpr int kMbTile = kMbStep * kMbSteps;
constexpr int kMbStride = 288;                 // LDS bytes per staged row: measured conflict free for the straight 16-byte
                                               // reads and for the transposing reads (272 was not, for the straight ones)
constexpr float kMbLog2e = 1.4426950408889634f;

constexpr int kMbFewBlocks = 512;              // dkv grids below this leave compute units idle or wait for their longest block

__device__ __forceinline__ float mb_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bf16x8_t mb_read_straight(const unsigned char* p) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(p));
}

// B operand of a product whose K dimension runs over the 32 staged rows of a step: lane (r, c) gets,
// for output column c of column tile ct, rows 4r..4r+3 and 16+4r..16+4r+3 (the K-slot order in which
// the first products leave their results)
__device__ __forceinline__ bf16x8_t mb_read_transposed(const unsigned char* rows, int stride, int r, int c, int ct) {
  const unsigned char* base = rows + (4 * r + (c >> 2)) * stride + ct * 32 + (c & 3) * 8;
  const s16x4_t v0 =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(base));
  const s16x4_t v1 =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(base + 16 * stride));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Permutation of the 16-byte pieces of staged row `row`: piece p lies at slot p ^ row_turn(row).  With it neither the
// straight reads (16 rows of one piece) nor the transposing ones (32 bytes of each of eight rows at a time) meet a bank
// twice (measured; 2 (row % 8) + row / 8 and two others cost 18 to 29 % of the kernel's cycles in conflicts).
__device__ __forceinline__ int row_turn(int row) { return 2 * row & 15; }

// the same from rows whose 16-byte pieces are permuted: p is where the lane's rows 4r + c / 4 (and 16 further on) hold its channels
__device__ __forceinline__ bf16x8_t mb_read_turned(const unsigned char* p) {
  const s16x4_t v0 =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p));
  const s16x4_t v1 =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p + 16 * 256));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
}

}  // namespace

// ---- dQ ------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
constexpr int kDqQB = 2;                       // 16-query column blocks per wave
constexpr int kDqWaveQ = 16 * kDqQB;
constexpr int kDqBlockQ = kMbWaves * kDqWaveQ;
constexpr int kDqRow = 256;                    // LDS bytes per staged row: rows lie as in memory, their 16-byte pieces permuted
constexpr int kDqRows = kMbStep * kDqRow;      // the K or V rows of a step
static_assert(kDqBlockQ == 4 * kMbStep, "the steps below the diagonal of a block come in fours");

// Bound by instruction issue and, for long sequences, by the power that the products draw.  Steps of 32 keys are pipelined
// inside a wave, as in the forward kernel: products of step s - 1 with its key rows, dS of step s, S and dP of step s + 1.
// Left to itself the compiler puts the exponentials of a step behind all of its products (9 % slower), so the step is cut
// into eight pieces of six products, the operands of the next piece and an eighth of the dS, which it may not mix.  The
// rows go from memory to LDS directly; a ring of four K slots holds what steps s - 1 to s + 2 need, two V slots s + 1 and
// s + 2 (53 KB, two blocks per compute unit; tiles of 64 keys would need 80 KB).  D_i is summed here on the way in, from
// rows that the block needs anyhow, and left for the dK/dV kernel: a launch of its own took 65 us at 16384 tokens, 9.4 at
// 2345.  32 query heads, 8 KV heads, in turn with a kernel that did one thing after the other and staged through
// registers: 2960 -> 2690 us at 16384 tokens (1225 TFLOP/s), 216 -> 193 at 4096, 97 -> 85 at 2345; 8 and 8 heads of 4096
// 143 -> 108.
__global__ void __launch_bounds__(kMbThreads, 2)
masked_attn_bwd_dq_kernel(const uint16_t* __restrict__ q, const uint4* __restrict__ k, const uint4* __restrict__ v,
                          const float* __restrict__ m, const float* __restrict__ lse, float* __restrict__ dvec,
                          const float* __restrict__ o, const uint16_t* __restrict__ d_o, int T, int n_heads, int G,
                          float scale, float* __restrict__ dq) {
  // An array per slot: the compiler then knows that reads of one do not touch the rows on their way to another.  K slots
  // hold the rows of a step and then its mask weights.
  __shared__ __align__(1024) unsigned char k_a[kDqRows + 256], k_b[kDqRows + 256], k_c[kDqRows + 256], k_d[kDqRows + 256];
  __shared__ __align__(1024) unsigned char v_a[kDqRows], v_b[kDqRows];
  const int n_qtiles = (T + kDqBlockQ - 1) / kDqBlockQ;
  const CausalBlock mine = causal_block(blockIdx.x, n_qtiles, n_heads);
  const int qtile = mine.tile;
  const int hq = mine.head;
  const int h = hq / G;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane >> 4;
  const int c = lane & 15;
  const int q0 = qtile * kDqBlockQ;
  const int qw0 = q0 + wave * kDqWaveQ;
  const float qscale = scale * kMbLog2e;

  const unsigned char* kh = reinterpret_cast<const unsigned char*>(k + (size_t)h * T * kChunksPerRow);
  const unsigned char* vh = reinterpret_cast<const unsigned char*>(v + (size_t)h * T * kChunksPerRow);
  const float* mh = m + (size_t)h * T;
  const int srow = tid >> 4;
  const uint32_t piece = (uint32_t)(((tid & 15) ^ row_turn(srow)) * 16);
  // the rows of step s, straight from memory to LDS; rows outside the sequence repeat its first or last one
  auto fill = [&](unsigned char* k_dst, unsigned char* v_dst, int s, auto both_tag) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t at = (uint32_t)min(max(s * kMbStep + srow + 16 * j, 0), T - 1) * 256u + piece;
      lds_fill16(kh + at, k_dst + (16 * j + 4 * wave) * kDqRow);
      if (decltype(both_tag)::value) lds_fill16(vh + at, v_dst + (16 * j + 4 * wave) * kDqRow);
    }
    if (wave == 0) lds_fill4(mh + min(max(s * kMbStep + lane, 0), T - 1), k_dst + kDqRows);
  };
  fill(k_a, v_a, 0, std::true_type{});
  fill(k_b, v_b, 1, std::true_type{});
  fill(k_d, v_a, -1, std::false_type{});

  // B operands of the first products: lane (query c of block qb, K-block r) holds 8 channels of q and of dO
  bf16x8_t qfrag[kDqQB][4], gfrag[kDqQB][4];
  float lse2[kDqQB], dneg[kDqQB];   // log-normaliser (log2 domain), -D
#pragma unroll
  for (int qb = 0; qb < kDqQB; ++qb) {
    const int query = min(qw0 + 16 * qb + c, T - 1);   // queries past the end repeat the last one; never stored
    const size_t row = (size_t)hq * T + query;
    float d = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      qfrag[qb][ks] = __builtin_bit_cast(bf16x8_t, reinterpret_cast<const uint4*>(q + row * kHeadDim)[ks * 4 + r]);
      gfrag[qb][ks] = __builtin_bit_cast(bf16x8_t, reinterpret_cast<const uint4*>(d_o + row * kHeadDim)[ks * 4 + r]);
      const float4 o0 = reinterpret_cast<const float4*>(o + row * kHeadDim)[ks * 8 + 2 * r];
      const float4 o1 = reinterpret_cast<const float4*>(o + row * kHeadDim)[ks * 8 + 2 * r + 1];
      const float ov[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) d = fmaf(ov[i], (float)gfrag[qb][ks][i], d);
    }
    d = sum_over_row_blocks(d);
    if (r == 0 && qw0 + 16 * qb + c < T) dvec[row] = d;
    dneg[qb] = -d;
    const float l = lse[row];
    lse2[qb] = l == -INFINITY ? INFINITY : l * kMbLog2e;   // no weight in the prefix: every e_ij becomes 0
  }
  f32x4_t acc[kDqQB][8];              // dQ[query 4 r + e of block qb][channel 16 ct + c], before the scale
  f32x4_t sacc[kDqQB][2], pacc[kDqQB][2];   // S^T and dP^T - D of a step: lane (rb = r, query c) has keys 16 tt + 4 r + e
  bf16x8_t dsfrag[kDqQB];             // dS of the step before, not yet multiplied with its key rows
#pragma unroll
  for (int qb = 0; qb < kDqQB; ++qb) {
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc[qb][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) dsfrag[qb][i] = (__bf16)0.f;
  }
  const uint32_t straight = c * kDqRow + ((r ^ row_turn(c)) * 16);
  const int trow = 4 * r + (c >> 2);
  const uint32_t turned = trow * kDqRow + ((((c >> 1) & 1) ^ row_turn(trow)) * 16) + (c & 1) * 8;

  auto logits = [&](f32x4_t (&sx)[kDqQB][2], f32x4_t (&px)[kDqQB][2], const unsigned char* k_lds, const unsigned char* v_lds)
      __attribute__((always_inline)) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
#pragma unroll
      for (int qb = 0; qb < kDqQB; ++qb) {
        sx[qb][tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        px[qb][tt] = f32x4_t{dneg[qb], dneg[qb], dneg[qb], dneg[qb]};
      }
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bf16x8_t kx = mb_read_straight(k_lds + tt * 16 * kDqRow + (straight ^ (64 * ks)));
        const bf16x8_t vx = mb_read_straight(v_lds + tt * 16 * kDqRow + (straight ^ (64 * ks)));
#pragma unroll
        for (int qb = 0; qb < kDqQB; ++qb) {
          sx[qb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kx, qfrag[qb][ks], sx[qb][tt], 0, 0, 0);
          px[qb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vx, gfrag[qb][ks], px[qb][tt], 0, 0, 0);
        }
      }
    }
  };
  // dQ += dS K: B operand from the K rows by the transposing read
  auto products = [&](const unsigned char* k_lds) __attribute__((always_inline)) {
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      const bf16x8_t kb = mb_read_turned(k_lds + (turned ^ (32 * ct)));
#pragma unroll
      for (int qb = 0; qb < kDqQB; ++qb)
        acc[qb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dsfrag[qb], kb, acc[qb][ct], 0, 0, 0);
    }
  };
  auto pointwise = [&](auto diag_tag, const unsigned char* k_lds, int s) __attribute__((always_inline)) {
    constexpr bool kDiag = decltype(diag_tag)::value;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const float4 mw4 = *reinterpret_cast<const float4*>(k_lds + kDqRows + (16 * tt + 4 * r) * 4);
      const float mw[4] = {mw4.x, mw4.y, mw4.z, mw4.w};
#pragma unroll
      for (int qb = 0; qb < kDqQB; ++qb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float ev = mb_exp2(fmaf(sacc[qb][tt][e], qscale, -lse2[qb]));
          if (kDiag) ev = s * kMbStep + 16 * tt + 4 * r + e > qw0 + 16 * qb + c ? 0.f : ev;
          dsfrag[qb][tt * 4 + e] = (__bf16)(ev * mw[e] * pacc[qb][tt][e]);
        }
    }
#pragma unroll
    for (int qb = 0; qb < kDqQB; ++qb) asm volatile("" : "+v"(dsfrag[qb]));   // due here, beside the products
  };
  // One pipeline step: the products of step s - 1, dS of step s, the logits of step s + 1
  auto step = [&](const unsigned char* k_prev, const unsigned char* k_cur, const unsigned char* k_next,
                  const unsigned char* v_next) __attribute__((always_inline)) {
    f32x4_t sx[kDqQB][2], px[kDqQB][2];
    bf16x8_t kx = mb_read_straight(k_next + straight), vx = mb_read_straight(v_next + straight), kb = mb_read_turned(k_prev + turned);
    uint32_t ds[kDqQB][4];
    float mw[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int tt = i >> 2, ks = i & 3, qp = (i >> 1) & 1, e0 = 2 * (i & 1);
      if (ks == 0) {
        const float4 mw4 = *reinterpret_cast<const float4*>(k_cur + kDqRows + (16 * tt + 4 * r) * 4);
        mw[0] = mw4.x; mw[1] = mw4.y; mw[2] = mw4.z; mw[3] = mw4.w;
      }
#pragma unroll
      for (int qb = 0; qb < kDqQB; ++qb) {
        if (ks == 0) {
          sx[qb][tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          px[qb][tt] = f32x4_t{dneg[qb], dneg[qb], dneg[qb], dneg[qb]};
        }
        sx[qb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kx, qfrag[qb][ks], sx[qb][tt], 0, 0, 0);
        px[qb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vx, gfrag[qb][ks], px[qb][tt], 0, 0, 0);
      }
      float ev[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) ev[j] = mb_exp2(fmaf(sacc[qp][tt][e0 + j], qscale, -lse2[qp]));
      __builtin_amdgcn_sched_barrier(0);   // the next operands after these products have taken theirs: 24 registers less
      if (i < 7) {
        const uint32_t at = ((i + 1) >> 2) * 16 * kDqRow + (straight ^ (64 * ((i + 1) & 3)));
        kx = mb_read_straight(k_next + at);
        vx = mb_read_straight(v_next + at);
      }
#pragma unroll
      for (int qb = 0; qb < kDqQB; ++qb) acc[qb][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dsfrag[qb], kb, acc[qb][i], 0, 0, 0);
      bf16x2_t pair;
#pragma unroll
      for (int j = 0; j < 2; ++j) pair[j] = (__bf16)(ev[j] * mw[e0 + j] * pacc[qp][tt][e0 + j]);
      uint32_t& word = ds[qp][2 * tt + (i & 1)];
      word = __builtin_bit_cast(uint32_t, pair);
      asm volatile("" : "+v"(word));   // due here, beside the products
      __builtin_amdgcn_sched_barrier(0);
      if (i < 7) kb = mb_read_turned(k_prev + (turned ^ (32 * (i + 1))));
    }
#pragma unroll
    for (int qb = 0; qb < kDqQB; ++qb) {
      dsfrag[qb] = __builtin_bit_cast(bf16x8_t, make_uint4(ds[qb][0], ds[qb][1], ds[qb][2], ds[qb][3]));
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) { sacc[qb][tt] = sx[qb][tt]; pacc[qb][tt] = px[qb][tt]; }
    }
  };
  const int n_full = q0 / kMbStep;   // steps that lie wholly below the diagonal of every wave of the block
  const bool live = qw0 < T;
  lds_fill_barrier();
  logits(sacc, pacc, k_a, v_a);
#pragma unroll 1
  for (int s = 0; s < n_full; s += 4) {
    lds_fill_barrier();
    fill(k_c, v_a, s + 2, std::true_type{});
    step(k_d, k_a, k_b, v_b);
    lds_fill_barrier();
    fill(k_d, v_b, s + 3, std::true_type{});
    step(k_a, k_b, k_c, v_a);
    lds_fill_barrier();
    fill(k_a, v_a, s + 4, std::true_type{});
    step(k_b, k_c, k_d, v_b);
    lds_fill_barrier();
    fill(k_b, v_b, s + 5, std::true_type{});
    step(k_c, k_d, k_a, v_a);
  }
  // The steps around the diagonal, where the waves of the block end one after the other: step n_full + w is wave w's last
#pragma unroll 1
  for (int j = 0; j <= 4; ++j) {
    lds_fill_barrier();
    unsigned char* k_prev = j == 0 ? k_d : j == 1 ? k_a : j == 2 ? k_b : j == 3 ? k_c : k_d;
    unsigned char* k_cur = j == 0 ? k_a : j == 1 ? k_b : j == 2 ? k_c : k_d;
    unsigned char* k_next = j == 0 ? k_b : j == 1 ? k_c : k_d;
    unsigned char* v_next = j & 1 ? v_a : v_b;
    if (j == 0) fill(k_c, v_a, n_full + 2, std::true_type{});
    else if (j == 1) fill(k_d, v_b, n_full + 3, std::true_type{});
    if (!live) continue;
    if (j <= wave + 1) products(k_prev);
    if (j < wave) {
      f32x4_t sx[kDqQB][2], px[kDqQB][2];
      pointwise(std::false_type{}, k_cur, n_full + j);
      logits(sx, px, k_next, v_next);
#pragma unroll
      for (int qb = 0; qb < kDqQB; ++qb)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) { sacc[qb][tt] = sx[qb][tt]; pacc[qb][tt] = px[qb][tt]; }
    } else if (j == wave) {
      pointwise(std::true_type{}, k_cur, n_full + j);
    }
  }

#pragma unroll
  for (int qb = 0; qb < kDqQB; ++qb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int qrow = qw0 + 16 * qb + 4 * r + e;
      if (qrow < T) {
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) dq[((size_t)hq * T + qrow) * kHeadDim + 16 * ct + c] = acc[qb][ct][e] * scale;
      }
    }
}

// ---- dK, dV, dm ----------------------------------------------------------------------------------
constexpr int kDkvThreads = 512;
constexpr int kDkvKB = 2;                      // 16-key column blocks per wave
constexpr int kDkvWaveK = 16 * kDkvKB;
constexpr int kDkvBlockK = kDkvThreads / 64 * kDkvWaveK;
constexpr int kDkvRow = 256;                   // LDS bytes per staged row: rows lie as in memory, their 16-byte pieces permuted
constexpr int kDkvTileLds = 2 * kMbTile * kDkvRow;   // Q rows, dO rows of one item

// Bound by instruction issue and by waiting for it: at 16384 tokens the matrix pipe is busy for 45 % of the cycles and
// the vector pipe for 40 %, 7 % of them together, so a fifth of the cycles issue to neither; the LDS is busy 43 % (78 %
// with 16 keys per wave and 64 KB of operands per 32 queries; a wave reads 40 KB here for 64 matrix instructions).  32
// keys per wave need 128 accumulator and 32 K operand registers; V operands come from LDS so that the rest fits 256.  32 query
// heads, 8 KV heads: 4.65 -> 4.33 ms at 16384 tokens; the whole backward pass 7.74 -> 7.30 ms, 1971 -> 1868 us at 8192,
// 562 -> 524 us at 4096.  Measured and dropped: separate loops without the edge branch (the compiler then hoists
// operand reads into spills: 7.72 ms).
__global__ void __launch_bounds__(kDkvThreads, 2)
masked_attn_bwd_dkv_kernel(const uint4* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                           const float* __restrict__ m, const float* __restrict__ lse, const float* __restrict__ dvec,
                           const uint4* __restrict__ d_o, int T, int n_kv_heads, int G, int split, float scale,
                           float* __restrict__ dk, float* __restrict__ dv, float* __restrict__ dm) {
  // Two arrays and not one: the compiler then knows that reads of one do not touch the rows on their way to the other.
  __shared__ __align__(1024) unsigned char tile_a[kDkvTileLds];
  __shared__ __align__(1024) unsigned char tile_b[kDkvTileLds];
  __shared__ __align__(1024) unsigned char v_rows[kDkvBlockK * kDkvRow];   // the block's V rows, read as operands in every step
  __shared__ __align__(16) float aux_a[2 * kMbTile];   // lse (log2 domain) and D of the item's queries
  __shared__ __align__(16) float aux_b[2 * kMbTile];
  // A block owns 256 keys of one KV head and the query heads g_lo .. g_lo + g_cnt - 1 of its group: all of them
  // (split = 1, results go straight to dk, dv, dm) or an equal share (split divides G: results are partial sums, row
  // `unit` of buffers the host passes in place of the outputs, added up by the reduce kernel).  Blocks in order of
  // decreasing work: early keys have the most queries after them; key tile slow, unit fast.
  const int n_units = n_kv_heads * split;
  const int unit = (int)blockIdx.x % n_units;
  const int h = unit / split;
  const int g_cnt = G / split;
  const int g_lo = (unit - h * split) * g_cnt;
  const int k0 = (int)blockIdx.x / n_units * kDkvBlockK;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane >> 4;
  const int c = lane & 15;
  const int kw0 = k0 + wave * kDkvWaveK;
  const float qscale = scale * kMbLog2e;

  // streamed items: for every query head of the group, the 64-query tiles from the one that holds query k0 on
  const int n_items = g_cnt * ((T - k0 + kMbTile - 1) / kMbTile);
  // Staging, straight from memory into LDS: a wave instruction fills 1 KB, four rows; lane (row slot, piece slot) fetches
  // piece `slot ^ f(row)` of its row (row_turn below), so that both the straight reads (eight rows of one piece at a time)
  // and the transposing reads (four rows of 32 bytes) find their banks apart.
  const int srow = tid >> 4;
  const uint32_t piece = (uint32_t)(((tid & 15) ^ row_turn(srow)) * 16);
  float aux = 0.f;   // threads 0..63: lse of query tid; threads 64..127: D of query tid - 64
  // From the last query down to the block's diagonal: blocks of one KV head run on one XCD (where the units divide by 8)
  // and meet the same rows at the same time, in its L2 (4096 tokens, 8 x 4 heads: 295 -> 288 us; 16384: 4731 -> 4706).
  const int q_last = k0 + (T - 1 - k0) / kMbTile * kMbTile;   // first query of the last tile
  int next_head = 0, next_q0 = q_last;   // the item to be fetched next: query head of the group, first query
  auto fetch = [&](unsigned char* dst) __attribute__((always_inline)) {
    const size_t base = ((size_t)h * G + g_lo + next_head) * T;
    const unsigned char* qs = reinterpret_cast<const unsigned char*>(q + base * kChunksPerRow);
    const unsigned char* gs = reinterpret_cast<const unsigned char*>(d_o + base * kChunksPerRow);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t at = (uint32_t)min(next_q0 + srow + 32 * j, T - 1) * 256u + piece;   // past the end: the last row, masked later
      lds_fill16(qs + at, dst + (32 * j + 4 * wave) * kDkvRow);
      lds_fill16(gs + at, dst + (kMbTile + 32 * j + 4 * wave) * kDkvRow);
    }
    const int query = min(next_q0 + lane, T - 1);
    aux = (wave & 1) ? dvec[base + query] : lse[base + query];
    next_q0 -= kMbTile;
    if (next_q0 < k0) {
      next_q0 = q_last;
      next_head = next_head + 1 < g_cnt ? next_head + 1 : 0;
    }
  };
  auto put_aux = [&](float* dst) __attribute__((always_inline)) {
    // lse goes to the log2 domain; -inf (no weight in the prefix) becomes +inf so that every e_ij is 0
    if (tid < 2 * kMbTile) dst[tid] = wave == 1 ? aux : (aux == -INFINITY ? INFINITY : aux * kMbLog2e);
  };
  fetch(tile_a);
#pragma unroll
  for (int j = 0; j < kDkvBlockK / 32; ++j)
    lds_fill16(reinterpret_cast<const unsigned char*>(v) +
                   ((size_t)h * T + min(k0 + srow + 32 * j, T - 1)) * (kHeadDim * 2) + piece,
               v_rows + (32 * j + 4 * wave) * kDkvRow);

  // B operands of the first products: lane (key c of block kb, K-block r) holds 8 channels of k; those of v do not fit
  // the registers and come from LDS in every step
  bf16x8_t kfrag[kDkvKB][4];
  float mkey[kDkvKB], dm_acc[kDkvKB];
#pragma unroll
  for (int kb = 0; kb < kDkvKB; ++kb) {
    const int key = min(kw0 + 16 * kb + c, T - 1);      // keys past the end repeat the last one; never stored
    const size_t row = (size_t)h * T + key;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      kfrag[kb][ks] = __builtin_bit_cast(bf16x8_t, reinterpret_cast<const uint4*>(k + row * kHeadDim)[ks * 4 + r]);
    mkey[kb] = m[row];
    dm_acc[kb] = 0.f;
  }
  f32x4_t acc_v[kDkvKB][8], acc_k[kDkvKB][8];   // dV, dK[key 4 r + e of block kb][channel 16 ct + c]
#pragma unroll
  for (int kb = 0; kb < kDkvKB; ++kb)
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      acc_v[kb][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      acc_k[kb][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  // where this lane reads: rows 16 tt + c, pieces 4 ks + r (at straight ^ 64 ks); rows 4 r + c / 4, channels
  // 16 ct + 4 (c % 4) (at turned ^ 32 ct)
  const uint32_t straight = c * kDkvRow + ((r ^ row_turn(c)) * 16);
  const int trow = 4 * r + (c >> 2);
  const uint32_t turned = trow * kDkvRow + ((((c >> 1) & 1) ^ row_turn(trow)) * 16) + (c & 1) * 8;

  const unsigned char* v_mine = v_rows + wave * kDkvWaveK * kDkvRow;

  // 32 queries (half a tile) against this wave's keys
  auto step = [&](const unsigned char* tile, const float* aux_lds, int qs0) __attribute__((always_inline)) {
    // wave-uniform: the plain path needs every query of the step at or after every key of the wave, and inside T
    const bool edge = qs0 < kw0 + kDkvWaveK - 1 || qs0 + kMbStep > T;
    const unsigned char* q_lds = tile;
    const unsigned char* g_lds = tile + kMbTile * kDkvRow;
    bf16x8_t pfrag[kDkvKB], dsfrag[kDkvKB];
    // dP and S: lane (rb = r, key c) gets queries 16 tt + 4 r + e
    f32x4_t pacc[2][kDkvKB];
#pragma unroll
    for (int kb = 0; kb < kDkvKB; ++kb) pacc[0][kb] = pacc[1][kb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      bf16x8_t vx[kDkvKB];
#pragma unroll
      for (int kb = 0; kb < kDkvKB; ++kb) vx[kb] = mb_read_straight(v_mine + kb * 16 * kDkvRow + (straight ^ (64 * ks)));
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const bf16x8_t gx = mb_read_straight(g_lds + tt * 16 * kDkvRow + (straight ^ (64 * ks)));
#pragma unroll
        for (int kb = 0; kb < kDkvKB; ++kb)
          pacc[tt][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gx, vx[kb], pacc[tt][kb], 0, 0, 0);
      }
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      f32x4_t sacc[kDkvKB];
#pragma unroll
      for (int kb = 0; kb < kDkvKB; ++kb) sacc[kb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bf16x8_t qx = mb_read_straight(q_lds + tt * 16 * kDkvRow + (straight ^ (64 * ks)));
#pragma unroll
        for (int kb = 0; kb < kDkvKB; ++kb)
          sacc[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qx, kfrag[kb][ks], sacc[kb], 0, 0, 0);
      }
      const float4 l4 = *reinterpret_cast<const float4*>(aux_lds + 16 * tt + 4 * r);
      const float4 d4 = *reinterpret_cast<const float4*>(aux_lds + kMbTile + 16 * tt + 4 * r);
      const float lq[4] = {l4.x, l4.y, l4.z, l4.w};
      const float dq_[4] = {d4.x, d4.y, d4.z, d4.w};
      auto pointwise = [&](auto edge_tag) __attribute__((always_inline)) {
        constexpr bool kEdge = decltype(edge_tag)::value;
#pragma unroll
        for (int kb = 0; kb < kDkvKB; ++kb) {
          const int key = kw0 + 16 * kb + c;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int query = qs0 + 16 * tt + 4 * r + e;
            float ev = mb_exp2(fmaf(sacc[kb][e], qscale, -lq[e]));
            if (kEdge) ev = (key > query || query >= T) ? 0.f : ev;
            const float diff = pacc[tt][kb][e] - dq_[e];
            dm_acc[kb] = fmaf(ev, diff, dm_acc[kb]);
            const float p = ev * mkey[kb];
            pfrag[kb][tt * 4 + e] = (__bf16)p;
            dsfrag[kb][tt * 4 + e] = (__bf16)(p * diff);
          }
          asm volatile("" : "+v"(dm_acc[kb]));   // due here: the compiler would keep the summands and add them up later
        }
      };
      if (edge) pointwise(std::true_type{});
      else pointwise(std::false_type{});
    }
    // dV += P^T dO and dK += dS^T Q: B operands from the dO and Q rows by the transposing read
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      const bf16x8_t gb = mb_read_turned(g_lds + (turned ^ (32 * ct)));
      const bf16x8_t qb = mb_read_turned(q_lds + (turned ^ (32 * ct)));
#pragma unroll
      for (int kb = 0; kb < kDkvKB; ++kb) {
        acc_v[kb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pfrag[kb], gb, acc_v[kb][ct], 0, 0, 0);
        acc_k[kb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dsfrag[kb], qb, acc_k[kb][ct], 0, 0, 0);
      }
    }
  };
  int q0 = q_last;   // first query of the current item
  auto item = [&](const unsigned char* tile, const float* aux_lds) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < kMbSteps; ++st) {
      const int qs0 = q0 + st * kMbStep;
      // wave-uniform: nothing to do when all 32 queries come before this wave's keys, or lie past the end
      if (qs0 + kMbStep - 1 >= kw0 && qs0 < T && kw0 < T) step(tile + st * kMbStep * kDkvRow, aux_lds + st * kMbStep, qs0);
    }
    q0 = q0 > k0 ? q0 - kMbTile : q_last;
  };
  // One barrier per item: every wave waits for its transfers of the item before it, so it makes the item's rows visible,
  // and it means that every wave is done with the other array, which the next item then fills.
  put_aux(aux_a);
#pragma unroll 1
  for (int it = 0; it < n_items; it += 2) {
    lds_fill_barrier();
    fetch(tile_b);
    item(tile_a, aux_a);
    put_aux(aux_b);
    if (it + 1 >= n_items) break;
    lds_fill_barrier();
    fetch(tile_a);
    item(tile_b, aux_b);
    put_aux(aux_a);
  }

#pragma unroll
  for (int kb = 0; kb < kDkvKB; ++kb) {
    float s = dm_acc[kb];
    s = sum_over_row_blocks(s);
    const int key = kw0 + 16 * kb + c;
    if (r == 0 && key < T) dm[(size_t)unit * T + key] = s;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int krow = kw0 + 16 * kb + 4 * r + e;
      if (krow < T) {
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) {
          dv[((size_t)unit * T + krow) * kHeadDim + 16 * ct + c] = acc_v[kb][ct][e];
          dk[((size_t)unit * T + krow) * kHeadDim + 16 * ct + c] = acc_k[kb][ct][e] * scale;
        }
      }
    }
  }
}

// The same with 16 keys per wave and 128 per block, everything but the streamed rows in registers: twice the LDS reads
// per product, but half as long a chain of items per key, which is what short sequences wait for.
// per 32-query step buffer: Q rows, dO rows (both also read transposed), 32 x lse (log2 domain), 32 x D
constexpr int kNarrowStepLds = kMbStep * 2 * kMbStride + 2 * kMbStep * 4;
constexpr int kNarrowLds = 2 * kMbSteps * kNarrowStepLds;

constexpr int kNarrowWaves = 8;                   // two per SIMD
constexpr int kNarrowThreads = 64 * kNarrowWaves;
constexpr int kNarrowBlockK = 16 * kNarrowWaves;

__global__ void __launch_bounds__(kNarrowThreads, 2)
masked_attn_bwd_dkv_narrow_kernel(const uint4* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                           const float* __restrict__ m, const float* __restrict__ lse, const float* __restrict__ dvec,
                           const uint4* __restrict__ d_o, int T, int n_kv_heads, int G, int split, float scale,
                           float* __restrict__ dk, float* __restrict__ dv, float* __restrict__ dm) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kKB = 1;
  constexpr int kWaveK = 16 * kKB;
  constexpr int kBlockK = kNarrowBlockK;
  constexpr int kTileLds = kMbSteps * kNarrowStepLds;
  constexpr int kRowSlots = 4 * kNarrowWaves;               // staged rows covered by one pass of the block: 32, half a tile
  // A block owns 128 keys of one KV head and the query heads g_lo .. g_lo + g_cnt - 1 of its group: all of them
  // (split = 1, results go straight to dk, dv, dm) or one each (split = G: results are per-query-head partial sums,
  // row `unit` of buffers the host passes in place of the outputs, added up by the reduce kernel).  Blocks in order
  // of decreasing work: early keys have the most queries after them; key tile slow, unit fast.
  const int n_units = n_kv_heads * split;
  const int unit = (int)blockIdx.x % n_units;
  const int h = unit / split;
  const int g_cnt = G / split;
  const int g_lo = (unit - h * split) * g_cnt;
  const int k0 = (int)blockIdx.x / n_units * kBlockK;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int r = lane >> 4;
  const int c = lane & 15;
  const int kw0 = k0 + wave * kWaveK;
  const float qscale = scale * kMbLog2e;

  // B operands of the first products: lane (key c of block kb, K-block r) holds 8 channels of k and of v
  bf16x8_t kfrag[kKB][4], vfrag[kKB][4];
  float mkey[kKB], dm_acc[kKB];
#pragma unroll
  for (int kb = 0; kb < kKB; ++kb) {
    const int key = min(kw0 + 16 * kb + c, T - 1);      // keys past the end repeat the last one; never stored
    const size_t row = (size_t)h * T + key;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      kfrag[kb][ks] = __builtin_bit_cast(bf16x8_t, reinterpret_cast<const uint4*>(k + row * kHeadDim)[ks * 4 + r]);
      vfrag[kb][ks] = __builtin_bit_cast(bf16x8_t, reinterpret_cast<const uint4*>(v + row * kHeadDim)[ks * 4 + r]);
    }
    mkey[kb] = m[row];
    dm_acc[kb] = 0.f;
  }
  f32x4_t acc_v[kKB][8], acc_k[kKB][8];   // dV, dK[key 4 r + e of block kb][channel 16 ct + c]
#pragma unroll
  for (int kb = 0; kb < kKB; ++kb)
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      acc_v[kb][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      acc_k[kb][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

  // streamed items: for every query head of the group, the 64-query tiles from the one that holds query k0 on
  const int q_first = k0 / kMbTile * kMbTile;
  const int tiles_per_head = (T - q_first + kMbTile - 1) / kMbTile;
  const int n_items = g_cnt * tiles_per_head;
  const int srow = tid >> 4, spiece = tid & 15;
  uint4 q_s0, q_s1, g_s0, g_s1;   // thread (row slot tid / 16 in 0..31, piece tid % 16) moves rows slot and slot + 32
  float aux;   // threads 0..63: lse of query tid; threads 64..127: D of query tid - 64
#define LKV_MB_LOAD_ROW(j_, qreg_, greg_, base_, q0_)                                                       \
  {                                                                                                         \
    const int query = min((q0_) + srow + kRowSlots * (j_), T - 1); /* past the end: the last row, masked later */ \
    const uint32_t off = (uint32_t)query * 256u + (uint32_t)spiece * 16u; /* 32-bit offset, uniform base */ \
    qreg_ = *reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned char*>(q + (base_) * kChunksPerRow) + off);   \
    greg_ = *reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned char*>(d_o + (base_) * kChunksPerRow) + off); \
  }
#define LKV_MB_LOAD_ITEM(it_)                                                       \
  {                                                                                 \
    const int g_ = (it_) / tiles_per_head;                                          \
    const int q0_ = q_first + ((it_) - g_ * tiles_per_head) * kMbTile;              \
    const size_t base_ = ((size_t)h * G + g_lo + g_) * T;                           \
    LKV_MB_LOAD_ROW(0, q_s0, g_s0, base_, q0_)                                      \
    LKV_MB_LOAD_ROW(1, q_s1, g_s1, base_, q0_)                                      \
    const int query_ = min(q0_ + (tid & (kMbTile - 1)), T - 1);                     \
    aux = (tid & kMbTile) ? dvec[base_ + query_] : lse[base_ + query_];             \
  }
  /* staged row srow + kRowSlots * j of the 64-row tile: step (row / 32), row-in-step (row % 32) */
#define LKV_MB_STORE_ROW(j_, qreg_, greg_)                                                                   \
  {                                                                                                          \
    const int trow = srow + kRowSlots * (j_);                                                                \
    unsigned char* step_buf = buf + (trow >> 5) * kNarrowStepLds;                                               \
    const int row = trow & 31;                                                                               \
    *reinterpret_cast<uint4*>(step_buf + row * kMbStride + spiece * 16) = qreg_;                            \
    *reinterpret_cast<uint4*>(step_buf + kMbStep * kMbStride + row * kMbStride + spiece * 16) = greg_;     \
  }
  LKV_MB_LOAD_ITEM(0)

#pragma unroll 1
  for (int it = 0; it < n_items; ++it) {
    unsigned char* buf = smem + (it & 1) * kTileLds;
    LKV_MB_STORE_ROW(0, q_s0, g_s0)
    LKV_MB_STORE_ROW(1, q_s1, g_s1)
    if (tid < 2 * kMbTile) {
      // lse goes to the log2 domain; -inf (no weight in the prefix) becomes +inf so that every e_ij is 0
      const float val = (tid & kMbTile) ? aux : (aux == -INFINITY ? INFINITY : aux * kMbLog2e);
      float* aux_lds = reinterpret_cast<float*>(buf + ((tid >> 5) & 1) * kNarrowStepLds + 2 * kMbStep * kMbStride);
      aux_lds[(tid & kMbTile ? kMbStep : 0) + (tid & 31)] = val;
    }
    const int g_cur = it / tiles_per_head;
    const int qt0 = q_first + (it - g_cur * tiles_per_head) * kMbTile;   // first query of the staged tile
    LKV_MB_LOAD_ITEM(min(it + 1, n_items - 1))   // the last iteration re-reads its own item: no branch around the loads
    __syncthreads();                             // two buffers: one barrier per item is enough
#pragma unroll
    for (int st = 0; st < kMbSteps; ++st) {
      const int qs0 = qt0 + st * kMbStep;
      // wave-uniform: nothing to do when all 32 queries come before this wave's keys, or lie past the end
      if (qs0 + kMbStep - 1 < kw0 || qs0 >= T || kw0 >= T) continue;
      const unsigned char* q_lds = buf + st * kNarrowStepLds;
      const unsigned char* g_lds = q_lds + kMbStep * kMbStride;
      const float* aux_lds = reinterpret_cast<const float*>(g_lds + kMbStep * kMbStride);
      // S and dP: lane (rb = r, key c) gets queries 16 tt + 4 r + e
      f32x4_t sacc[kKB][2], pacc[kKB][2];
#pragma unroll
      for (int kb = 0; kb < kKB; ++kb)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
          sacc[kb][tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          pacc[kb][tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const bf16x8_t qx = mb_read_straight(q_lds + (tt * 16 + c) * kMbStride + ks * 64 + r * 16);
          const bf16x8_t gx = mb_read_straight(g_lds + (tt * 16 + c) * kMbStride + ks * 64 + r * 16);
#pragma unroll
          for (int kb = 0; kb < kKB; ++kb) {
            sacc[kb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qx, kfrag[kb][ks], sacc[kb][tt], 0, 0, 0);
            pacc[kb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gx, vfrag[kb][ks], pacc[kb][tt], 0, 0, 0);
          }
        }
      bf16x8_t pfrag[kKB], dsfrag[kKB];
      auto pointwise = [&](auto edge_tag) {
        constexpr bool kEdge = decltype(edge_tag)::value;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
          const float4 l4 = *reinterpret_cast<const float4*>(aux_lds + 16 * tt + 4 * r);
          const float4 d4 = *reinterpret_cast<const float4*>(aux_lds + kMbStep + 16 * tt + 4 * r);
          const float lq[4] = {l4.x, l4.y, l4.z, l4.w};
          const float dq_[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int kb = 0; kb < kKB; ++kb) {
            const int key = kw0 + 16 * kb + c;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int query = qs0 + 16 * tt + 4 * r + e;
              float ev = mb_exp2(fmaf(sacc[kb][tt][e], qscale, -lq[e]));
              if (kEdge) ev = (key > query || query >= T) ? 0.f : ev;
              const float diff = pacc[kb][tt][e] - dq_[e];
              dm_acc[kb] = fmaf(ev, diff, dm_acc[kb]);
              const float p = ev * mkey[kb];
              pfrag[kb][tt * 4 + e] = (__bf16)p;
              dsfrag[kb][tt * 4 + e] = (__bf16)(p * diff);
            }
          }
        }
      };
      // wave-uniform: the plain path needs every query of the step at or after every key of the wave, and inside T
      if (qs0 < kw0 + kWaveK - 1 || qs0 + kMbStep > T) pointwise(std::true_type{});
      else pointwise(std::false_type{});
      // dV += P^T dO and dK += dS^T Q: B operands from the dO and Q rows by the transposing read
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) {
        const bf16x8_t gb = mb_read_transposed(g_lds, kMbStride, r, c, ct);
        const bf16x8_t qb = mb_read_transposed(q_lds, kMbStride, r, c, ct);
#pragma unroll
        for (int kb = 0; kb < kKB; ++kb) {
          acc_v[kb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pfrag[kb], gb, acc_v[kb][ct], 0, 0, 0);
          acc_k[kb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dsfrag[kb], qb, acc_k[kb][ct], 0, 0, 0);
        }
      }
    }
  }
#undef LKV_MB_LOAD_ROW
#undef LKV_MB_LOAD_ITEM
#undef LKV_MB_STORE_ROW

#pragma unroll
  for (int kb = 0; kb < kKB; ++kb) {
    float s = dm_acc[kb];
    s = sum_over_row_blocks(s);
    const int key = kw0 + 16 * kb + c;
    if (r == 0 && key < T) dm[(size_t)unit * T + key] = s;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int krow = kw0 + 16 * kb + 4 * r + e;
      if (krow < T) {
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) {
          dv[((size_t)unit * T + krow) * kHeadDim + 16 * ct + c] = acc_v[kb][ct][e];
          dk[((size_t)unit * T + krow) * kHeadDim + 16 * ct + c] = acc_k[kb][ct][e] * scale;
        }
      }
    }
  }
}

// dk, dv and dm of every KV head: the sums of its `split` partial results, in a fixed order (reproducible).  Block row
// 0 of the grid's z takes dk, 1 dv, 2 dm.
__global__ void __launch_bounds__(256)
masked_attn_bwd_reduce_kernel(const float4* __restrict__ dk_part, const float4* __restrict__ dv_part,
                              const float* __restrict__ dm_part, float4* __restrict__ dk, float4* __restrict__ dv,
                              float* __restrict__ dm, int T, int split) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int h = blockIdx.y;
  if (blockIdx.z == 2) {
    if (i >= T) return;
    const float* src = dm_part + (size_t)h * split * T + i;
    float acc = src[0];
    for (int g = 1; g < split; ++g) acc += src[(size_t)g * T];
    dm[(size_t)h * T + i] = acc;
    return;
  }
  const int64_t per_head = (int64_t)T * kHeadDim / 4;
  if (i >= per_head) return;
  const float4* src = (blockIdx.z == 0 ? dk_part : dv_part) + (size_t)h * split * per_head + i;
  float4 acc = src[0];
  for (int g = 1; g < split; ++g) {
    const float4 x = src[(size_t)g * per_head];
    acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
  }
  (blockIdx.z == 0 ? dk : dv)[(size_t)h * per_head + i] = acc;
}

hipError_t masked_attn_bwd_prepare() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(masked_attn_bwd_dkv_narrow_kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, kNarrowLds);
}

// Which dK/dV kernel, and into how many blocks the query heads of a group are dealt: the blocks of a KV head's whole
// group are few and long for short sequences (the longest walks G * T / 64 staged tiles one after the other).  The wide
// kernel where one block per query head gives it kMbFewBlocks blocks, and then the smallest divisor of G that does so;
// each more costs the partial sums' way through memory.  The narrow one below that, one block per query head when a
// group's would be fewer.  Wide against narrow, whole backward pass: 2345 tokens, 8 x 4 heads (320 wide blocks) 253
// against 234 us; 12000, 8 x 1 (376) 1158 : 1150; 4096, 8 x 4 (512) 532 : 567; 5000, 4 x 7 (560) 703 : 743.  Split and
// wide against the narrow kernel's whole groups: 8192, 8 x 4 (135 MB of partial sums) 1867 : 1976; 16384, 4 x 7 (470
// MB) 6542 : 7111; 20000, 4 x 7 (580 MB) 9616 : 11371; 5000, 16 x 2 (164 MB) 810 : 814.  Parts of unlike size, two of 4
// and 3 heads in place of seven, would take 136 MB and 7077 us at 16384, 4 x 7.
struct DkvPlan {
  bool wide;
  int split;
};
// without the wide kernel's split: what a caller gets whose workspace does not hold the partial sums
static DkvPlan dkv_narrow_plan(int n_kv_heads, int G, int T) {
  const int64_t narrow = (int64_t)((T + kNarrowBlockK - 1) / kNarrowBlockK) * n_kv_heads;
  return {false, narrow < kMbFewBlocks ? G : 1};
}
static DkvPlan dkv_plan(int n_kv_heads, int G, int T) {
  const int64_t wide = (int64_t)((T + kDkvBlockK - 1) / kDkvBlockK) * n_kv_heads;
  for (int s = 1; s <= G; ++s)
    if (G % s == 0 && wide * s >= kMbFewBlocks) return {true, s};
  return dkv_narrow_plan(n_kv_heads, G, T);
}

static size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

// workspace: D (one float per query row), then, when the dK/dV kernel is split, the partial dK, dV
// [n_kv_heads * split, T, 128] and dm [n_kv_heads * split, T]
static size_t plan_bytes(int n_q_heads, int n_kv_heads, int T, const DkvPlan& plan) {
  size_t bytes = align256((size_t)n_q_heads * (size_t)T * sizeof(float));
  const size_t units = (size_t)n_kv_heads * plan.split;
  if (plan.split > 1) bytes += 2 * align256(units * T * kHeadDim * sizeof(float)) + align256(units * T * sizeof(float));
  return bytes;
}
size_t masked_attn_bwd_workspace_bytes(int n_q_heads, int n_kv_heads, int T) {
  if (n_kv_heads < 1 || n_q_heads % n_kv_heads != 0) return align256((size_t)n_q_heads * (size_t)T * sizeof(float));
  return plan_bytes(n_q_heads, n_kv_heads, T, dkv_plan(n_kv_heads, n_q_heads / n_kv_heads, T));
}
size_t masked_attn_bwd_least_workspace_bytes(int n_q_heads, int n_kv_heads, int T) {
  const size_t narrow = plan_bytes(n_q_heads, n_kv_heads, T, dkv_narrow_plan(n_kv_heads, n_q_heads / n_kv_heads, T));
  const size_t bytes = masked_attn_bwd_workspace_bytes(n_q_heads, n_kv_heads, T);
  return narrow < bytes ? narrow : bytes;
}

void launch_masked_attn_bwd(const void* q, const void* k, const void* v, const float* m, const float* o,
                            const float* lse, const void* d_o, int n_q_heads, int n_kv_heads, int T, float scale,
                            float* dq, float* dk, float* dv, float* dm, float* workspace, size_t workspace_bytes,
                            hipStream_t stream) {
  const int G = n_q_heads / n_kv_heads;
  const int64_t n_rows = (int64_t)n_q_heads * T;
  hipLaunchKernelGGL(masked_attn_bwd_dq_kernel, dim3((T + kDqBlockQ - 1) / kDqBlockQ * n_q_heads), dim3(kMbThreads), 0,
                     stream, static_cast<const uint16_t*>(q), static_cast<const uint4*>(k), static_cast<const uint4*>(v), m,
                     lse, workspace, o, static_cast<const uint16_t*>(d_o), T, n_q_heads, G, scale, dq);
  DkvPlan plan = dkv_plan(n_kv_heads, G, T);
  if (workspace_bytes < plan_bytes(n_q_heads, n_kv_heads, T, plan)) plan = dkv_narrow_plan(n_kv_heads, G, T);
  const int split = plan.split;
  const int n_units = n_kv_heads * split;
  unsigned char* ws = reinterpret_cast<unsigned char*>(workspace);
  float* dk_part = reinterpret_cast<float*>(ws + align256((size_t)n_rows * sizeof(float)));
  float* dv_part = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(dk_part) + align256((size_t)n_units * T * kHeadDim * sizeof(float)));
  float* dm_part = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(dv_part) + align256((size_t)n_units * T * kHeadDim * sizeof(float)));
  const int block_keys = plan.wide ? kDkvBlockK : kNarrowBlockK;
  hipLaunchKernelGGL(plan.wide ? masked_attn_bwd_dkv_kernel : masked_attn_bwd_dkv_narrow_kernel,
                     dim3((T + block_keys - 1) / block_keys * n_units), dim3(plan.wide ? kDkvThreads : kNarrowThreads),
                     plan.wide ? 0 : kNarrowLds, stream, static_cast<const uint4*>(q), static_cast<const uint16_t*>(k),
                     static_cast<const uint16_t*>(v), m, lse, workspace, static_cast<const uint4*>(d_o), T, n_kv_heads, G,
                     split, scale, split > 1 ? dk_part : dk, split > 1 ? dv_part : dv, split > 1 ? dm_part : dm);
  if (split > 1)
    hipLaunchKernelGGL(masked_attn_bwd_reduce_kernel, dim3((unsigned)(((int64_t)T * kHeadDim / 4 + 255) / 256), n_kv_heads, 3),
                       dim3(256), 0, stream, reinterpret_cast<const float4*>(dk_part), reinterpret_cast<const float4*>(dv_part),
                       dm_part, reinterpret_cast<float4*>(dk), reinterpret_cast<float4*>(dv), dm, T, split);
}

}  // namespace lkv
