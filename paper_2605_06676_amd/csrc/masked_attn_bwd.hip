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
//   masked_attn_bwd_dkv_kernel    one block of eight waves per KV head and 256 (or 128) keys, 32 keys a wave: the K rows
//                                 stay in registers as matrix operands, the V rows in LDS, the Q and dO rows of
//                                 all later queries (and of every query head of the group) stream through LDS; yields
//                                 dK, dV and dm of its keys.  When that gives too few blocks the query heads of a group
//                                 are dealt to several and a reduce kernel adds the partial results in a fixed order.
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

constexpr float kMbLog2e = 1.4426950408889634f;

constexpr int kMbFewBlocks = 512;              // dK/dV grids below this leave compute units idle or wait for their longest block

__device__ __forceinline__ float mb_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bf16x8_t mb_read_straight(const unsigned char* p) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(p));
}

// Permutation of the 16-byte pieces of staged row `row`: piece p lies at slot p ^ row_turn(row).  With it neither the
// straight reads (16 rows of one piece) nor the transposing ones (32 bytes of each of eight rows at a time) meet a bank
// twice (measured; 2 (row % 8) + row / 8 and two others cost 18 to 29 % of the kernel's cycles in conflicts).
__device__ __forceinline__ int row_turn(int row) { return 2 * row & 15; }

// base ^ kBits, worked out where it is used: the compiler would keep every such address in a register of its own
template <uint32_t kBits>
__device__ __forceinline__ uint32_t address_xor(uint32_t base) {
  uint32_t at;
  asm volatile("v_xor_b32 %0, %2, %1" : "=v"(at) : "v"(base), "i"(kBits));
  return at;
}

// B operand of a product whose K dimension runs over the 32 staged rows of a step: lane (r, c) gets, for output column c,
// rows 4r..4r+3 and 16+4r..16+4r+3 (the K-slot order in which the first products leave their results); p is where the
// lane's rows 4r + c / 4 (and 16 further on) hold its channels
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
// into eight pieces of six products, the operands of the next piece and an eighth of the dS, which it may not mix.  K rows
// for the products are read a piece ahead, the others as soon as the products before have taken theirs (with all of them so
// 85.6 instead of 82.3 us at 2345 tokens, 113 instead of 102 for 8 and 8 heads of 4096; all a piece ahead does not fit).  The
// rows go from memory to LDS directly; a ring of four K slots holds what steps s - 1 to s + 2 need, two V slots s + 1 and
// s + 2 (53 KB, two blocks per compute unit; tiles of 64 keys would need 80 KB).  D_i is summed here on the way in, from
// rows that the block needs anyhow, and left for the dK/dV kernel: a launch of its own took 65 us at 16384 tokens, 9.4 at
// 2345.  32 query heads, 8 KV heads, in turn with a kernel that did one thing after the other and staged through
// registers: 2960 -> 2680 us at 16384 tokens (1230 TFLOP/s), 216 -> 191 at 4096, 97 -> 82 at 2345; 8 and 8 heads of 4096
// 143 -> 102.
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
    auto piece_of_step = [&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value;
      constexpr int tt = i >> 2, ks = i & 3, qp = (i >> 1) & 1, e0 = 2 * (i & 1);
      bf16x8_t kbn = kb;
      if constexpr (i < 7) kbn = mb_read_turned(k_prev + address_xor<32 * (i + 1)>(turned));
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
        const uint32_t at = ((i + 1) >> 2) * 16 * kDqRow + (((i + 1) & 3) == 0 ? straight : address_xor<64 * ((i + 1) & 3)>(straight));
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
      kb = kbn;
    };
    piece_of_step(std::integral_constant<int, 0>());
    piece_of_step(std::integral_constant<int, 1>());
    piece_of_step(std::integral_constant<int, 2>());
    piece_of_step(std::integral_constant<int, 3>());
    piece_of_step(std::integral_constant<int, 4>());
    piece_of_step(std::integral_constant<int, 5>());
    piece_of_step(std::integral_constant<int, 6>());
    piece_of_step(std::integral_constant<int, 7>());
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
constexpr int dkv_block_keys(int groups) { return kDkvThreads / 64 / groups * kDkvWaveK; }
constexpr int kDkvRow = 256;                   // LDS bytes per staged row: rows lie as in memory, their 16-byte pieces permuted
constexpr int kDkvStepLds = 2 * kMbStep * kDkvRow;   // Q rows, dO rows of one step of 32 queries

// kGroups = 1: eight waves of 32 keys, each takes every step of 32 queries.  kGroups = 2: four times 32 keys, two waves
// take the steps in turn and their sums are joined at the end, which halves the chain of steps per key (short sequences).
//
// Bound by instruction issue (16384 tokens: matrix pipe busy for 53 % of the cycles, vector pipe 47 %, 14 % together, LDS
// 57 %, no conflicts) and by waiting for LDS operands, at 2.0 GHz where the dQ kernel, busy for 97 %, holds 1.9.  A step
// is a pipeline inside the wave: P and dS of its first 16 queries beside S and dP of the other 16, theirs beside S and dP
// of the next step's first 16, then the products with all 32; the pieces are fenced so that the compiler keeps
// exponentials beside products.  Operands are read a piece ahead, also from one half to the next, into the products and
// on to the next step (without that over these seams: 4.37 ms instead of 4.19 at 16384 tokens, 129 us instead of 126 at
// 2345, 127 instead of 120 for 8 and 8 heads of 4096).  32 keys per wave need 128 accumulator and 32 K operand registers;
// V operands come from LDS, 48 KB are read per 64 matrix instructions.  256 registers are just enough, without a spill, and
// only so: one loop with one way out (with breaks or a second loop for the diagonal the compiler keeps several sets of sums,
// and spills), masks set in place in a branch around nothing else, addresses worked out where they are used.  A step wholly
// above a wave's diagonal passes through the pipeline with S = -inf and dP - D = 0 and leaves the products out: its weights
// are 0, but 0 times a row that is not finite is not (whole backward pass, in turn with multiplying it all the same: 79.0 ->
// 77.1 us at 1024 tokens, 1674 -> 1648 at 8192, 6549 -> 6422 at 16384; a branch around the whole step
// spills, 3 % slower).  32 query heads, 8 KV heads, in turn with a kernel that did one thing after the other: 4.59 -> 4.10 ms
// at 16384 tokens, 136 -> 126 us at 2345 (kGroups = 2); 8 and 8 heads of 4096 140 -> 120.  Measured and dropped: P and dS of the first 16 beside the
// products (spills; 3 to 20 % slower), 16 keys per wave with V in registers (64 KB of operands per 64 matrix
// instructions, LDS busy 78 %; 136 us at 2345), pairs of waves that share 32 keys, halve the queries of S and dP and the
// channels of dK and dV and swap P and dS through LDS (one barrier between any two uses; 133 us at 2345, 5.12 ms at
// 16384), four waves and 128 keys a block, two blocks per compute unit (143 us and 4.9 ms).
template <int kGroups>
__global__ void __launch_bounds__(kDkvThreads, 2)
masked_attn_bwd_dkv_kernel(const uint4* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                           const float* __restrict__ m, const float* __restrict__ lse, const float* __restrict__ dvec,
                           const uint4* __restrict__ d_o, int T, int n_kv_heads, int G, int split, float scale,
                           float* __restrict__ dk, float* __restrict__ dv, float* __restrict__ dm) {
  constexpr int kBlockK = dkv_block_keys(kGroups);
  constexpr int kItemQ = kGroups * kMbStep;      // queries of an item: a step for every group
  // An array per slot: the compiler then knows that reads of one do not touch the rows on their way to another.
  __shared__ __align__(1024) unsigned char slot_a[kGroups * kDkvStepLds], slot_b[kGroups * kDkvStepLds], slot_c[kGroups * kDkvStepLds];
  __shared__ __align__(1024) unsigned char v_rows[kBlockK * kDkvRow];   // the block's V rows, read as operands in every step
  __shared__ __align__(16) float aux_a[2 * kItemQ], aux_b[2 * kItemQ], aux_c[2 * kItemQ];   // per step: lse (log2 domain), -D
  // A block owns kBlockK keys of one KV head and the query heads g_lo .. g_lo + g_cnt - 1 of its group: all of them
  // (split = 1, results go straight to dk, dv, dm) or an equal share (split divides G: results are partial sums, row
  // `unit` of buffers the host passes in place of the outputs, added up by the reduce kernel).  Blocks in order of
  // decreasing work: early keys have the most queries after them; key tile slow, unit fast.
  const int n_units = n_kv_heads * split;
  const int unit = (int)blockIdx.x % n_units;
  const int h = unit / split;
  const int g_cnt = G / split;
  const int g_lo = (unit - h * split) * g_cnt;
  const int k0 = (int)blockIdx.x / n_units * kBlockK;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane >> 4;
  const int c = lane & 15;
  const int key_wave = wave & (kDkvThreads / 64 / kGroups - 1);   // the wave's 32 keys
  const int group = wave / (kDkvThreads / 64 / kGroups);          // and, of kGroups = 2, its 32 queries of an item
  const int kw0 = k0 + key_wave * kDkvWaveK;
  const float qscale = scale * kMbLog2e;

  // Streamed items: for every query head of the group, tiles of queries from the last one down to the block's diagonal.
  // Blocks of one KV head run on one XCD (where the units divide by 8) and meet the same rows at the same time, in its L2
  // (4096 tokens, 8 x 4 heads: 295 -> 288 us against walking up from the diagonal; 16384: 4731 -> 4706).
  const int n_items = g_cnt * ((T - k0 + kItemQ - 1) / kItemQ);
  // Staging, straight from memory into LDS: a wave instruction fills 1 KB, four rows; lane (row slot, piece slot) fetches
  // piece `slot ^ f(row)` of its row (row_turn above), so that both the straight reads (eight rows of one piece at a time)
  // and the transposing reads (four rows of 32 bytes) find their banks apart.
  const int srow = tid >> 4;
  const uint32_t piece = (uint32_t)(((tid & 15) ^ row_turn(srow)) * 16);
  float aux = 0.f;   // wave w < kGroups: lse of query lane % 32 of step w; the next kGroups waves: its D
  const int q_last = k0 + (T - 1 - k0) / kItemQ * kItemQ;   // first query of the last item
  int next_head = 0, next_q0 = q_last;   // the item to be fetched next: query head of the group, first query
  int aux_q0 = 0;                        // first query of this wave's aux
  auto fetch = [&](unsigned char* dst) __attribute__((always_inline)) {
    const size_t base = ((size_t)h * G + g_lo + next_head) * T;
    const unsigned char* qs = reinterpret_cast<const unsigned char*>(q + base * kChunksPerRow);
    const unsigned char* gs = reinterpret_cast<const unsigned char*>(d_o + base * kChunksPerRow);
#pragma unroll
    for (int j = 0; j < kGroups; ++j) {
      const uint32_t at = (uint32_t)min(next_q0 + srow + kMbStep * j, T - 1) * 256u + piece;   // past the end: the last row, masked later
      lds_fill16(qs + at, dst + j * kDkvStepLds + 4 * wave * kDkvRow);
      lds_fill16(gs + at, dst + j * kDkvStepLds + (kMbStep + 4 * wave) * kDkvRow);
    }
    aux_q0 = next_q0 + kMbStep * (wave % kGroups);
    if (wave < 2 * kGroups) {
      const uint32_t at = (uint32_t)min(aux_q0 + (lane & 31), T - 1) * 4u;
      aux = *reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>((wave < kGroups ? lse : dvec) + base) + at);
    }
    next_q0 -= kItemQ;
    if (next_q0 < k0) {              // past the last item this wraps to rows nobody multiplies
      next_q0 = q_last;
      next_head = next_head + 1 < g_cnt ? next_head + 1 : 0;
    }
  };
  auto put_aux = [&](float* dst) __attribute__((always_inline)) {
    // lse goes to the log2 domain; -inf (no weight in the prefix, or a query past the end) becomes +inf: every e_ij is 0
    if (wave < 2 * kGroups) {
      float val = -aux;
      if (wave < kGroups) val = aux == -INFINITY || aux_q0 + (lane & 31) >= T ? INFINITY : aux * kMbLog2e;
      int at = lane & 31;
      asm volatile("" : "+v"(at));   // or the compiler keeps the address in each of the three arrays
      dst[at + kMbStep * (2 * (wave % kGroups) + wave / kGroups)] = val;   // (lanes 32 apart write the same)
    }
  };
  fetch(slot_a);
  put_aux(aux_a);
  fetch(slot_b);
#pragma unroll
  for (int j = 0; j < kBlockK / 32; ++j)
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

  const uint32_t v_straight = straight + key_wave * kDkvWaveK * kDkvRow;

  // carried from step to step: S and dP - D of a step's first 16 queries: lane (rb = r, key c) has queries 4 r + e
  f32x4_t sx[kDkvKB], px[kDkvKB];
  uint32_t pw[kDkvKB][4], dw[kDkvKB][4];   // P and dS of a step, as operands
  auto frag = [&](const uint32_t (&w)[4]) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
  };
  // S and dP - D of 16 queries of a step
  auto logits = [&](const unsigned char* rows, const float* aux_lds, int tt) __attribute__((always_inline)) {
    const f32x4_t nd = *reinterpret_cast<const f32x4_t*>(aux_lds + kMbStep + 16 * tt + 4 * r);
#pragma unroll
    for (int kb = 0; kb < kDkvKB; ++kb) { sx[kb] = f32x4_t{0.f, 0.f, 0.f, 0.f}; px[kb] = nd; }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const bf16x8_t gx = mb_read_straight(rows + (kMbStep + tt * 16) * kDkvRow + (straight ^ (64 * ks)));
      const bf16x8_t qx = mb_read_straight(rows + tt * 16 * kDkvRow + (straight ^ (64 * ks)));
#pragma unroll
      for (int kb = 0; kb < kDkvKB; ++kb) {
        const bf16x8_t vx = mb_read_straight(v_rows + kb * 16 * kDkvRow + (v_straight ^ (64 * ks)));
        px[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gx, vx, px[kb], 0, 0, 0);
        sx[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qx, kfrag[kb][ks], sx[kb], 0, 0, 0);
      }
    }
  };
  bf16x8_t gx, qx, vx0, vx1;   // operands of the next products of S and dP, on their way
  auto first_operands = [&](const unsigned char* rows) __attribute__((always_inline)) {   // those of a step's last 16 queries
    gx = mb_read_straight(rows + (kMbStep + 16) * kDkvRow + straight);
    qx = mb_read_straight(rows + 16 * kDkvRow + straight);
    vx0 = mb_read_straight(v_rows + v_straight);
    vx1 = mb_read_straight(v_rows + v_straight + 16 * kDkvRow);
  };
  // dV += P^T dO and dK += dS^T Q: B operands from the dO and Q rows by the transposing read, gb and qb the first of them;
  // the first operands of the step that follows come after the last
  auto products = [&](const unsigned char* rows, bf16x8_t gb, bf16x8_t qb, const unsigned char* next) __attribute__((always_inline)) {
    auto tile = [&](auto ct_tag) __attribute__((always_inline)) {
      constexpr int ct = decltype(ct_tag)::value;
      bf16x8_t g1, q1;
      if constexpr (ct < 7) {
        const uint32_t at = address_xor<32 * (ct + 1)>(turned);
        g1 = mb_read_turned(rows + kMbStep * kDkvRow + at);
        q1 = mb_read_turned(rows + at);
      } else {
        first_operands(next);
      }
#pragma unroll
      for (int kb = 0; kb < kDkvKB; ++kb) {
        acc_v[kb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(pw[kb]), gb, acc_v[kb][ct], 0, 0, 0);
        acc_k[kb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(dw[kb]), qb, acc_k[kb][ct], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (ct < 7) { gb = g1; qb = q1; }
    };
    tile(std::integral_constant<int, 0>());
    tile(std::integral_constant<int, 1>());
    tile(std::integral_constant<int, 2>());
    tile(std::integral_constant<int, 3>());
    tile(std::integral_constant<int, 4>());
    tile(std::integral_constant<int, 5>());
    tile(std::integral_constant<int, 6>());
    tile(std::integral_constant<int, 7>());
  };
  // P and dS of two queries: elements e, e + 1 of key block kb
  auto pair = [&](const f32x4_t (&sv)[kDkvKB], const f32x4_t (&pv)[kDkvKB], float to_log2, const float (&lq)[4], int tt, int kb, int e)
      __attribute__((always_inline)) {
    bf16x2_t a, b;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float ev = mb_exp2(fmaf(sv[kb][e + j], to_log2, -lq[e + j]));
      dm_acc[kb] = fmaf(ev, pv[kb][e + j], dm_acc[kb]);
      const float p = ev * mkey[kb];
      a[j] = (__bf16)p;
      b[j] = (__bf16)(p * pv[kb][e + j]);
    }
    uint32_t &pa = pw[kb][2 * tt + (e >> 1)], &da = dw[kb][2 * tt + (e >> 1)];
    pa = __builtin_bit_cast(uint32_t, a);
    da = __builtin_bit_cast(uint32_t, b);
    asm volatile("" : "+v"(pa), "+v"(da), "+v"(dm_acc[kb]));   // due here, beside the products
  };
  // One step of the pipeline: P and dS of its first 16 queries beside S and dP of the others, theirs beside S and dP of the
  // next step's first 16, then the products.  below: query less key of element 0 of key block 0 in this lane; meets: some
  // query of the step, inside the sequence, sees some key of the wave.
  auto step = [&](const unsigned char* cur, const float* aux_cur, const unsigned char* next, const float* aux_next,
                  bool diagonal, int below, bool meets) __attribute__((always_inline)) {
    f32x4_t s1[kDkvKB], p1[kDkvKB];
    bf16x8_t gb, qb;
    auto half = [&](auto tt_tag) __attribute__((always_inline)) {
      // tt = 0: from sx, px of `cur` to s1, p1 of its second half; tt = 1: from those to sx, px of `next`
      constexpr int tt = decltype(tt_tag)::value;
      const float4 l4 = *reinterpret_cast<const float4*>(aux_cur + 16 * tt + 4 * r);
      float lq[4] = {l4.x, l4.y, l4.z, l4.w};
      const f32x4_t nd = *reinterpret_cast<const f32x4_t*>(tt == 0 ? aux_cur + kMbStep + 16 + 4 * r : aux_next + kMbStep + 4 * r);
      float to_log2 = qscale;
      if (diagonal) {   // wave-uniform: some key of the wave comes after some query of the step
        // such a pair weighs 0 whatever the query's normaliser and D are, so the normaliser comes off here and not in pair()
#pragma unroll
        for (int kb = 0; kb < kDkvKB; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            f32x4_t &s = (tt == 0 ? sx : s1)[kb], &p = (tt == 0 ? px : p1)[kb];
            const bool unseen = below < 16 * kb - (16 * tt + e);
            s[e] = unseen ? -INFINITY : fmaf(s[e], qscale, -lq[e]);
            p[e] = unseen ? 0.f : p[e];
          }
#pragma unroll
        for (int e = 0; e < 4; ++e) lq[e] = 0.f;
        to_log2 = 1.f;
      }
      const unsigned char* g_at = tt == 0 ? cur + (kMbStep + 16) * kDkvRow : next + kMbStep * kDkvRow;
      const unsigned char* q_at = tt == 0 ? cur + 16 * kDkvRow : next;
      f32x4_t(&so)[kDkvKB] = tt == 0 ? s1 : sx;
      f32x4_t(&po)[kDkvKB] = tt == 0 ? p1 : px;
      auto part = [&](auto ks_tag) __attribute__((always_inline)) {
        constexpr int ks = decltype(ks_tag)::value;
        po[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gx, vx0, ks == 0 ? nd : po[0], 0, 0, 0);
        po[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gx, vx1, ks == 0 ? nd : po[1], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);   // the next operands after these products have taken theirs
        uint32_t at = straight;
        if constexpr (ks < 3) {
          at = address_xor<64 * (ks + 1)>(straight);
          const uint32_t v_at = address_xor<64 * (ks + 1)>(v_straight);
          gx = mb_read_straight(g_at + at);
          vx0 = mb_read_straight(v_rows + v_at);
          vx1 = mb_read_straight(v_rows + v_at + 16 * kDkvRow);
        } else if constexpr (tt == 0) {
          gx = mb_read_straight(next + kMbStep * kDkvRow + straight);
          vx0 = mb_read_straight(v_rows + v_straight);
          vx1 = mb_read_straight(v_rows + v_straight + 16 * kDkvRow);
        } else {
          gb = mb_read_turned(cur + kMbStep * kDkvRow + turned);
        }
#pragma unroll
        for (int kb = 0; kb < kDkvKB; ++kb)
          so[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qx, kfrag[kb][ks], ks == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : so[kb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ks < 3) qx = mb_read_straight(q_at + at);
        else if constexpr (tt == 0) qx = mb_read_straight(next + straight);
        else qb = mb_read_turned(cur + turned);
        if (tt == 0) pair(sx, px, to_log2, lq, 0, ks >> 1, 2 * (ks & 1));
        else pair(s1, p1, to_log2, lq, 1, ks >> 1, 2 * (ks & 1));
        __builtin_amdgcn_sched_barrier(0);
      };
      part(std::integral_constant<int, 0>());
      part(std::integral_constant<int, 1>());
      part(std::integral_constant<int, 2>());
      part(std::integral_constant<int, 3>());
    };
    half(std::integral_constant<int, 0>());
    half(std::integral_constant<int, 1>());
    if (meets) products(cur, gb, qb, next);   // wave-uniform
    else first_operands(next);
  };
  int q0 = q_last;   // first query of the current item
  const int lane_below = group * kMbStep + 4 * r - kw0 - c;
  // One barrier per item: every wave waits for its transfers of the item before it, so it makes the rows of the next
  // item visible, and it means that every wave is done with the slot that is filled now.  What it takes of a next item
  // that is not there is not used.
  auto item = [&](const unsigned char* cur, const float* aux_cur, const unsigned char* next, const float* aux_next,
                  unsigned char* fill, float* aux_fill) __attribute__((always_inline)) {
    lds_fill_barrier();
    fetch(fill);
    const int at = group * kDkvStepLds, aux_at = group * 2 * kMbStep;
    const int qs0 = q0 + group * kMbStep;
    step(cur + at, aux_cur + aux_at, next + at, aux_next + aux_at, qs0 < kw0 + kDkvWaveK, q0 + lane_below,
         qs0 + kMbStep > kw0 && (kGroups == 1 || qs0 < T));
    put_aux(aux_fill);
    q0 = q0 > k0 ? q0 - kItemQ : q_last;
  };
  put_aux(aux_b);
  lds_fill_barrier();
  logits(slot_a + group * kDkvStepLds, aux_a + group * 2 * kMbStep, 0);
  first_operands(slot_a + group * kDkvStepLds);
#pragma unroll 1
  for (int it = 0; it < n_items; it += 3) {
    item(slot_a, aux_a, slot_b, aux_b, slot_c, aux_c);
    if (it + 1 < n_items) item(slot_b, aux_b, slot_c, aux_c, slot_a, aux_a);
    if (it + 2 < n_items) item(slot_c, aux_c, slot_a, aux_a, slot_b, aux_b);
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): no copy may still be on its way to LDS that this block gives back

  if constexpr (kGroups == 2) {
    // the second group's sums join the first's: 16 KB per wave and matrix, lane by lane
    f32x4_t* mine = reinterpret_cast<f32x4_t*>(key_wave & 2 ? slot_b : slot_a) + (key_wave & 1) * 1024 + lane;
    auto join = [&](f32x4_t (&acc)[kDkvKB][8]) __attribute__((always_inline)) {
      lds_fill_barrier();
      if (group == 1) {
#pragma unroll
        for (int kb = 0; kb < kDkvKB; ++kb)
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) mine[(kb * 8 + ct) * 64] = acc[kb][ct];
      }
      __syncthreads();
      if (group == 0) {
#pragma unroll
        for (int kb = 0; kb < kDkvKB; ++kb)
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) acc[kb][ct] += mine[(kb * 8 + ct) * 64];
      }
    };
    join(acc_v);
    join(acc_k);
    float* dm_all = reinterpret_cast<float*>(v_rows);
    __syncthreads();
    if (group == 1)
#pragma unroll
      for (int kb = 0; kb < kDkvKB; ++kb) dm_all[(key_wave * kDkvKB + kb) * 64 + lane] = dm_acc[kb];
    __syncthreads();
    if (group == 1) return;
#pragma unroll
    for (int kb = 0; kb < kDkvKB; ++kb) dm_acc[kb] += dm_all[(key_wave * kDkvKB + kb) * 64 + lane];
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

// How many groups of waves, and into how many blocks the query heads of a group are dealt: the blocks of a KV head's whole
// group are few and long for short sequences (the longest walks G * T / 32 steps one after the other).  256 keys a block
// where one block per query head gives kMbFewBlocks blocks, and then the smallest divisor of G that does so; each more
// costs the partial sums' way through memory.  Below that 128 keys and two groups, one block per query head when a group's
// would be fewer.  Whole backward pass, this rule : kMbFewBlocks = 256 for 256 keys : 128 keys throughout.  8 x 4 heads: 2345
// tokens 207 : 226 : 207, 4096 475 : 616 : 498, 8192 1687 : 2321 : 1745, 16384 6672 : 6629 : 6721; 4 x 7: 5000 625 : 633 : 647,
// 16384 5935 : 8809 : 6089; 2 x 8: 5001 395 : 437 : 395, 16384 3209 : 4745 : 3365; 8 x 1: 9000 593 : 717 : 593.  Whole
// groups cut into equal pieces that cross key tiles, 256 blocks of equal length, gained up to 7 % at some sizes between 3000
// and 5000 tokens and lost 10 % at 1024 to its partial sums.
struct DkvPlan {
  int groups;
  int split;
};
// without a split of the 256-key blocks: what a caller gets whose workspace does not hold the partial sums
static DkvPlan dkv_short_plan(int n_kv_heads, int G, int T) {
  const int64_t blocks = (int64_t)((T + dkv_block_keys(2) - 1) / dkv_block_keys(2)) * n_kv_heads;
  return {2, blocks < kMbFewBlocks ? G : 1};
}
static DkvPlan dkv_plan(int n_kv_heads, int G, int T) {
  const int64_t blocks = (int64_t)((T + dkv_block_keys(1) - 1) / dkv_block_keys(1)) * n_kv_heads;
  for (int s = 1; s <= G; ++s)
    if (G % s == 0 && blocks * s >= kMbFewBlocks) return {1, s};
  return dkv_short_plan(n_kv_heads, G, T);
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
  const size_t shorter = plan_bytes(n_q_heads, n_kv_heads, T, dkv_short_plan(n_kv_heads, n_q_heads / n_kv_heads, T));
  const size_t bytes = masked_attn_bwd_workspace_bytes(n_q_heads, n_kv_heads, T);
  return shorter < bytes ? shorter : bytes;
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
  if (workspace_bytes < plan_bytes(n_q_heads, n_kv_heads, T, plan)) plan = dkv_short_plan(n_kv_heads, G, T);
  const int split = plan.split;
  const int n_units = n_kv_heads * split;
  unsigned char* ws = reinterpret_cast<unsigned char*>(workspace);
  float* dk_part = reinterpret_cast<float*>(ws + align256((size_t)n_rows * sizeof(float)));
  float* dv_part = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(dk_part) + align256((size_t)n_units * T * kHeadDim * sizeof(float)));
  float* dm_part = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(dv_part) + align256((size_t)n_units * T * kHeadDim * sizeof(float)));
  const int block_keys = dkv_block_keys(plan.groups);
  hipLaunchKernelGGL(plan.groups == 1 ? masked_attn_bwd_dkv_kernel<1> : masked_attn_bwd_dkv_kernel<2>,
                     dim3((T + block_keys - 1) / block_keys * n_units), dim3(kDkvThreads),
                     0, stream, static_cast<const uint4*>(q), static_cast<const uint16_t*>(k),
                     static_cast<const uint16_t*>(v), m, lse, workspace, static_cast<const uint4*>(d_o), T, n_kv_heads, G,
                     split, scale, split > 1 ? dk_part : dk, split > 1 ? dv_part : dv, split > 1 ? dm_part : dm);
  if (split > 1)
    hipLaunchKernelGGL(masked_attn_bwd_reduce_kernel, dim3((unsigned)(((int64_t)T * kHeadDim / 4 + 255) / 256), n_kv_heads, 3),
                       dim3(256), 0, stream, reinterpret_cast<const float4*>(dk_part), reinterpret_cast<const float4*>(dv_part),
                       dm_part, reinterpret_cast<float4*>(dk), reinterpret_cast<float4*>(dv), dm, T, split);
}

}  // namespace lkv
