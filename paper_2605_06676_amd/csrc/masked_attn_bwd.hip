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
// Three kernels (four for short sequences), no atomics, every output element written once:
//   masked_attn_bwd_prep_kernel   D_i for every query row.
//   masked_attn_bwd_dkv_kernel    one block (eight waves, 32 keys each) per KV head and 256 keys: the K rows of
//                                 the block stay in registers as matrix operands, its V rows in LDS, the Q and dO rows of
//                                 all later queries (and of every query head of the group) stream through LDS; yields
//                                 dK, dV and dm of its keys.  When that gives too few blocks the query heads of a group
//                                 are dealt to several and a reduce kernel adds the partial results in a fixed order.
//   masked_attn_bwd_dkv_narrow_kernel   the same with 16 keys per wave, for short sequences.
//   masked_attn_bwd_dq_kernel     one block per query head and 128 queries: Q and dO rows in registers,
//                                 K and V rows of all earlier keys stream through LDS; yields dQ.
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

// D_i = dO_i . o_i: sixteen lanes per row, eight channels of each tensor per lane
__global__ void __launch_bounds__(256)
masked_attn_bwd_prep_kernel(const float4* __restrict__ o, const uint4* __restrict__ d_o, int64_t n_rows,
                            float* __restrict__ dvec) {
  const int64_t row = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int c = threadIdx.x & 15;
  const int64_t src = min(row, n_rows - 1);
  const float4 a0 = o[(src * kChunksPerRow + c) * 2], a1 = o[(src * kChunksPerRow + c) * 2 + 1];
  float b[8];
  unpack8(d_o[src * kChunksPerRow + c], b);
  float acc = a0.x * b[0];
  acc = fmaf(a0.y, b[1], acc);
  acc = fmaf(a0.z, b[2], acc);
  acc = fmaf(a0.w, b[3], acc);
  acc = fmaf(a1.x, b[4], acc);
  acc = fmaf(a1.y, b[5], acc);
  acc = fmaf(a1.z, b[6], acc);
  acc = fmaf(a1.w, b[7], acc);
  acc = row16_allreduce_sum(acc);
  if (c == 0 && row < n_rows) dvec[row] = acc;
}

// ---- dQ ------------------------------------------------------------------------------------------
// per 32-key step buffer: K rows (also read transposed), V rows, the 32 mask weights
constexpr int kDqStepLds = kMbStep * 2 * kMbStride + kMbStep * 4;
constexpr int kDqLds = 2 * kMbSteps * kDqStepLds;

template <int kQB>
__global__ void __launch_bounds__(kMbThreads, 2)
masked_attn_bwd_dq_kernel(const uint16_t* __restrict__ q, const uint4* __restrict__ k, const uint4* __restrict__ v,
                          const float* __restrict__ m, const float* __restrict__ lse, const float* __restrict__ dvec,
                          const uint16_t* __restrict__ d_o, int T, int n_heads, int G, float scale, float* __restrict__ dq) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kWaveQ = 16 * kQB;
  constexpr int kBlockQ = kMbWaves * kWaveQ;
  constexpr int kTileLds = kMbSteps * kDqStepLds;
  const int n_qtiles = (T + kBlockQ - 1) / kBlockQ;
  // blocks in order of decreasing work: query tile slow, head fast
  const int qtile = n_qtiles - 1 - (int)blockIdx.x / n_heads;
  const int hq = (int)blockIdx.x % n_heads;
  const int h = hq / G;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int r = lane >> 4;
  const int c = lane & 15;
  const int q0 = qtile * kBlockQ;
  const int qw0 = q0 + wave * kWaveQ;
  const int n_tiles = (min(q0 + kBlockQ, T) + kMbTile - 1) / kMbTile;
  const float qscale = scale * kMbLog2e;

  // B operands of the first products: lane (query c of block qb, K-block r) holds 8 channels of q and of dO
  bf16x8_t qfrag[kQB][4], gfrag[kQB][4];
  float lse2[kQB], dsum[kQB];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) {
    const int query = min(qw0 + 16 * qb + c, T - 1);   // queries past the end repeat the last one; never stored
    const size_t row = (size_t)hq * T + query;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      qfrag[qb][ks] = __builtin_bit_cast(bf16x8_t, reinterpret_cast<const uint4*>(q + row * kHeadDim)[ks * 4 + r]);
      gfrag[qb][ks] = __builtin_bit_cast(bf16x8_t, reinterpret_cast<const uint4*>(d_o + row * kHeadDim)[ks * 4 + r]);
    }
    const float l = lse[row];
    lse2[qb] = l == -INFINITY ? INFINITY : l * kMbLog2e;   // no weight in the prefix: every e_ij becomes 0
    dsum[qb] = dvec[row];
  }
  f32x4_t acc[kQB][8];              // dQ[query 4 r + e of block qb][channel 16 ct + c], before the scale
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc[qb][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const uint4* kh = k + (size_t)h * T * kChunksPerRow;
  const uint4* vh = v + (size_t)h * T * kChunksPerRow;
  const float* mh = m + (size_t)h * T;
  const int srow = tid >> 4, spiece = tid & 15;
  // named staging registers (arrays of them ended up in scratch memory)
  uint4 k_s0, k_s1, k_s2, k_s3, v_s0, v_s1, v_s2, v_s3;
  float mk;
#define LKV_MB_LOAD_ROW(j_, kreg_, vreg_, t_)                                                             \
  {                                                                                                       \
    const int key = min((t_) * kMbTile + srow + 16 * (j_), T - 1); /* past the end: the last row, unused */ \
    const uint32_t off = (uint32_t)key * 256u + (uint32_t)spiece * 16u; /* 32-bit offset, uniform base */ \
    kreg_ = *reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned char*>(kh) + off);            \
    vreg_ = *reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned char*>(vh) + off);            \
  }
#define LKV_MB_LOAD_TILE(t_)                                      \
  {                                                               \
    LKV_MB_LOAD_ROW(0, k_s0, v_s0, t_)                            \
    LKV_MB_LOAD_ROW(1, k_s1, v_s1, t_)                            \
    LKV_MB_LOAD_ROW(2, k_s2, v_s2, t_)                            \
    LKV_MB_LOAD_ROW(3, k_s3, v_s3, t_)                            \
    mk = mh[min((t_) * kMbTile + (tid & (kMbTile - 1)), T - 1)];  \
  }
#define LKV_MB_STORE_ROW(j_, kreg_, vreg_)                                                                   \
  {                                                                                                          \
    unsigned char* step_buf = buf + ((j_) >> 1) * kDqStepLds;                                                \
    const int row = srow + 16 * ((j_) & 1);                                                                  \
    *reinterpret_cast<uint4*>(step_buf + row * kMbStride + spiece * 16) = kreg_;                            \
    *reinterpret_cast<uint4*>(step_buf + kMbStep * kMbStride + row * kMbStride + spiece * 16) = vreg_;     \
  }
  LKV_MB_LOAD_TILE(0)

#pragma unroll 1
  for (int t = 0; t < n_tiles; ++t) {
    unsigned char* buf = smem + (t & 1) * kTileLds;
    LKV_MB_STORE_ROW(0, k_s0, v_s0)
    LKV_MB_STORE_ROW(1, k_s1, v_s1)
    LKV_MB_STORE_ROW(2, k_s2, v_s2)
    LKV_MB_STORE_ROW(3, k_s3, v_s3)
    if (tid < kMbTile)
      reinterpret_cast<float*>(buf + (tid >> 5) * kDqStepLds + kMbStep * 2 * kMbStride)[tid & 31] = mk;
    LKV_MB_LOAD_TILE(min(t + 1, n_tiles - 1))   // the last iteration re-reads its own tile: no branch around the loads
    __syncthreads();                            // two buffers: one barrier per tile is enough
    const int key0 = t * kMbTile;
    if (key0 <= qw0 + kWaveQ - 1 && qw0 < T) {  // wave-uniform: otherwise the tile lies above this wave's diagonal
      const bool diagonal = key0 + kMbTile - 1 > qw0;   // some key of the tile lies above some query's diagonal
#pragma unroll
      for (int st = 0; st < kMbSteps; ++st) {
        const unsigned char* k_lds = buf + st * kDqStepLds;
        const unsigned char* v_lds = k_lds + kMbStep * kMbStride;
        const float* m_lds = reinterpret_cast<const float*>(v_lds + kMbStep * kMbStride);
        // S^T and dP^T for the two 16-key halves of the step: lane (rb = r, query c) gets keys 16 tt + 4 r + e
        f32x4_t sacc[kQB][2], pacc[kQB][2];
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) {
            sacc[qb][tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            pacc[qb][tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const bf16x8_t kx = mb_read_straight(k_lds + (tt * 16 + c) * kMbStride + ks * 64 + r * 16);
            const bf16x8_t vx = mb_read_straight(v_lds + (tt * 16 + c) * kMbStride + ks * 64 + r * 16);
#pragma unroll
            for (int qb = 0; qb < kQB; ++qb) {
              sacc[qb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kx, qfrag[qb][ks], sacc[qb][tt], 0, 0, 0);
              pacc[qb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vx, gfrag[qb][ks], pacc[qb][tt], 0, 0, 0);
            }
          }
        bf16x8_t dsfrag[kQB];
        auto pointwise = [&](auto diag_tag) {
          constexpr bool kDiag = decltype(diag_tag)::value;
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) {
            const float4 mw4 = *reinterpret_cast<const float4*>(m_lds + 16 * tt + 4 * r);
            const float mw[4] = {mw4.x, mw4.y, mw4.z, mw4.w};
#pragma unroll
            for (int qb = 0; qb < kQB; ++qb) {
              const int query = qw0 + 16 * qb + c;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                float ev = mb_exp2(fmaf(sacc[qb][tt][e], qscale, -lse2[qb]));
                if (kDiag) ev = key0 + 32 * st + 16 * tt + 4 * r + e > query ? 0.f : ev;
                const float ds = ev * mw[e] * (pacc[qb][tt][e] - dsum[qb]);
                dsfrag[qb][tt * 4 + e] = (__bf16)ds;
              }
            }
          }
        };
        if (diagonal) pointwise(std::true_type{});   // wave-uniform
        else pointwise(std::false_type{});
        // dQ += dS K: B operand from the K rows by the transposing read
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) {
          const bf16x8_t kb = mb_read_transposed(k_lds, kMbStride, r, c, ct);
#pragma unroll
          for (int qb = 0; qb < kQB; ++qb)
            acc[qb][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dsfrag[qb], kb, acc[qb][ct], 0, 0, 0);
        }
      }
    }
  }
#undef LKV_MB_LOAD_ROW
#undef LKV_MB_LOAD_TILE
#undef LKV_MB_STORE_ROW

#pragma unroll
  for (int qb = 0; qb < kQB; ++qb)
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
  int next_head = 0, next_q0 = k0;   // the item to be fetched next: query head of the group, first query
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
    next_q0 += kMbTile;
    if (next_q0 >= T) {              // past the last item this wraps to rows nobody multiplies
      next_q0 = k0;
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
  int q0 = k0;   // first query of the current item
  auto item = [&](const unsigned char* tile, const float* aux_lds) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < kMbSteps; ++st) {
      const int qs0 = q0 + st * kMbStep;
      // wave-uniform: nothing to do when all 32 queries come before this wave's keys, or lie past the end
      if (qs0 + kMbStep - 1 >= kw0 && qs0 < T && kw0 < T) step(tile + st * kMbStep * kDkvRow, aux_lds + st * kMbStep, qs0);
    }
    q0 = q0 + kMbTile < T ? q0 + kMbTile : k0;
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
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(masked_attn_bwd_dq_kernel<2>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kDqLds);
  if (e != hipSuccess) return e;
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
  hipLaunchKernelGGL(masked_attn_bwd_prep_kernel, dim3((unsigned)((n_rows + 15) / 16)), dim3(256), 0, stream,
                     reinterpret_cast<const float4*>(o), static_cast<const uint4*>(d_o), n_rows, workspace);
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
  hipLaunchKernelGGL(masked_attn_bwd_dq_kernel<2>, dim3((T + 127) / 128 * n_q_heads), dim3(kMbThreads), kDqLds, stream,
                     static_cast<const uint16_t*>(q), static_cast<const uint4*>(k), static_cast<const uint4*>(v), m, lse,
                     workspace, static_cast<const uint16_t*>(d_o), T, n_q_heads, G, scale, dq);
  if (split > 1)
    hipLaunchKernelGGL(masked_attn_bwd_reduce_kernel, dim3((unsigned)(((int64_t)T * kHeadDim / 4 + 255) / 256), n_kv_heads, 3),
                       dim3(256), 0, stream, reinterpret_cast<const float4*>(dk_part), reinterpret_cast<const float4*>(dv_part),
                       dm_part, reinterpret_cast<float4*>(dk), reinterpret_cast<float4*>(dv), dm, T, split);
}

}  // namespace lkv
