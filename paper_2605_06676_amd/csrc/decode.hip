// One decode step of grouped-query attention over the ragged packed cache:
// Eq. 1 of the paper restricted to the kept tokens of each KV head, with all
// query heads of a GQA group reading the same segment (Sec. 3.1).
//
// Work decomposition.  Split-K over a flat list of equal chunks of packed rows:
// block c owns packed rows [c*C, (c+1)*C) whatever segments they belong to, so
// every block streams the same number of bytes however skewed the head budgets
// are.  C is chosen on the host so that the grid is a few blocks per compute
// unit.  A chunk that crosses segment boundaries is processed piece by piece.
// Each piece yields, per query head of its segment, an online-softmax partial
// (running max m, denominator l, unnormalised output acc[128]).  A piece that
// is a whole segment is normalised and written straight to the output; other
// pieces go to workspace slot (segment + chunk) -- distinct pieces get distinct
// slots because segment and chunk indices both grow along the packed rows --
// and a second, small kernel merges the slots of each segment.
//
// A chunk of several pieces is a chain of memory latencies and block barriers, one link per piece, and launches of middle
// size are bound by it.  So the four waves share only the pieces for which that pays (three barriers and a merge through
// LDS are worth about two tiles of rows); the others are dealt to single waves, which run them from load to store, each
// to the wave with least to do.  Which lengths those are is settled per chunk, from its own pieces (deal_pieces).  And a
// wave asks for the query rows and the first tile of its next piece before it multiplies the last tile of the one at hand.
// Whole call in a captured graph, when only pieces of at most 64 rows were dealt out and nothing was asked for ahead : now
// (us): 1024 segments of 400 thousand rows 58.0 : 46.4; 2048 of 500 thousand 60.0 : 53.6; 512 of 110 thousand 21.7 : 19.7; 256 of
// 1.26 million 105.2 : 102.7 (6.3 TB/s).  The prefetch alone is 1 to 7 % of it; with it, but only up to 64 rows dealt out, the
// shared pieces first: 47.9, 54.3, 19.9, 102.0.
//
// A step over up to 256 segments (all layers of a small model, one layer of a batch) is such a chain even so where the
// segments are short: there the chunks start at the segments
// instead: every wave loads the bounds of all segments at once, one or four per lane, and a prefix sum over the chunks of each
// tells its block which segment and which rows are its own.  The grid is the most chunks that any split of the rows
// over the segments can give.  (8 heads, 5 thousand rows, in a captured graph: 11.4 us with flat chunks, 8.7 us with
// these; 40 thousand rows 18.1 and 13.4 us, 160 thousand 29.6 and 25.8 us, and 18.8 us since the merge shares a segment's
// pieces out among threads; one head with nearly all of 5 thousand rows 17.8 and 10.6 us.)  Over many long segments the flat
// chunks are the better ones: they are equally long, and their grid is one round of resident blocks however the rows are
// spread.  Flat as above : starting at the segments (us, captured graph): 128 segments of 8 thousand rows in all 14.3 : 9.5 (flat with
// no pieces dealt out), 90 thousand 18.9 : 13.8, 500 thousand 47.7 : 44.6, 1.6 million 127 : 125; 256 segments of 30 thousand
// 12.6 : 11.5, 90 thousand 17.5 : 15, 250 thousand 29 : 27, 350 thousand 36.5 : 36, 500 thousand 46.9 : 48, 800 thousand 69 : 73.
//
// (Merging inside the first kernel, by the block that delivers a segment's last piece, needs device-scope fences; with
// one L2 per XCD those write back and invalidate L2 and were measured to cost more than the second launch.)
//
// Arithmetic.  With up to 16 query heads per KV head the two products are
// skinny GEMMs, and doing them on the vector ALUs costs more issue slots per
// byte than the HBM stream leaves room for, so both run on the matrix cores
// (v_mfma_f32_16x16x32_bf16, fp32 accumulate):
//   S^T[token, head] = K[token, :] . Q[head, :]^T     (A = K tile, B = Q^T)
//   O[head, ch]     += P[head, token] V[token, ch]    (A = P,      B = V tile)
// The accumulator layout of S^T (lane (rb, head) holds tokens 4rb..4rb+3 of a
// 16-token tile) is exactly the A-operand layout of P for a K-step made of two
// such tiles, so probabilities go from the first product to the second without
// leaving their lanes.  Rows are read from HBM once with coalesced 16-byte
// loads, staged in a wave-private LDS tile, and read back as operands: K by
// 16-byte reads (row stride 272 B), V by the transposing 8-byte LDS read of
// gfx950 (row stride 288 B); both strides make the reads bank-conflict free.
// The next 32 rows are prefetched into registers while the current 32 are
// multiplied.  Softmax runs in fp32 in the log2 domain.
//
// P is rounded to bf16, exactly 1 at the largest logit a wave has met.  The fewer waves a segment is cut among, the fewer such
// exact weights, and the error of the output against 64 bits rose by 1 to 3 % with chunks that start at the segments and
// with pieces dealt to single waves; so what the rounding left is multiplied too, in matrix cores that are idle next to the memory
// latencies: 1.2e-3 -> 1.8e-6, for 0 to 3 % of the time (2048 segments, 500 thousand rows 52.3 -> 53.6 us; 256 segments, 1.26
// million rows 102.3 -> 102.7), a third of it the look for infinite values, which must stay infinite.
#include <type_traits>

#include "lkv_common.h"

namespace lkv {

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / 64;
constexpr int kDecTile = 32;                 // rows per wave iteration: one K-step of the P.V product
constexpr int kDecKStride = 272;             // LDS bytes per staged K row
constexpr int kDecVStride = 288;             // LDS bytes per staged V row
constexpr int kDecWaveLds = kDecTile * (kDecKStride + kDecVStride);   // 17920
constexpr int kDecMaxGroup = 16;
constexpr int kDecSmallPiece = 2 * kDecTile; // a chunk that starts at its segment is left to one wave if it has at most this many rows
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

constexpr int kDecTargetBlocks = 512;        // chunks per launch: one round of resident blocks (2 per compute unit)
constexpr int kDecMinChunk = 128;            // rows; shorter chunks only add partials to merge
constexpr int kDecSegsPerWave = 64;          // segments whose bounds a wave loads at once
// Chunks start at the segments in launches over up to 128 segments, and over up to 256 while flat chunks would have at most
// this many rows (393 thousand in all; both sides above).
constexpr int kDecAlignedChunk = 768;
// Flat chunks, in quarters of the time of a tile: what a piece costs on top of its tiles, dealt to one wave (times four) and
// shared by all.  Shared costs of 2, 6, 12 and 20: short segments get slower below 6 (2048 segments 48.1 : 46.7 : 45.4 : 45.0
// us), 1.26 million rows above 12 (102.1 : 102.0 : 102.3 : 103.4), where waves that wait for each other's rows cost more.
constexpr int kDecAloneCost = 1;
constexpr int kDecSharedCost = 8;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Per-block LDS: the four wave tiles; after a piece, reused for the cross-wave merge.
struct DecMerge {
  float m[kDecWaves][kDecMaxGroup];
  float l[kDecWaves][kDecMaxGroup];
  float acc[kDecWaves][kDecMaxGroup][kHeadDim];
};
static_assert(sizeof(DecMerge) <= (size_t)kDecWaves * kDecWaveLds, "merge scratch must fit the staging tiles");

__device__ __forceinline__ s16x4_t lds_read_tr16(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4_t*)(p));
}

// Inclusive prefix sum over the lanes of a wave.
__device__ __forceinline__ int prefix_sum(int x) {
#define LKV_SCAN_STEP(ctrl, rows) x += __builtin_amdgcn_update_dpp(0, x, ctrl, rows, 0xf, true)
  LKV_SCAN_STEP(0x111, 0xf);   // row_shr:1, 2, 4, 8
  LKV_SCAN_STEP(0x112, 0xf);
  LKV_SCAN_STEP(0x114, 0xf);
  LKV_SCAN_STEP(0x118, 0xf);
  LKV_SCAN_STEP(0x142, 0xa);   // the last lane of a row into the rows after it
  LKV_SCAN_STEP(0x143, 0xc);
#undef LKV_SCAN_STEP
  return x;
}

// Chunks that start at the segments: which rows of which segment chunk `chunk` is, and the segment's share of the chunks.
struct AlignedChunk {
  int segment;      // -1: there are fewer chunks
  int lo, hi;       // the segment's rows in use
  int first, n;     // its chunks
};

// kSegs segments of this lane, in order over the lanes: bounds, chunk counts, and the chunks up to the lane's last.  The last
// lanes start so that their segments end with the table (n_segments >= kSegs); those that an earlier lane has count no chunks.
template <int kSegs>
struct LaneSegments {
  int lo[kSegs], hi[kSegs], n[kSegs];
  int all, upto;
};

template <int kSegs>
__device__ __forceinline__ int first_of_lane(int n_segments, int lane) { return min(kSegs * lane, n_segments - kSegs); }

template <int kSegs>
__device__ __forceinline__ LaneSegments<kSegs> lane_segments(const int32_t* __restrict__ offsets, const int32_t* __restrict__ lengths,
                                                             int n_segments, int chunk_rows, int lane) {
  LaneSegments<kSegs> x;
  const int s0 = first_of_lane<kSegs>(n_segments, lane);
#pragma unroll
  for (int j = 0; j < kSegs; ++j) x.lo[j] = offsets[s0 + j];
  if (lengths != nullptr) {
#pragma unroll
    for (int j = 0; j < kSegs; ++j) x.hi[j] = lengths[s0 + j];
#pragma unroll
    for (int j = 0; j < kSegs; ++j) x.hi[j] += x.lo[j];
  } else {
#pragma unroll
    for (int j = 0; j + 1 < kSegs; ++j) x.hi[j] = x.lo[j + 1];
    x.hi[kSegs - 1] = offsets[s0 + kSegs];
  }
  x.all = 0;
#pragma unroll
  for (int j = 0; j < kSegs; ++j) {
    const uint32_t rows = (uint32_t)max(x.hi[j] - x.lo[j], 0);
    x.n[j] = s0 + j >= kSegs * lane ? (int)((rows + (uint32_t)chunk_rows - 1u) / (uint32_t)chunk_rows) : 0;
    x.all += x.n[j];
  }
  x.upto = prefix_sum(x.all);
  return x;
}

// Of the segments of lane `at`, the one that `mine(its number, its first chunk, its chunks)` is true for.
template <int kSegs, typename Mine>
__device__ __forceinline__ AlignedChunk pick_segment(const LaneSegments<kSegs>& x, int n_segments, int at, Mine mine) {
  AlignedChunk found = {-1, 0, 0, 0, 0};
  const int s0 = first_of_lane<kSegs>(n_segments, at);
  int first = __builtin_amdgcn_readlane(x.upto, at) - __builtin_amdgcn_readlane(x.all, at);
#pragma unroll
  for (int j = 0; j < kSegs; ++j) {
    const int n = __builtin_amdgcn_readlane(x.n[j], at);
    if (mine(s0 + j, first, n))
      found = {s0 + j, __builtin_amdgcn_readlane(x.lo[j], at), __builtin_amdgcn_readlane(x.hi[j], at), first, n};
    first += n;
  }
  return found;
}

// By all lanes of a wave.
template <int kSegs>
__device__ __forceinline__ AlignedChunk find_aligned_chunk(const int32_t* offsets, const int32_t* lengths, int n_segments,
                                                           int chunk_rows, int chunk, int lane) {
  const LaneSegments<kSegs> x = lane_segments<kSegs>(offsets, lengths, n_segments, chunk_rows, lane);
  const unsigned long long later = __ballot(x.upto > chunk);
  if (later == 0) return {-1, 0, 0, 0, 0};
  return pick_segment(x, n_segments, __builtin_ctzll(later), [&](int, int first, int n) { return chunk >= first && chunk < first + n; });
}

// Rows of one segment inside a chunk.
struct DecPiece {
  int s;        // -1: none
  int a;        // its first row
  int n_rows;
  int owner;    // the wave that takes it alone, or -1: all share it
  bool whole;   // all rows of the segment
};

// kMasked: every row carries a retention weight m in [0, 1] and the probabilities are
// p_i = e^{s_i} m_i / sum_j e^{s_j} m_j (the multiplicative mask of App. B.2, which is softmax(s + log m));
// the rows are then those of the uncompacted cache.  kAligned: chunks start at the segments.
template <bool kMasked, int kSegs>
__global__ void __launch_bounds__(kDecThreads, 2)
decode_partial_kernel(const uint16_t* __restrict__ q, const uint4* __restrict__ kp,
                      const uint4* __restrict__ vp, const int32_t* __restrict__ offsets,
                      const int32_t* __restrict__ lengths /* rows in use per segment, or null: all of them */,
                      int n_segments, int64_t total_kept, int chunk_rows, int G, float scale, float* __restrict__ out,
                      float* __restrict__ lse, float* __restrict__ ws_acc, float* __restrict__ ws_m,
                      float* __restrict__ ws_l, const float* __restrict__ mask) {
  constexpr bool kAligned = kSegs > 0;
  extern __shared__ __align__(16) unsigned char smem[];

  const int chunk = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  AlignedChunk mine = {};
  if constexpr (kAligned) {
    mine = find_aligned_chunk<kSegs>(offsets, lengths, n_segments, chunk_rows, chunk, lane);
    if (mine.segment < 0) return;   // the whole block
  }
  const int64_t p0 = kAligned ? (int64_t)mine.lo + (int64_t)(chunk - mine.first) * chunk_rows : (int64_t)chunk * chunk_rows;
  const int64_t p1 = min(p0 + (int64_t)chunk_rows, total_kept);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane >> 4;     // load view: row slot.   operand view: K-block kb / accumulator row block rb
  const int c = lane & 15;     // load view: 16-byte piece. operand view: token / head / channel index
  unsigned char* k_lds = smem + wave * kDecWaveLds;
  unsigned char* v_lds = k_lds + kDecTile * kDecKStride;
  DecMerge& mg = *reinterpret_cast<DecMerge*>(smem);
  const float qscale = scale * kLog2e;

  // Flat chunks: the pieces in 64 segments at a time, one per lane, from the segment that contains row p0 on (the last with
  // offsets[s] <= p0).  `shared` and `alone` are the pieces still to do that the four waves share and that one takes.
  int listed = 0, alone_tiles = 0;
  int lane_a = 0, lane_rows = 0;
  unsigned long long shared = 0, alone = 0, whole_ones = 0;
  bool more = false;
  int load[kDecWaves] = {};
  auto list_pieces = [&](int from) __attribute__((always_inline)) {
    listed = from;
    const int s = min(from + lane, n_segments - 1);
    const int lo = offsets[s];
    // rows behind the ones in use (spare rows for later tokens) are never read
    const int hi = lengths != nullptr ? lo + lengths[s] : offsets[s + 1];
    lane_a = (int)max(p0, (int64_t)lo);
    lane_rows = from + lane < n_segments ? (int)(min(p1, (int64_t)hi) - lane_a) : 0;   // none: empty (zeroed by the merge kernel)
    whole_ones = __ballot(lo >= p0 && hi <= p1);
    more = from + 64 < n_segments && __builtin_amdgcn_readlane(lo, 63) < p1;
  };
  auto deal_pieces = [&]() __attribute__((always_inline)) {
    shared = __ballot(lane_rows > alone_tiles * kDecTile);
    alone = __ballot(lane_rows > 0) & ~shared;
  };
  if (!kAligned) {
    list_pieces(wave_upper_segment(offsets, n_segments, p0, lane));
    const int t = lane_rows > 0 ? (lane_rows + kDecTile - 1) / kDecTile : 0;
    int best = 0x7fffffff;
    alone_tiles = 2;
    if (__ballot(t > 2) != 0)   // else all go to single waves
#pragma unroll
    for (int tiles = 2; tiles <= 32; tiles *= 2) {
      // in quarters of a tile: what the waves do alone (the longest of it last) and what they share
      const unsigned long long longest = __ballot(t > tiles / 2 && t <= tiles);
      if (tiles > 2 && longest == 0) continue;
      const int cost_here = t == 0 ? 0 : t <= tiles ? t + kDecAloneCost : (4 * ((t + 3) / 4) + kDecSharedCost) << 12;
      int cost = __builtin_amdgcn_readlane(prefix_sum(cost_here), 63);
      const int by_one = cost & 4095;
      cost = (cost >> 12) + (by_one == 0 ? 0 : max(by_one + 2 * tiles, 4 * tiles));
      if (cost < best) { best = cost; alone_tiles = tiles; }
    }
    deal_pieces();
  }
  // The next piece that this wave has a part in.
  auto next_piece = [&]() __attribute__((always_inline)) {
    for (;;) {
      if (shared != 0) {
        const int i = __builtin_ctzll(shared);
        shared &= shared - 1;
        return DecPiece{listed + i, __builtin_amdgcn_readlane(lane_a, i), __builtin_amdgcn_readlane(lane_rows, i), -1,
                        (whole_ones >> i & 1) != 0};
      }
      while (alone != 0) {
        const int i = __builtin_ctzll(alone);
        alone &= alone - 1;
        const int n_rows = __builtin_amdgcn_readlane(lane_rows, i);
        int who = 0, least = load[0];
#pragma unroll
        for (int w = 1; w < kDecWaves; ++w)
          if (load[w] < least) { least = load[w]; who = w; }
#pragma unroll
        for (int w = 0; w < kDecWaves; ++w) load[w] += w == who ? (n_rows + kDecTile - 1) / kDecTile + kDecAloneCost : 0;
        if (who == wave) return DecPiece{listed + i, __builtin_amdgcn_readlane(lane_a, i), n_rows, who, (whole_ones >> i & 1) != 0};
      }
      if (!more) return DecPiece{-1, 0, 0, -1, false};
      list_pieces(listed + 64);
      asm volatile("" : "+v"(lane_a), "+v"(lane_rows));   // waited for here, not in every turn of the loop
      deal_pieces();
    }
  };
  // B operand of the first product: Q^T, lane (head c, K-block r) holds q[head c][32 ks + 8 r .. +7].  Columns past the
  // group repeat its last head and are not used; zeroed behind a branch they made every load wait for the one before.
  bf16x8_t qfrag[4];
  uint4 kk[8], vv[8];
  auto load_q = [&](const DecPiece& piece) __attribute__((always_inline)) {
    const uint4* row = reinterpret_cast<const uint4*>(q + ((size_t)piece.s * G + min(c, G - 1)) * kHeadDim);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) qfrag[ks] = __builtin_bit_cast(bf16x8_t, row[ks * 4 + r]);
  };
  auto load_tile = [&](const DecPiece& piece, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      int row = t * kDecTile + 4 * j + r;
      row = row < piece.n_rows ? row : piece.n_rows - 1;   // rows past the piece re-read its last row; zeroed when staged
      kk[j] = load_stream16(kp + ((int64_t)piece.a + row) * kChunksPerRow + c);
      vv[j] = load_stream16(vp + ((int64_t)piece.a + row) * kChunksPerRow + c);
      asm volatile("" ::: "memory");   // in this order, so that the staging can wait for them one by one
    }
  };

  // this wave's first tile (of a piece without one for it: rows that it does not use)
  auto load_first = [&](const DecPiece& piece) __attribute__((always_inline)) {
    load_tile(piece, piece.owner < 0 ? wave : 0);
  };

  DecPiece next;
  if (kAligned) {
    const int n_rows = (int)(min(p1, (int64_t)mine.hi) - p0);
    const bool small = n_rows <= kDecSmallPiece;
    if (n_rows <= 0 || (small && wave != 0)) return;
    next = DecPiece{mine.segment, (int)p0, n_rows, small ? 0 : -1, mine.n == 1};
  } else {
    next = next_piece();
    if (next.s < 0) return;
  }
  load_q(next);
  load_first(next);

#pragma unroll 1
  for (;;) {
    const DecPiece now = next;
    const int s = now.s, a = now.a, n_rows = now.n_rows;
    const int n_tiles = (n_rows + kDecTile - 1) / kDecTile;
    const bool small = now.owner >= 0, whole = now.whole;
    const int t_first = small ? 0 : wave, t_step = small ? 1 : kDecWaves;
    if (!kAligned) {
      next = next_piece();   // while the rows are on their way (behind the wait: 288 heads of 60 rows 12.4 us, 12.0 so)
      // waited for here: inside the loop the wait would reach the rows to come as well
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(qfrag[ks]));
      if (next.s >= 0 && t_first >= n_tiles) load_first(next);
    }
    float m_run = -INFINITY;   // running max of head c (log2 domain), identical in the four lanes of a head
    float l_run = 0.f;         // this lane's share of the denominator
    f32x4_t acc_o[8];          // O[head 4r+e][channel 16 ct + c]
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc_o[ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};

#pragma unroll 1
    for (int t = t_first; t < n_tiles; t += t_step) {
      // The weights of the tile's rows: asked for ahead of the rows to come, which would have to arrive first (loads are waited for
      // in order).  After them: 200 heads of 2000 rows 46.9 us, 41.0 so; 512 of 500 36.5 and 32.6; 288 of 60 16.6 and 15.3.
      float weight[8];
      if constexpr (kMasked) {
#pragma unroll
        for (int i = 0; i < 8; ++i) weight[i] = mask[(int64_t)a + min(t * kDecTile + (i >> 2) * 16 + 4 * r + (i & 3), n_rows - 1)];
        asm volatile("" ::: "memory");
      }
      // stage 32 rows: row 4j + r, piece c
      if ((t + 1) * kDecTile <= n_rows) {   // wave-uniform: a full tile
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          *reinterpret_cast<uint4*>(k_lds + (4 * j + r) * kDecKStride + c * 16) = kk[j];
          *reinterpret_cast<uint4*>(v_lds + (4 * j + r) * kDecVStride + c * 16) = vv[j];
        }
      } else {   // last tile of the piece: zero the rows past its end
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t keep = t * kDecTile + 4 * j + r < n_rows ? 0xffffffffu : 0u;
          *reinterpret_cast<uint4*>(k_lds + (4 * j + r) * kDecKStride + c * 16) =
              make_uint4(kk[j].x & keep, kk[j].y & keep, kk[j].z & keep, kk[j].w & keep);
          *reinterpret_cast<uint4*>(v_lds + (4 * j + r) * kDecVStride + c * 16) =
              make_uint4(vv[j].x & keep, vv[j].y & keep, vv[j].z & keep, vv[j].w & keep);
        }
      }
      if (t + t_step < n_tiles) load_tile(now, t + t_step);   // prefetch
      else if (!kAligned && next.s >= 0) load_first(next);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

      // S^T for the two 16-token halves: lane (rb = r, head c) gets tokens 16 tt + 4 r + e
      f32x4_t sacc[2];
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        sacc[tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const uint4 kx = *reinterpret_cast<const uint4*>(k_lds + (tt * 16 + c) * kDecKStride + ks * 64 + r * 16);
          sacc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kx), qfrag[ks], sacc[tt],
                                                             0, 0, 0);
        }
      }
      // online softmax for head c over the 8 tokens of this lane and the other three lanes of the head
      float sv[8];
      float mx = m_run;
      const int tok0 = t * kDecTile;
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int tok = tok0 + tt * 16 + 4 * r + e;
          const bool ok = tok < n_rows;
          float sc = sacc[tt][e] * qscale;
          if constexpr (kMasked) sc += __log2f(weight[tt * 4 + e]);   // log2(0) = -inf drops the row
          sv[tt * 4 + e] = ok ? sc : -INFINITY;
          mx = fmaxf(mx, sv[tt * 4 + e]);
        }
      mx = max_over_row_blocks(mx);
      const float ref = mx == -INFINITY ? 0.f : mx;
      const float alpha = fast_exp2(m_run - ref);     // exp2(-inf) = 0 on the first tile
      m_run = mx;
      float psum = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) { sv[i] = fast_exp2(sv[i] - ref); psum += sv[i]; }
      l_run = l_run * alpha + psum;
      // A operand of the second product: P[head c][K-slots 8 r .. 8 r + 7] = this lane's own 8 values
      bf16x8_t pfrag, plow;   // rounded, and what the rounding left
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        pfrag[i] = (__bf16)sv[i];
        plow[i] = (__bf16)(sv[i] - (float)pfrag[i]);
      }
      // rescale the output rows (heads 4r+e) when any running max moved
      if (__ballot(alpha != 1.f) != 0ull) {
        float al[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) al[e] = __shfl(alpha, 4 * r + e, 64);
#pragma unroll
        for (int ct = 0; ct < 8; ++ct)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc_o[ct][e] *= al[e];
      }
      // O += P V: B operand lane (channel c of tile ct, K-block r) holds V[tokens 4r..4r+3 and 16+4r..16+4r+3][ch]
      s16x8_t vb[8];
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) {
        const unsigned char* base = v_lds + (4 * r + (c >> 2)) * kDecVStride + ct * 32 + (c & 3) * 8;
        const s16x4_t v0 = lds_read_tr16(base);
        const s16x4_t v1 = lds_read_tr16(base + 16 * kDecVStride);
        vb[ct] = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
        acc_o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pfrag, __builtin_bit_cast(bf16x8_t, vb[ct]), acc_o[ct], 0, 0, 0);
      }
      // An infinite value would meet a zero or the other sign in what the rounding left and become NaN: not multiplied then.
      float top = 0.f;
#pragma unroll
      for (int ct = 0; ct < 8; ++ct)
#pragma unroll
        for (int e = 0; e < 4; e += 2) top = fmaxf(fmaxf(top, fabsf(acc_o[ct][e])), fabsf(acc_o[ct][e + 1]));
      if (__ballot(top == INFINITY) == 0) {
#pragma unroll
        for (int ct = 0; ct < 8; ++ct)
          acc_o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plow, __builtin_bit_cast(bf16x8_t, vb[ct]), acc_o[ct], 0, 0, 0);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (!kAligned && next.s >= 0) load_q(next);
    l_run = sum_over_row_blocks(l_run);
    const size_t slot = kAligned ? (size_t)chunk : (size_t)s + (size_t)chunk;
    if (small) {
      // ---- one wave had the whole piece: it writes the result (or the partial) straight from its registers;
      // head h's maximum and denominator sit in lane h ----
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int h = 4 * r + e;
        const float mxh = __shfl(m_run, h, 64);
        const float den = __shfl(l_run, h, 64);
        if (h < G) {
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) {
            const float num = acc_o[ct][e];
            if (whole) out[((size_t)s * G + h) * kHeadDim + ct * 16 + c] = den > 0.f ? num / den : 0.f;
            else ws_acc[(slot * G + h) * kHeadDim + ct * 16 + c] = num;
          }
          if (c == 0) {
            if (whole) {
              if (lse != nullptr) lse[(size_t)s * G + h] = den > 0.f ? mxh * kLn2 + __logf(den) : -INFINITY;
            } else {
              ws_m[slot * G + h] = mxh;
              ws_l[slot * G + h] = den;
            }
          }
        }
      }
      if (kAligned || next.s < 0) return;
      continue;
    }
    // ---- combine the four waves through LDS (the staging tiles are free now) ----
    __syncthreads();   // every wave is done with its staging tile
    if (r == 0 && c < G) { mg.m[wave][c] = m_run; mg.l[wave][c] = l_run; }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int h = 4 * r + e;
      if (h < G) {
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) mg.acc[wave][h][ct * 16 + c] = acc_o[ct][e];
      }
    }
    __syncthreads();
    for (int o = tid; o < G * kHeadDim; o += kDecThreads) {
      const int h = o / kHeadDim, ch = o - h * kHeadDim;
      float mxw = -INFINITY;
#pragma unroll
      for (int w = 0; w < kDecWaves; ++w) mxw = fmaxf(mxw, mg.m[w][h]);
      const float refw = mxw == -INFINITY ? 0.f : mxw;   // -inf: no row of this piece carries weight
      float num = 0.f, den = 0.f;
#pragma unroll
      for (int w = 0; w < kDecWaves; ++w) {
        const float wgt = fast_exp2(mg.m[w][h] - refw);   // 0 for a wave that saw no row (m = -inf)
        num = fmaf(mg.acc[w][h][ch], wgt, num);
        den = fmaf(mg.l[w][h], wgt, den);
      }
      if (whole) {
        // den = 0 only when every row of the segment carries weight 0: zero output, lse = -inf
        out[((size_t)s * G + h) * kHeadDim + ch] = den > 0.f ? num / den : 0.f;
        if (ch == 0 && lse != nullptr) lse[(size_t)s * G + h] = den > 0.f ? mxw * kLn2 + __logf(den) : -INFINITY;
      } else {
        ws_acc[(slot * G + h) * kHeadDim + ch] = num;
        if (ch == 0) { ws_m[slot * G + h] = mxw; ws_l[slot * G + h] = den; }
      }
    }
    if (kAligned) return;
    __syncthreads();   // the merge scratch becomes staging tiles again
    if (next.s < 0) return;
  }
}

// Merge of the per-piece partials of one segment; also zeroes the output of empty segments.
// Each thread owns one output element (query head h, channel ch); a segment takes
// ceil(G * 128 / 256) blocks.  The kernel is a short chain of dependent memory latencies, so
// the partials of up to eight pieces are loaded together and folded in with a running maximum:
// the chain is the offsets load plus one round per eight pieces.
// kParts > 1, for segments of many pieces: a block of kParts times 128 threads for every query head, the pieces of an
// element shared out among kParts threads, whose sums meet in LDS: one round per 8 kParts pieces.  A segment of one round
// is left to the first 128 threads alone.
constexpr int decode_merge_threads(int parts) { return parts == 1 ? kDecThreads : parts * kHeadDim; }
template <int kSegs, int kParts>
__global__ void __launch_bounds__(decode_merge_threads(kParts))
decode_merge_kernel(const int32_t* __restrict__ offsets, const int32_t* __restrict__ lengths, int n_segments, int G,
                    int blocks_per_segment, int chunk_rows,
                    const float* __restrict__ ws_acc, const float* __restrict__ ws_m,
                    const float* __restrict__ ws_l, float* __restrict__ out, float* __restrict__ lse) {
  constexpr bool kAligned = kSegs > 0;
  const int s = blockIdx.x / blocks_per_segment;
  const int part = kParts == 1 ? 0 : threadIdx.x / kHeadDim;
  const int o = kParts == 1 ? (blockIdx.x - s * blocks_per_segment) * kDecThreads + threadIdx.x
                            : (blockIdx.x - s * blocks_per_segment) * kHeadDim + threadIdx.x % kHeadDim;
  AlignedChunk seg = {};
  if constexpr (kAligned)   // by all lanes, before any leaves
    seg = pick_segment(lane_segments<kSegs>(offsets, lengths, n_segments, chunk_rows, threadIdx.x & 63), n_segments, s / kSegs,
                       [&](int at, int, int) { return at == s; });
  if (o >= G * kHeadDim) return;
  const int h = o / kHeadDim, ch = o - h * kHeadDim;
  const int64_t a = kAligned ? seg.lo : offsets[s];
  const int64_t b = kAligned ? seg.hi : lengths != nullptr ? a + lengths[s] : (int64_t)offsets[s + 1];
  const size_t row = (size_t)s * G + h;
  if (b <= a) {   // empty segment: zero output, lse = -inf
    out[row * kHeadDim + ch] = 0.f;
    if (ch == 0 && lse != nullptr) lse[row] = -INFINITY;
    return;
  }
  // the segment's chunks; their slots are counted by chunk, and with flat chunks by segment too
  const int c_first = kAligned ? seg.first : (int)(a / chunk_rows);
  const int c_last = kAligned ? seg.first + seg.n - 1 : (int)((b - 1) / chunk_rows);
  const size_t slot0 = kAligned ? 0 : (size_t)s;
  if (c_first == c_last) return;   // a whole segment inside one chunk was finished by the first kernel
  constexpr int kU = 8;
  const bool shared_out = kParts > 1 && c_last - c_first >= kU;   // the same in the whole block
  if (part > 0 && !shared_out) return;
  float mx = -INFINITY, num = 0.f, den = 0.f;
  for (int c0 = c_first + part * kU; c0 <= c_last; c0 += kParts * kU) {
    float mv[kU], lv[kU], av[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int cc = min(c0 + u, c_last);
      const size_t sl = slot0 + cc;
      mv[u] = ws_m[sl * G + h];
      lv[u] = ws_l[sl * G + h];
      av[u] = ws_acc[(sl * G + h) * kHeadDim + ch];
    }
    float mnew = mx;
#pragma unroll
    for (int u = 0; u < kU; ++u) mnew = fmaxf(mnew, mv[u]);   // -inf only if every row so far carries weight 0
    const float ref = mnew == -INFINITY ? 0.f : mnew;
    const float keep = fast_exp2(mx - ref);                    // 0 in the first round
    num *= keep;
    den *= keep;
    mx = mnew;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const bool mine = c0 + u <= c_last;   // the last piece is read again past it, and may be infinite
      const float wgt = mine ? fast_exp2(mv[u] - ref) : 0.f;
      num = fmaf(mine ? av[u] : 0.f, wgt, num);
      den = fmaf(lv[u], wgt, den);
    }
  }
  if (shared_out) {
    __shared__ float num_lds[kParts][kHeadDim], mx_lds[kParts], den_lds[kParts];
    num_lds[part][ch] = num;
    if (ch == 0) { mx_lds[part] = mx; den_lds[part] = den; }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int p = 1; p < kParts; ++p) mx = fmaxf(mx, mx_lds[p]);
    const float ref = mx == -INFINITY ? 0.f : mx;
    num = den = 0.f;
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
      const float wgt = fast_exp2(mx_lds[p] - ref);   // 0 for a part without pieces
      num = fmaf(num_lds[p][ch], wgt, num);
      den = fmaf(den_lds[p], wgt, den);
    }
  }
  out[row * kHeadDim + ch] = den > 0.f ? num / den : 0.f;
  if (ch == 0 && lse != nullptr) lse[row] = den > 0.f ? mx * kLn2 + __logf(den) : -INFINITY;
}

// Rows per block: a multiple of the wave tile, sized for kDecTargetBlocks blocks.
int decode_chunk_rows(int64_t total_kept) {
  int64_t c = (total_kept + kDecTargetBlocks - 1) / kDecTargetBlocks;
  c = (c + kDecTile - 1) / kDecTile * kDecTile;
  if (c < kDecMinChunk) c = kDecMinChunk;
  return (int)c;
}

// Rows per chunk where chunks start at the segments: every segment may end in a short one, and the grid with all of those
// is still about one round of resident blocks.  Never less than decode_chunk_rows, whose slots hold these chunks too.
static int decode_aligned_chunk_rows(int n_segments, int64_t total_kept) {
  if (n_segments > kDecSegsPerWave) {
    // Half of a chunk a segment is what its end costs on average.  For 256 segments a share of 55, 67 or 80 % of a chunk each
    // was equal within 4 % but for a second round here and there.
    const int64_t c = total_kept / (kDecTargetBlocks - n_segments * 5 / 8) + 1;
    return max(decode_chunk_rows(total_kept), (int)((c + kDecTile - 1) / kDecTile * kDecTile));
  }
  const int64_t c = (total_kept + kDecTargetBlocks - n_segments - 1) / (kDecTargetBlocks - n_segments);
  return (int)(c <= kDecMinChunk ? kDecMinChunk : (c + kDecTile - 1) / kDecTile * kDecTile);
}

static size_t decode_slots(int n_segments, int64_t total_kept) {
  const int chunk = decode_chunk_rows(total_kept);
  return (size_t)n_segments + (size_t)((total_kept + chunk - 1) / chunk);
}

size_t decode_workspace_bytes(int n_segments, int64_t total_kept, int G) {
  const size_t per_head = (size_t)(kHeadDim + 2) * sizeof(float);
  const size_t bytes = decode_slots(n_segments, total_kept) * (size_t)G * per_head;
  return (bytes + 255) & ~(size_t)255;
}

// Split-K partials of the decode call that allocates nothing and takes no workspace argument: a
// fixed array in the library's device image.  Every GPU the library runs on holds its own copy at
// its own address until the process ends.  The name below is only a host-side handle for the
// symbol; the device address is looked up once per device and everything on the host side uses
// that address.
constexpr size_t kDecStaticBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kDecStaticBytes];
constexpr int kDecMaxDevices = 64;
static void* g_scratch_ptr[kDecMaxDevices] = {};

size_t decode_static_scratch_bytes() { return kDecStaticBytes; }

// Device address of the static scratch array on `device`, or null if decode_prepare has not run there.
void* decode_static_scratch(int device) {
  return device >= 0 && device < kDecMaxDevices ? g_scratch_ptr[device] : nullptr;
}

// Once per device, with that device current (lkv_create calls it right after selecting the device).
// The four staging tiles exceed the default 64 KB of LDS per workgroup.
hipError_t decode_prepare(int device) {
  const void* kernels[] = {
      reinterpret_cast<const void*>(decode_partial_kernel<false, 0>), reinterpret_cast<const void*>(decode_partial_kernel<false, 1>),
      reinterpret_cast<const void*>(decode_partial_kernel<false, 4>), reinterpret_cast<const void*>(decode_partial_kernel<true, 0>),
      reinterpret_cast<const void*>(decode_partial_kernel<true, 1>),  reinterpret_cast<const void*>(decode_partial_kernel<true, 4>)};
  hipError_t e = hipSuccess;
  for (const void* k : kernels) {
    e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kDecWaves * kDecWaveLds);
    if (e != hipSuccess) return e;
  }
  if (device < 0 || device >= kDecMaxDevices) return hipErrorInvalidDevice;
  if (g_scratch_ptr[device] == nullptr) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (ptr == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
  }
  return hipSuccess;
}

// offsets[s] = s * len for s = 0..n_segments: the uncompacted cache of one sequence seen as a packed cache
__global__ void uniform_offsets_kernel(int n_segments, int len, int32_t* __restrict__ offsets) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s <= n_segments) offsets[s] = s * len;
}

void launch_uniform_offsets(int n_segments, int len, int32_t* offsets, hipStream_t stream) {
  hipLaunchKernelGGL(uniform_offsets_kernel, dim3((n_segments + 256) / 256), dim3(256), 0, stream, n_segments, len,
                     offsets);
}

hipError_t launch_decode(int G, const void* q, const void* kp, const void* vp, const int32_t* offsets,
                         const int32_t* lengths, int n_segments, int64_t total_kept, float scale, float* out, float* lse, float* ws,
                         hipStream_t stream, const float* mask) {
  if (G < 1 || G > kDecMaxGroup) return hipErrorInvalidValue;
  const size_t slots = decode_slots(n_segments, total_kept);
  float* ws_acc = ws;
  float* ws_m = ws + slots * G * kHeadDim;
  float* ws_l = ws_m + slots * G;
  auto launch = [&](auto masked_tag, auto segs_tag) {
    constexpr bool kMasked = decltype(masked_tag)::value;
    constexpr int kSegs = decltype(segs_tag)::value;
    constexpr bool kAligned = kSegs > 0;
    const int chunk_rows = kAligned ? decode_aligned_chunk_rows(n_segments, total_kept) : decode_chunk_rows(total_kept);
    const int chunks = kAligned ? (int)(total_kept / chunk_rows) + n_segments   // each segment may end in a short one
                                : (int)((total_kept + chunk_rows - 1) / chunk_rows);
    if (total_kept > 0)
      hipLaunchKernelGGL((decode_partial_kernel<kMasked, kSegs>), dim3(chunks), dim3(kDecThreads), kDecWaves * kDecWaveLds,
                         stream, reinterpret_cast<const uint16_t*>(q), reinterpret_cast<const uint4*>(kp),
                         reinterpret_cast<const uint4*>(vp), offsets, lengths, n_segments, total_kept, chunk_rows, G, scale,
                         out, lse, ws_acc, ws_m, ws_l, mask);
    auto merge = [&](auto parts_tag) {
      constexpr int kParts = decltype(parts_tag)::value;
      const int blocks_per_segment = kParts == 1 ? (G * kHeadDim + kDecThreads - 1) / kDecThreads : G;
      hipLaunchKernelGGL((decode_merge_kernel<kSegs, kParts>), dim3(n_segments * blocks_per_segment),
                         dim3(decode_merge_threads(kParts)), 0, stream, offsets, lengths, n_segments, G, blocks_per_segment,
                         chunk_rows, ws_acc, ws_m, ws_l, out, lse);
    };
    if constexpr (kAligned) {
      // From three chunks a segment on, eight threads to an element where the launch has up to 256 blocks of
      // them and four where it has more (each block then starts half the waves).  Flat chunks
      // keep one thread per element.  In a captured graph, whole call, one thread : eight : four (us):
      // 8 heads of 4 queries, 24 chunks a call 9.0 : 9.2, 100 11.1 : 9.5, 375 18.3 : 10.8, 491 of 320 rows 28.1 : 18.8; 64 heads of 16
      // queries, 5 chunks each 11.0 : 13.4 : 11.7, 10 each 14.5 : 16.8 : 14.9, one of them with nearly all of 300 and 600 29.8 : 15.9 :
      // 17.0 and 39.2 : 20.7 : 22.3.
      const int64_t heads = (int64_t)n_segments * G;
      if (total_kept / chunk_rows >= 3 * (int64_t)n_segments) {
        if (heads <= 256) return merge(std::integral_constant<int, 8>{});
        return merge(std::integral_constant<int, 4>{});
      }
    }
    merge(std::integral_constant<int, 1>{});
  };
  auto launch_segs = [&](auto segs_tag) {
    if (mask != nullptr) launch(std::true_type{}, segs_tag); else launch(std::false_type{}, segs_tag);
  };
  if (n_segments <= kDecSegsPerWave) launch_segs(std::integral_constant<int, 1>{});
  else if (n_segments <= 4 * kDecSegsPerWave && (n_segments <= 2 * kDecSegsPerWave || decode_chunk_rows(total_kept) <= kDecAlignedChunk))
    launch_segs(std::integral_constant<int, 4>{});
  else launch_segs(std::integral_constant<int, 0>{});
  return hipGetLastError();
}

}  // namespace lkv
