// Head-wise budgeted hard top-k: m = TopK(u, b) per KV head (Sec. 3.4 of the
// paper, inference), with the budget b an input (LKV-H, Sec. 3.3).
//
// One workgroup of 1024 threads per segment (sequence, layer, head).
//   1. Scores are compared as order-preserving uint32 keys (NaN -> -inf first).
//   2. A histogram over 2048 bins that do not decrease with the key, scanned from the top, gives the bin of the b-th
//      largest key: linear bins over the bulk of the scores, or the first 11 bits of the keys when the scoring launch has
//      counted those or the linear bins do not spread a sample of the scores (heavy tails, ties).  Tokens above the bin are kept, tokens below it are not, tokens inside it are listed.
//   3. The listed tokens are narrowed by a radix descent over their keys (11 + 11 + 10 bits) until no more than 256 are
//      left in question, and those are ranked against one another by (key, token): the lower-index tie rule.  Where more
//      than that share one key (ties), the descent ends at that threshold key and the first `need` of its copies are kept.
//   4. Emission in ascending token order from bitmaps of the kept tokens (1024 tokens per wave step): every lane expands
//      its 16 bits into the wave's LDS staging buffer at the position given by a prefix count, then the wave copies
//      the staged indices out with fully coalesced stores.  No atomic decides a position, so the result is unique and
//      reproducible bit for bit.
// Where the scores live depends on the head length T:
//   * T <= 34816: in the registers of the workgroup (select_held_kernel), read once.
//   * longer heads (select_kernel) read them from memory for the first histogram and once more to settle every token outside
//     the undecided bin and to list those inside it (up to 16384 indices, in the LDS the emission stages through later); the rest
//     happens on the listed tokens, in registers.  If more tokens than that share the bin, all three levels and the
//     classification re-read the scores instead.
//   * T <= 327680 is the limit for the bitmaps; longer heads re-read the scores in order during
//     emission, 64 tokens a step.
// A layer's eviction (few heads) chooses in every block that copies rows and copies in the same launch: select_compact_kernel,
// select_compact_long_kernel.
// All global reads are issued many at a time per thread before any is used: the kernels are
// latency-bound, not bandwidth-bound, so what counts is how few dependent round trips each pass
// makes.  A launch can also rank ragged pieces of one flat score array (the re-eviction of a
// packed cache) instead of the heads of a [L, H, T] tensor.
#include <type_traits>

#include "lkv_common.h"
#include "lkv_shares.h"

namespace lkv {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelBins = 2048;
constexpr int kSelRegionBytes = 144 * 1024;                 // LDS after the histogram: bitmaps, then the staging buffer
constexpr int kSelMaxHeld = 34;                             // scores per thread held in registers
constexpr int kSelMaxHeldT = kSelMaxHeld * kSelThreads;     // 34816: longer heads re-read their scores
constexpr int kSelRankMax = 256;                            // tokens left undecided from which ranking them one by one pays
constexpr int kSelCopies = 8;                               // copies of a histogram while it is counted
constexpr float kSelBinSpan = 5.f;                          // linear bins cover the mean of the scores +- this many deviations
constexpr int kSelStageWords = 1024;                        // staged indices per wave and step (one per token of the step)
constexpr int kSelStageBytes = kSelWaves * kSelStageWords * 4;   // 64 KB
constexpr int kSelCandCap = kSelStageBytes / 4;             // candidate tokens of a long head (they overlay the staging buffer)
constexpr int kSelMaxBitmapT = (kSelRegionBytes - kSelStageBytes) / 8 * 32;   // 327680 tokens: two bitmaps + staging
static_assert(kSelMaxHeld * kSelWaves <= kSelThreads, "one mask of a round per thread");
static_assert(kSelBins * kSelCopies * 4 <= kSelStageBytes, "the copies lie where the emission stages later");
static_assert(4 * kSelRankMax <= kSelThreads, "four threads rank a token");
static_assert(2 * kSelRankMax <= kSelBins, "the tokens to rank are listed where the histogram was");
constexpr int kSelBatch = 8;                                // loads in flight per thread
constexpr int kSelInlineOffsets = 640;                      // offsets that fit the kernel arguments next to the launch table
constexpr int kSelSplitMaxHeads = 64;                       // launches with at most this many (long) heads split each head's pass
constexpr int kSelSplitTargetBlocks = 256;                  // over about this many workgroups in all,
constexpr int kFuseMaxHeads = 64;                           // one lane each
constexpr int kFuseLongHeads = 16;                          // heads too long for the registers, in one launch at most
constexpr int kSelSplitMax = 32;                            // at most this many per head

struct InlineOffsets {
  int32_t v[kSelInlineOffsets];
};

struct SelShared {
  alignas(16) uint32_t bins[64 + kSelBins];   // bins -1 to -64 take what lies past the end of a head
  uint32_t wave_tot[kSelWaves];
  uint32_t wave_gt[kSelWaves];
  uint32_t wave_eq[kSelWaves];
  float stat[3][kSelWaves];
  uint32_t found_bin;
  uint32_t found_above;
  uint32_t found_count;
  uint32_t cand_count;
  uint32_t first_key;
  __device__ __forceinline__ uint32_t* hist() { return bins + 64; }
};

// Inclusive prefix sum over the 64 lanes of a wave: four shifts within the rows of 16 lanes, then the last lane of a row
// joins the rows after it.  On the vector ALU; the same through the LDS crossbar waits for six round trips.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp_add(uint32_t x) {
  return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, kRows, 0xf, true);
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
  x = dpp_add<0x111, 0xf>(x);   // row_shr:1, 2, 4, 8 (zeros move in)
  x = dpp_add<0x112, 0xf>(x);
  x = dpp_add<0x114, 0xf>(x);
  x = dpp_add<0x118, 0xf>(x);
  x = dpp_add<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
}

// The value of the last lane (a scalar).
__device__ __forceinline__ uint32_t last_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }

// Sum of x over the 64 lanes of a wave, in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) { return last_lane(wave_inclusive_scan(x)); }

// Sum of the per-wave totals of the waves ahead of `wave`: one LDS read per lane and a wave
// reduction instead of a chain of dependent reads.
__device__ __forceinline__ uint32_t waves_before(const uint32_t* totals, int wave, int lane) {
  return wave_sum(lane < wave ? totals[lane] : 0u);
}

// Calls f(score, token) for every token of the head, in no particular order, reading the fp32
// scores from global memory with kSelBatch loads in flight per thread (16-byte loads when the
// head is 16-byte aligned and its length a multiple of four).
template <typename F>
__device__ __forceinline__ void for_each_global_score(const float* __restrict__ u, int T, F f) {
  const int tid = threadIdx.x;
  if ((T & 3) == 0 && (reinterpret_cast<uintptr_t>(u) & 15u) == 0) {
    const float4* u4 = reinterpret_cast<const float4*>(u);
    const int n4 = T >> 2;
    for (int base = tid; base < n4; base += kSelThreads * kSelBatch) {
      float4 v[kSelBatch];
#pragma unroll
      for (int k = 0; k < kSelBatch; ++k) {
        const int i = base + k * kSelThreads;
        v[k] = u4[i < n4 ? i : base];
      }
#pragma unroll
      for (int k = 0; k < kSelBatch; ++k) {
        const int i = base + k * kSelThreads;
        if (i < n4) {
          f(v[k].x, 4 * i);
          f(v[k].y, 4 * i + 1);
          f(v[k].z, 4 * i + 2);
          f(v[k].w, 4 * i + 3);
        }
      }
    }
  } else {
    for (int base = tid; base < T; base += kSelThreads * kSelBatch) {
      float v[kSelBatch];
#pragma unroll
      for (int k = 0; k < kSelBatch; ++k) {
        const int i = base + k * kSelThreads;
        v[k] = u[i < T ? i : base];
      }
#pragma unroll
      for (int k = 0; k < kSelBatch; ++k) {
        const int i = base + k * kSelThreads;
        if (i < T) f(v[k], i);
      }
    }
  }
}

template <typename F>
__device__ __forceinline__ void for_each_global_key(const float* __restrict__ u, int T, F f) {
  for_each_global_score(u, T, [&](float s, int i) { f(order_key(s), i); });
}

// Digits of the keys are counted in kSelCopies copies of a histogram, side by side, lane l in copy l mod kSelCopies:
// atomics on one address run one after the other (about two cycles a lane), and ties or the leading digits of scores
// of one magnitude put most of a wave into one bin.  (8 heads of 32768 equal scores: 124 us with one copy, 29 us with
// eight.  Linear bins that spread the scores need one: clearing and adding up the copies costs 1 us.)
__device__ __forceinline__ void count_bin(uint32_t* copies, uint32_t bin) {
  atomicAdd(&copies[bin * kSelCopies + (threadIdx.x & (kSelCopies - 1))], 1u);
}
__device__ __forceinline__ void clear_copies(uint32_t* copies) {
  for (int i = threadIdx.x; i < kSelBins * kSelCopies / 4; i += kSelThreads)
    reinterpret_cast<uint4*>(copies)[i] = make_uint4(0, 0, 0, 0);
}
__device__ __forceinline__ uint32_t sum_copies(const uint32_t* copies, int bin) {
  const uint4* c = reinterpret_cast<const uint4*>(copies + (size_t)bin * kSelCopies);
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < kSelCopies / 4; ++j) sum += c[j].x + c[j].y + c[j].z + c[j].w;
  return sum;
}

// Whether a wave's lanes crowd into few bins: 8 of them share one (the same answer in every lane).
__device__ __forceinline__ bool lanes_crowd(int bin) {
  return __popcll(__ballot(bin == __builtin_amdgcn_readfirstlane(bin))) >= 8 ||
         __popcll(__ballot(bin == __builtin_amdgcn_readlane(bin, 37))) >= 8;
}

// The bin that holds the key of rank `need` from the top: sh.found_bin, found_above (keys in higher bins) and
// found_count, to be read before the next barrier.  count_of(bin) reads the histogram, which must be complete (a barrier
// passed).
template <typename CountOf>
__device__ __forceinline__ void find_bin(SelShared& sh, int nbins, uint32_t need, CountOf count_of) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  // scan the bins from the top: thread t owns bins nbins-1-2t and nbins-2-2t
  uint32_t c0 = 0, c1 = 0;
  const int top = nbins - 1 - 2 * tid;
  if (top >= 0) c0 = count_of(top);
  if (top - 1 >= 0) c1 = count_of(top - 1);
  const uint32_t incl = wave_inclusive_scan(c0 + c1);
  if (lane == 63) sh.wave_tot[wave] = incl;
  __syncthreads();
  const uint32_t before = waves_before(sh.wave_tot, wave, lane);
  const uint32_t excl = before + incl - (c0 + c1);   // keys in bins above this thread's pair
  // exactly one bin satisfies: above < need <= above + count
  if (c0 && excl < need && need <= excl + c0) { sh.found_bin = (uint32_t)top; sh.found_above = excl; sh.found_count = c0; }
  if (c1 && excl + c0 < need && need <= excl + c0 + c1) {
    sh.found_bin = (uint32_t)(top - 1);
    sh.found_above = excl + c0;
    sh.found_count = c1;
  }
  __syncthreads();
}

// One level of the radix descent.  `count(fn)` must call fn(key) for every key of the head.
// On return prefix / prefix_mask / need are advanced by this level's digit.  Returns the number of
// keys in the bin the descent entered (the same value in every thread: it is published by the one
// thread that found the bin and read between two block barriers, so a branch on it is uniform).
__device__ __forceinline__ uint32_t enter_found_bin(SelShared& sh, int level, uint32_t& prefix, uint32_t& prefix_mask,
                                                    uint32_t& need) {
  const int shift = level == 0 ? 21 : (level == 1 ? 10 : 0);
  prefix |= sh.found_bin << shift;
  prefix_mask |= (uint32_t)((level == 2 ? 1024 : 2048) - 1) << shift;
  need -= sh.found_above;
  const uint32_t in_bin = sh.found_count;
  __syncthreads();   // found_* and the histogram are rewritten at the next level
  return in_bin;
}
template <typename Count>
__device__ __forceinline__ uint32_t descend_level(SelShared& sh, uint32_t* copies, int level, uint32_t& prefix,
                                                  uint32_t& prefix_mask, uint32_t& need, Count count) {
  const int shift = level == 0 ? 21 : (level == 1 ? 10 : 0);
  const int nbins = level == 2 ? 1024 : 2048;
  clear_copies(copies);
  __syncthreads();
  const uint32_t pfx = prefix, msk = prefix_mask;
  count([&](uint32_t key) {
    if ((key & msk) == pfx) count_bin(copies, (key >> shift) & (uint32_t)(nbins - 1));
  });
  __syncthreads();
  find_bin(sh, nbins, need, [&](int bin) { return sum_copies(copies, bin); });
  return enter_found_bin(sh, level, prefix, prefix_mask, need);
}
// The first level when sh.hist already holds its counts (and a barrier has passed).
__device__ __forceinline__ uint32_t descend_counted_level(SelShared& sh, uint32_t& prefix, uint32_t& prefix_mask, uint32_t& need) {
  find_bin(sh, kSelBins, need, [&](int bin) { return sh.hist()[bin]; });
  return enter_found_bin(sh, 0, prefix, prefix_mask, need);
}

// Ordered emission from a per-token key source `key_of(i)`: heads too long for the bitmaps, which re-read their scores.
// Nothing is written past the `budget` indices of the segment, also where the counters of another call's scores led to a
// threshold that more tokens pass.
template <typename KeyOf>
__device__ __forceinline__ void emit_from_keys(SelShared& sh, int T, uint32_t thr, uint32_t need, uint32_t budget,
                                               int32_t* __restrict__ out, KeyOf key_of) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  // wave w owns tokens [w*per, (w+1)*per), per a multiple of 64
  const int per = ((T + kSelWaves - 1) / kSelWaves + 63) & ~63;
  const int lo = wave * per;
  const int hi = min(T, lo + per);
  uint32_t n_gt = 0, n_eq = 0;
  for (int base = lo; base < hi; base += 64) {
    const int i = base + lane;
    const bool in = i < hi;
    const uint32_t key = in ? key_of(i) : 0u;
    n_gt += __popcll(__ballot(in && key > thr));
    n_eq += __popcll(__ballot(in && key == thr));
  }
  if (lane == 0) { sh.wave_gt[wave] = n_gt; sh.wave_eq[wave] = n_eq; }
  __syncthreads();
  const uint32_t gt_before = waves_before(sh.wave_gt, wave, lane);
  const uint32_t eq_before = waves_before(sh.wave_eq, wave, lane);
  uint32_t eq_seen = eq_before;                                  // copies of thr before the current 64 tokens
  uint32_t pos = gt_before + min(eq_before, need);               // kept tokens before the current 64 tokens
  for (int base = lo; base < hi; base += 64) {
    const int i = base + lane;
    const bool in = i < hi;
    const uint32_t key = in ? key_of(i) : 0u;
    const bool is_eq = in && key == thr;
    const unsigned long long eq_mask = __ballot(is_eq);
    const unsigned long long below = (1ull << lane) - 1ull;
    const uint32_t eq_rank = eq_seen + __popcll(eq_mask & below);
    const bool keep = in && (key > thr || (is_eq && eq_rank < need));
    const unsigned long long keep_mask = __ballot(keep);
    const uint32_t at = pos + __popcll(keep_mask & below);
    if (keep && at < budget) out[at] = i;
    pos += __popcll(keep_mask);
    eq_seen += __popcll(eq_mask);
  }
}

// The `k` lowest set bits of x (k <= popcount(x)); a fixed five-step search, no lane divergence.
__device__ __forceinline__ uint32_t lowest_set_bits(uint32_t x, uint32_t k) {
  if (k >= (uint32_t)__popc(x)) return x;
  // smallest m in [0, 31] with popcount(x & ((1 << m) - 1)) >= k  (m = 0 when k = 0)
  int lo = -1, hi = 31;   // invariant: the prefix of length hi holds >= k bits, that of length lo (if >= 0) fewer
#pragma unroll
  for (int it = 0; it < 5; ++it) {
    const int mid = (lo + hi + 1) >> 1;
    if ((uint32_t)__popc(x & ((1u << mid) - 1u)) >= k) hi = mid; else lo = mid;
  }
  return x & ((1u << hi) - 1u);
}

__device__ __forceinline__ void wave_lds_sync() {
  // orders this wave's LDS writes and reads of its private staging; no block barrier needed
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Ordered emission from the two LDS bitmaps (bit i of gt: key_i > thr; of eq: key_i == thr).
// Each wave owns a contiguous range of bitmap words and handles 32 words (1024 tokens) per step,
// one 16-bit half word per lane.  Loops whose trip count could differ between lanes are avoided
// (the expansion loop runs a fixed 16 times), and every cross-lane exchange of a step comes
// before the staging traffic.
// kEq = false: there is no map of equal keys, every kept token is in gt_map.  As above, `budget` indices at most.
template <bool kEq>
__device__ __forceinline__ void emit_from_bitmaps(SelShared& sh, int T, uint32_t need, uint32_t budget, int32_t* __restrict__ out,
                                                  const uint32_t* gt_map, const uint32_t* eq_map, uint32_t* stage_all) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  uint32_t* stage = stage_all + wave * kSelStageWords;
  const int n_words = (T + 31) >> 5;
  const int per = ((n_words + kSelWaves - 1) / kSelWaves + 31) & ~31;   // words per wave, a multiple of 32
  const int lo = wave * per;
  const int hi = min(n_words, lo + per);
  uint32_t n_gt = 0, n_eq = 0;
  for (int w = lo + lane; w < hi; w += 64) { n_gt += __popc(gt_map[w]); if (kEq) n_eq += __popc(eq_map[w]); }
  n_gt = wave_sum(n_gt);
  if (kEq) n_eq = wave_sum(n_eq);
  if (lane == 0) { sh.wave_gt[wave] = n_gt; sh.wave_eq[wave] = n_eq; }
  __syncthreads();
  const uint32_t gt_before = waves_before(sh.wave_gt, wave, lane);
  const uint32_t eq_before = kEq ? waves_before(sh.wave_eq, wave, lane) : 0u;
  uint32_t eq_seen = eq_before;
  uint32_t pos = gt_before + min(eq_before, need);
  const int half = lane & 1;
  for (int base = lo; base < hi; base += 32) {
    const int w = base + (lane >> 1);
    const bool in = w < hi;
    const uint32_t gth = in ? (gt_map[w] >> (16 * half)) & 0xffffu : 0u;
    uint32_t bits = gth;
    if (kEq) {
      const uint32_t eqh = in ? (eq_map[w] >> (16 * half)) & 0xffffu : 0u;
      // copies of thr before this lane's half word, and how many of its own copies are still kept
      const uint32_t eq_cnt = __popc(eqh);
      const uint32_t eq_incl = wave_inclusive_scan(eq_cnt);
      const uint32_t eq_rank = eq_seen + eq_incl - eq_cnt;
      const uint32_t take = eq_rank < need ? min(eq_cnt, need - eq_rank) : 0u;
      bits |= lowest_set_bits(eqh, take);
      eq_seen += last_lane(eq_incl);
    }
    const uint32_t cnt = __popc(bits);
    const uint32_t incl = wave_inclusive_scan(cnt);
    const uint32_t total = last_lane(incl);
    uint32_t p = incl - cnt;
    const uint32_t tok0 = ((uint32_t)w << 5) + 16u * half;
#pragma unroll
    for (int it = 0; it < 16; ++it) {
      if (bits) {
        stage[p++] = tok0 + __builtin_ctz(bits);
        bits &= bits - 1;
      }
    }
    wave_lds_sync();
    for (uint32_t j0 = 0; j0 < total; j0 += 64) {   // uniform trip count
      const uint32_t j = j0 + lane;
      if (j < total && pos + j < budget) out[pos + j] = stage[j];
    }
    pos += total;
    wave_lds_sync();   // the staging buffer is rewritten by the next step
  }
}

// Up to kSelInlineOffsets segment offsets travel in the kernel arguments instead of through a
// host-to-device copy (which costs an extra dependent transfer before the kernel can start);
// the blocks then also publish them to the device array that the later calls read.
// Segments that are not heads of a [L, H, T] score tensor but ragged pieces of one flat array
// (re-eviction of a packed cache): segment s has len[s] scores starting at flat[start[s]].
struct SelRagged {
  const float* flat;      // null: the launch table describes the scores
  const int32_t* start;
  const int32_t* len;
};

// Bins that spread the scores of a head evenly: equal steps over mean +- kSelBinSpan deviations, the rest in the end
// bins.  The radix digits of the scores do not: one head's lie within a few powers of two, so most of its tokens
// count into a few dozen of the 2048 digits, and atomics on one address run one after the other.  bin() does
// not decrease with the score (nor with its key; NaN and -inf are in bin 0), which is all that the selection asks of it.
struct LinearBins {
  float lo, scale;
  __device__ __forceinline__ int bin(float u) const {
    return (int)fminf(fmaxf((u - lo) * scale, 0.f), (float)(kSelBins - 1));   // a NaN product goes to 0
  }
};

// From every thread's sums over finite values (count, sum, sum of squares of value - shift); also clears the histogram.
__device__ __forceinline__ LinearBins linear_bins(SelShared& sh, float shift, float n, float sum, float sq) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  n = sum_over_row_blocks(row16_allreduce_sum(n));
  sum = sum_over_row_blocks(row16_allreduce_sum(sum));
  sq = sum_over_row_blocks(row16_allreduce_sum(sq));
  if (lane == 0) { sh.stat[0][wave] = n; sh.stat[1][wave] = sum; sh.stat[2][wave] = sq; }
  for (int i = tid; i < kSelBins; i += kSelThreads) sh.hist()[i] = 0;
  __syncthreads();
  n = fmaxf(row16_allreduce_sum(sh.stat[0][lane & 15]), 1.f);
  const float mean = row16_allreduce_sum(sh.stat[1][lane & 15]) / n;
  const float dev = sqrtf(fmaxf(row16_allreduce_sum(sh.stat[2][lane & 15]) / n - mean * mean, 0.f));
  return {shift + mean - kSelBinSpan * dev, (float)kSelBins / (2.f * kSelBinSpan * dev)};
}

__device__ __forceinline__ bool is_finite_score(float u) { return (__float_as_uint(u) & 0x7f800000u) != 0x7f800000u; }

// The same from a few scores of every lane of a wave, without a barrier.
template <int kN>
__device__ __forceinline__ LinearBins run_bins(const float (&x)[kN], float shift) {
  float n = 0.f, sum = 0.f, sq = 0.f;
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    const bool fin = is_finite_score(x[j]);
    const float d = fin ? x[j] - shift : 0.f;
    n += fin ? 1.f : 0.f;
    sum += d;
    sq = fmaf(d, d, sq);
  }
  n = fmaxf(sum_over_row_blocks(row16_allreduce_sum(n)), 1.f);
  const float mean = sum_over_row_blocks(row16_allreduce_sum(sum)) / n;
  const float dev = sqrtf(fmaxf(sum_over_row_blocks(row16_allreduce_sum(sq)) / n - mean * mean, 0.f));
  return {shift + mean - kSelBinSpan * dev, (float)kSelBins / (2.f * kSelBinSpan * dev)};
}

// A listed token as one number, larger for what is kept first: the key, then the lower index.
__device__ __forceinline__ uint64_t* ranking_list(SelShared& sh) { return reinterpret_cast<uint64_t*>(sh.hist()); }
__device__ __forceinline__ void list_for_ranking(SelShared& sh, uint32_t key, uint32_t token) {
  const uint32_t slot = atomicAdd(&sh.cand_count, 1u);
  if (slot < (uint32_t)kSelRankMax) ranking_list(sh)[slot] = ((uint64_t)key << 32) | (uint32_t)~token;
}

// How many of the n <= kSelRankMax listed tokens come before token threadIdx.x / 4, which must be one of them: a quad per token,
// a quarter of the list per thread.
__device__ __forceinline__ uint32_t listed_rank(const uint64_t* list, uint32_t n) {
  const uint64_t mine = list[threadIdx.x >> 2];
  uint32_t rank = 0;
#pragma unroll 4
  for (uint32_t i = threadIdx.x & 3; i < n; i += 4) rank += list[i] > mine ? 1u : 0u;
  rank += (uint32_t)__builtin_amdgcn_mov_dpp((int)rank, 0xb1, 0xf, 0xf, true);   // quad_perm [1, 0, 3, 2]
  rank += (uint32_t)__builtin_amdgcn_mov_dpp((int)rank, 0x4e, 0xf, 0xf, true);   // quad_perm [2, 3, 0, 1]
  return rank;
}

// The `need` best of the listed tokens join gt_map: those with fewer than `need` listed before them.
__device__ __forceinline__ void keep_best_listed(SelShared& sh, uint32_t n, uint32_t need, uint32_t* gt_map) {
  const uint64_t* list = ranking_list(sh);
  const uint32_t j = threadIdx.x >> 2;
  if (j < n) {
    const uint32_t token = ~(uint32_t)list[j];
    if (listed_rank(list, n) < need && (threadIdx.x & 3) == 0) atomicOr(&gt_map[token >> 5], 1u << (token & 31));
  }
}

// Heads of at most kE * 1024 tokens: every thread holds kE scores in registers and nothing is read twice.  What bounds
// it is a chain of short steps in one workgroup per head (load, histogram, scan, classification, emission), so the
// steps are few: a histogram over linear bins, the tokens above the bin of the threshold kept, the few dozen inside it
// ranked one by one.  Where a sample says that linear bins would not spread the scores (8 of a wave's 64 in one bin) or
// more than kSelRankMax tokens share the bin, the radix descent over the held keys narrows them instead.  8 heads of
// 32768 normal scores: 15 us, 256 heads 16 us, 8 heads of 4000: 7 us; of exp(3 x): 21 us; all equal: 29 us.  (With the
// keys cached in LDS, three radix levels over them and prefix sums through the LDS crossbar: 24, 30, 11, 24 and 99 us.)
// Emitting a run of 64 tokens at a time from a prefix count over runs instead of from the masks: 1.5 us more.
// The bins come from a few scores that every wave reads for itself (no barrier, no LDS), and the tokens inside a bin are gathered as
// bits of a round and listed afterwards, in place of a branch in each round: 16.4 -> 15.1 us for 8 heads of 32768, 18.0 -> 16.2 for 256.
// The first part of the choice among a head of at most kE * 1024 tokens, by the whole workgroup; thread t has tokens
// t, t + 1024, .. in rounds: v, their scores, and at_bin, whose values above `bin` are kept and below it not.  The n_left tokens
// at `bin` are to be ranked, `need` of them kept; more than kSelRankMax: they share one key, and the first `need` are kept.
// What lies past the end of the head is at a bin below 0, one to a lane: at one bin for all the atomics queued (8 heads of 2049 tokens 7.5 us, 6.8 so).
template <int kE>
__device__ __forceinline__ uint32_t held_bins(SelShared& sh, const float* __restrict__ u, int T, int budget, uint32_t* stage,
                                              float (&v)[kE], int (&at_bin)[kE], int& bin, uint32_t& need) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int rounds = (T + kSelThreads - 1) / kSelThreads;
  // the bins come from eight runs of 64 scores, the same in every wave: any bins give the same selection, these a short list
  // (158 of 256 from one to the next: unevenly spread, and not from the first tokens, whose scores can be unlike the others')
  constexpr int kRuns = 8;
  float x[kRuns];
#pragma unroll
  for (int j = 0; j < kRuns; ++j) x[j] = u[min((int)((int64_t)T * ((20 + 158 * j) & 255) >> 8) + lane, T - 1)];
  // round k, token k * 1024 + tid: a wave's 64 tokens of a round are two words of the bitmaps
#pragma unroll
  for (int k = 0; k < kE; ++k) v[k] = u[min(k * kSelThreads + tid, T - 1)];
  if (tid == 0) sh.cand_count = 0;
  for (int i = tid; i < kSelBins; i += kSelThreads) sh.hist()[i] = 0;
  need = (uint32_t)budget;   // rank of the threshold among the keys not yet decided (1-based)
  uint32_t prefix = 0, prefix_mask = 0;
  auto count = [&](auto fn) {
#pragma unroll
    for (int k = 0; k < kE; ++k)
      if (k * kSelThreads + tid < T) fn(order_key(v[k]));
  };
  const float first = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x[0])));
  const LinearBins bins = run_bins(x, is_finite_score(first) ? first : 0.f);
  bool crowded = false;
#pragma unroll
  for (int k = 0; k < kE; ++k) {
    at_bin[k] = bins.bin(v[k]);
    if (k % 8 == 0 && (k == 0 || (k + 1) * kSelThreads <= T)) crowded |= lanes_crowd(at_bin[k]);
    if (k * kSelThreads + tid >= T) at_bin[k] = ~lane;
  }
  uint32_t n_left = kSelRankMax + 1;
  bin = 0;
  if (!__syncthreads_or(crowded && wave * 64 + 64 <= T)) {
#pragma unroll
    for (int k = 0; k < kE; ++k)
      if (k < rounds) atomicAdd(&sh.hist()[at_bin[k]], 1u);   // uniform
    __syncthreads();
    find_bin(sh, kSelBins, need, [&](int b) { return sh.hist()[b]; });
    n_left = sh.found_count;
    bin = (int)sh.found_bin;
    if (n_left <= (uint32_t)kSelRankMax) need -= sh.found_above;
    __syncthreads();   // the histogram and found_* are rewritten
  }
  if (n_left > (uint32_t)kSelRankMax) {
#pragma unroll 1
    for (int level = 0; level < 3 && n_left > (uint32_t)kSelRankMax; ++level)
      n_left = descend_level(sh, stage, level, prefix, prefix_mask, need, count);
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      const uint32_t decided = order_key(v[k]) & prefix_mask;
      at_bin[k] = k * kSelThreads + tid >= T ? -1 : decided > prefix ? 2 : decided == prefix ? 1 : 0;
    }
    bin = 1;
  }
  return n_left;
}

// One bit per round of a thread: bit k is test(k).  The bits are shifted in from the highest round down.
template <int kE, typename Test>
__device__ __forceinline__ uint64_t round_bits(Test test) {
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int k = kE - 1; k >= 32; --k) hi = hi + hi + (test(k) ? 1u : 0u);
#pragma unroll
  for (int k = (kE < 32 ? kE : 32) - 1; k >= 0; --k) lo = lo + lo + (test(k) ? 1u : 0u);
  return (uint64_t)hi << 32 | lo;
}

// Lists the tokens of the rounds in `bits` for the ranking.  Their scores are read again: few threads have any, and a branch
// around each of the rounds' registers costs more.
__device__ __forceinline__ void list_rounds(SelShared& sh, const float* __restrict__ u, uint64_t bits) {
  while (__ballot(bits != 0ull) != 0ull) {
    if (bits) {
      const uint32_t token = (uint32_t)(__builtin_ctzll(bits) * kSelThreads) + threadIdx.x;
      list_for_ranking(sh, order_key(u[token]), token);
      bits &= bits - 1;
    }
  }
}

template <bool kInline, int kE>
__global__ void __launch_bounds__(kSelThreads)
select_held_kernel(SeqTable tab, InlineOffsets inl, SelRagged ragged, int32_t* __restrict__ offsets, int32_t* __restrict__ idx,
                   uint32_t* __restrict__ counts, int seg_base, int seg_stride, int map_words /* of the launch's longest head */) {
  extern __shared__ __align__(16) unsigned char smem[];
  SelShared& sh = *reinterpret_cast<SelShared*>(smem);
  uint32_t* gt_map = reinterpret_cast<uint32_t*>(smem + sizeof(SelShared));
  uint32_t* eq_map = gt_map + map_words;
  uint32_t* stage = eq_map + map_words;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int local_seg = blockIdx.x;
  const int seq = seq_of_unit(tab, local_seg);
  const int lh = local_seg - tab.first[seq];
  const int seg = seg_base + seq * seg_stride + lh;
  // a ragged segment can be no longer than the launch table says (registers and LDS are sized by it)
  const int T = ragged.flat != nullptr ? min(ragged.len[seg], tab.T[seq]) : tab.T[seq];
  if (tab.T[seq] > kE * kSelThreads) return;   // left to select_kernel
  const float* u = ragged.flat != nullptr ? ragged.flat + ragged.start[seg] : tab.scores[seq] + (size_t)lh * (size_t)T;
  const int off = kInline ? inl.v[seg] : offsets[seg];
  const int budget = (kInline ? inl.v[seg + 1] : offsets[seg + 1]) - off;
  if (kInline && tid == 0) {
    offsets[seg] = off;
    if (local_seg == (int)gridDim.x - 1) offsets[seg + 1] = off + budget;   // the total, by the launch's last block
  }
  int32_t* out = idx + off;
  if (counts != nullptr)   // not needed here, but left zero for the next scoring launch
    for (int i = tid; i < kLevel0Bins; i += kSelThreads) counts[(size_t)seg * kLevel0Bins + i] = 0;
  if (budget <= 0 || budget >= T) {   // nothing or everything is kept
    if (budget > 0)
      for (int i = tid; i < T; i += kSelThreads) out[i] = i;
    return;
  }

  float v[kE];
  int at_bin[kE], bin;
  uint32_t need;
  const uint32_t n_left = held_bins<kE>(sh, u, T, budget, stage, v, at_bin, bin, need);
  const int rounds = (T + kSelThreads - 1) / kSelThreads;
  if (n_left <= (uint32_t)kSelRankMax) {
    // tokens above the undecided bin to the bitmap, those inside it to the list
    list_rounds(sh, u, round_bits<kE>([&](int k) { return at_bin[k] == bin; }));
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      if (k < rounds) {   // uniform
        const unsigned long long m = __ballot(at_bin[k] > bin);
        if (lane == 0) reinterpret_cast<unsigned long long*>(gt_map)[k * kSelWaves + wave] = m;
      }
    }
    __syncthreads();
    keep_best_listed(sh, n_left, need, gt_map);
    __syncthreads();
    // kept tokens ahead of every wave and round, then every round's tokens straight to their places
    const unsigned long long* masks = reinterpret_cast<const unsigned long long*>(gt_map);
    const int n_masks = rounds * kSelWaves;   // at most 544: one per thread
    const uint32_t cnt = tid < n_masks ? (uint32_t)__popcll(masks[tid]) : 0u;
    const uint32_t incl = wave_inclusive_scan(cnt);
    if (lane == 63) sh.wave_tot[wave] = incl;
    __syncthreads();
    const uint32_t before_wave = waves_before(sh.wave_tot, wave, lane);   // by all lanes
    if (tid < n_masks) eq_map[tid] = before_wave + incl - cnt;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      if (k < rounds) {
        const unsigned long long m = masks[k * kSelWaves + wave];
        const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if ((m >> lane) & 1ull) out[eq_map[k * kSelWaves + wave] + before] = k * kSelThreads + tid;
      }
    }
    return;
  }
  // more than kSelRankMax copies of the threshold key
#pragma unroll
  for (int k = 0; k < kE; ++k) {
    if (k < rounds) {   // uniform
      const unsigned long long m_gt = __ballot(at_bin[k] > bin);
      const unsigned long long m_eq = __ballot(at_bin[k] == bin);
      if (lane == 0) {
        reinterpret_cast<unsigned long long*>(gt_map)[k * kSelWaves + wave] = m_gt;
        reinterpret_cast<unsigned long long*>(eq_map)[k * kSelWaves + wave] = m_eq;
      }
    }
  }
  __syncthreads();
  emit_from_bitmaps<true>(sh, T, need, (uint32_t)budget, out, gt_map, eq_map, stage);
}

// The share of a block of the one launch: rows p0 .. p1 - 1 (none: p0 >= p1) of the kept tokens of a head.
struct SelShare {
  int seq, lh, seg, T, off, budget, p0, p1;
};
__device__ __forceinline__ SelShare block_share(const SeqTable& tab, const int32_t* __restrict__ offsets, uint32_t* __restrict__ counts,
                                                int seg_base, int seg_stride, int rows_per_block) {
  SelShare x;
  const int lane = threadIdx.x & 63;
  const int n_segs = tab.first[tab.n];   // at most 64: a lane each
  // every head has one block for each rows_per_block of its rows, and at least one
  int my_off = 0, my_budget = 0, my_seg = 0;
  if (lane < n_segs) {
    int seq = 0;
    while (seq + 1 < tab.n && lane >= tab.first[seq + 1]) ++seq;
    my_seg = seg_base + seq * seg_stride + lane - tab.first[seq];
    my_off = offsets[my_seg];
    my_budget = offsets[my_seg + 1] - my_off;
  }
  const uint32_t my_blocks = lane < n_segs ? (uint32_t)max(1, (my_budget + rows_per_block - 1) / rows_per_block) : 0u;
  const uint32_t last = wave_inclusive_scan(my_blocks);
  const unsigned long long at = __ballot(last > blockIdx.x);
  const int local_seg = at == 0ull ? 0 : __builtin_ctzll(at);
  const int part = (int)blockIdx.x - __builtin_amdgcn_readlane((int)(last - my_blocks), local_seg);
  x.seg = __builtin_amdgcn_readlane(my_seg, local_seg);
  x.off = __builtin_amdgcn_readlane(my_off, local_seg);
  x.budget = __builtin_amdgcn_readlane(my_budget, local_seg);
  x.seq = seq_of_unit(tab, local_seg);
  x.lh = local_seg - tab.first[x.seq];
  x.T = tab.T[x.seq];
  x.p0 = part * rows_per_block;
  x.p1 = at == 0ull ? 0 : min(min(x.budget, x.T), x.p0 + rows_per_block);
  if (counts != nullptr && part == 0 && at != 0ull)   // no block reads them here: left zero for the next scoring launch
    for (int i = threadIdx.x; i < kLevel0Bins; i += kSelThreads) counts[(size_t)x.seg * kLevel0Bins + i] = 0;
  return x;
}

// The indices and the rows of a block's tokens (listed in LDS), 16 lanes a row, 64 rows a round of the workgroup.  Where the
// counters did not count these scores the list has gaps, and what lies there is clamped, never followed.
__device__ __forceinline__ void copy_share(const SeqTable& tab, const SelShare& x, const uint32_t* tokens, int32_t* __restrict__ idx,
                                           uint4* __restrict__ kp, uint4* __restrict__ vp) {
  const int tid = threadIdx.x;
  const int n_rows = x.p1 - x.p0;
  const uint32_t last = (uint32_t)x.T - 1u;
  for (int i = tid; i < n_rows; i += kSelThreads) idx[(size_t)x.off + x.p0 + i] = (int32_t)min(tokens[i], last);
  constexpr int kRound = kSelThreads / 16;
  constexpr int kU = 2;
  const int c = tid & 15;
  const uint4* kh = reinterpret_cast<const uint4*>(tab.k[x.seq]) + (size_t)x.lh * (size_t)x.T * kChunksPerRow + c;
  const uint4* vh = reinterpret_cast<const uint4*>(tab.v[x.seq]) + (size_t)x.lh * (size_t)x.T * kChunksPerRow + c;
  uint4* kd = kp + ((size_t)x.off + x.p0) * kChunksPerRow + c;
  uint4* vd = vp + ((size_t)x.off + x.p0) * kChunksPerRow + c;
#pragma unroll 1
  for (int i0 = tid >> 4; i0 < n_rows; i0 += kRound * kU) {
    uint4 kk[kU], vv[kU];
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      const size_t row = min(tokens[min(i0 + j * kRound, n_rows - 1)], last);
      kk[j] = load_stream16(kh + row * kChunksPerRow);
      vv[j] = load_stream16(vh + row * kChunksPerRow);
    }
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      const int i = i0 + j * kRound;
      if (i < n_rows) {
        store_stream16(kd + (size_t)i * kChunksPerRow, kk[j]);
        store_stream16(vd + (size_t)i * kChunksPerRow, vv[j]);
      }
    }
  }
}

// Top-k and compaction of few heads of at most kE * 1024 tokens in one launch (a layer evicted during prefill).  A head's
// choice is a chain of short steps in one workgroup, which leaves the rest of the chip idle, so it is made again in every block that copies rows
// of the head: blocks in proportion to the budgets, each with as many rows as the others (how many: lkv_shares.h).  What goes
// away is the second launch, the emission of all but a block's own indices, their way through memory and the search for a row's segment.  8 heads of 32768, 39 thousand rows: 26.8 us in two launches,
// 22.1 in one (the whole call with the linear scorer 51.4 -> 45.2, 46.9 with the two launches of today); of 4096 18.5 -> 14.7, 2 heads of
// 34000 30.3 -> 25.0.  Two rows' pieces
// in flight per thread: four were 0.1 to 0.8 us slower up to 100 rows a block, eight up to 1.6.
template <int kE>
__global__ void __launch_bounds__(kSelThreads)
select_compact_kernel(SeqTable tab, const int32_t* __restrict__ offsets, int32_t* __restrict__ idx, uint32_t* __restrict__ counts,
                      int seg_base, int seg_stride, int map_words, int rows_per_block, uint4* __restrict__ kp, uint4* __restrict__ vp) {
  extern __shared__ __align__(16) unsigned char smem[];
  SelShared& sh = *reinterpret_cast<SelShared*>(smem);
  uint32_t* gt_map = reinterpret_cast<uint32_t*>(smem + sizeof(SelShared));
  uint32_t* eq_map = gt_map + map_words;
  uint32_t* stage = eq_map + map_words;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const SelShare x = block_share(tab, offsets, counts, seg_base, seg_stride, rows_per_block);
  if (x.p0 >= x.p1) return;
  const int T = x.T, budget = x.budget, p0 = x.p0;
  const int n_rows = x.p1 - p0;
  uint32_t* tokens = stage;   // of the block's rows
  if (budget >= T) {   // everything is kept
    for (int i = tid; i < n_rows; i += kSelThreads) tokens[i] = (uint32_t)(p0 + i);
  } else {
    const float* u = tab.scores[x.seq] + (size_t)x.lh * (size_t)T;
    const int rounds = (T + kSelThreads - 1) / kSelThreads;
    const int groups = rounds * kSelWaves;   // of 64 tokens, at most 544: a thread each
    unsigned long long* masks = reinterpret_cast<unsigned long long*>(gt_map);
    float v[kE];
    int at_bin[kE], bin;
    uint32_t need;
    const uint32_t n_left = held_bins<kE>(sh, u, T, budget, stage, v, at_bin, bin, need);
    const bool ranked = n_left <= (uint32_t)kSelRankMax;
    if (ranked) list_rounds(sh, u, round_bits<kE>([&](int k) { return at_bin[k] == bin; }));
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      if (k < rounds) {   // uniform
        const unsigned long long m = __ballot(at_bin[k] > bin);
        if (lane == 0) masks[k * kSelWaves + wave] = m;
      }
    }
    if (!ranked) {
#pragma unroll
      for (int k = 0; k < kE; ++k) {
        if (k < rounds) {   // uniform
          const unsigned long long m = __ballot(at_bin[k] == bin);
          if (lane == 0) reinterpret_cast<unsigned long long*>(eq_map)[k * kSelWaves + wave] = m;
        }
      }
    }
    __syncthreads();
    if (ranked) {
      keep_best_listed(sh, n_left, need, gt_map);
      __syncthreads();
    }
    unsigned long long m = tid < groups ? masks[tid] : 0ull;
    if (!ranked) {   // the first `need` copies of the threshold key join the tokens above it
      const unsigned long long eq = tid < groups ? reinterpret_cast<const unsigned long long*>(eq_map)[tid] : 0ull;
      const uint32_t n_eq = (uint32_t)__popcll(eq);
      const uint32_t incl = wave_inclusive_scan(n_eq);
      if (lane == 63) sh.wave_eq[wave] = incl;
      __syncthreads();
      const uint32_t before = waves_before(sh.wave_eq, wave, lane) + incl - n_eq;
      const uint32_t take = before < need ? min(n_eq, need - before) : 0u;
      const uint32_t n_low = (uint32_t)__popc((uint32_t)eq);
      m |= lowest_set_bits((uint32_t)eq, min(take, n_low));
      if (take > n_low) m |= (unsigned long long)lowest_set_bits((uint32_t)(eq >> 32), take - n_low) << 32;
    }
    // the tokens of the block's rows in order
    const uint32_t cnt = (uint32_t)__popcll(m);
    const uint32_t incl = wave_inclusive_scan(cnt);
    if (lane == 63) sh.wave_tot[wave] = incl;
    __syncthreads();
    int at = (int)(waves_before(sh.wave_tot, wave, lane) + incl - cnt) - p0;   // place of the group's first among them
    const unsigned long long some = __ballot(at < n_rows && at + (int)cnt > 0);   // groups with a row of the block
    if (__popcll(some) <= 16) {   // few (a dense head): all lanes on one after the other
      for (unsigned long long left = some; left != 0ull; left &= left - 1) {
        const int g = __builtin_ctzll(left);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, g);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(m >> 32), g);
        const int i = __builtin_amdgcn_readlane(at, g) + (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
        if ((((lane < 32 ? lo : hi) >> (lane & 31)) & 1u) && i >= 0 && i < n_rows) tokens[i] = (uint32_t)((wave * 64 + g) * 64 + lane);
      }
    } else {
      unsigned long long bits = (some >> lane) & 1ull ? m : 0ull;
      while (__ballot(bits != 0ull) != 0ull) {
        if (bits) {
          if (at >= 0 && at < n_rows) tokens[at] = (uint32_t)(tid * 64 + __builtin_ctzll(bits));
          ++at;
          bits &= bits - 1;
        }
      }
    }
  }
  __syncthreads();
  copy_share(tab, x, tokens, idx, kp, vp);
}

// The words of a bitmap of up to kSelMaxBitmapT tokens, thread t's t, t + 1024, ..: all on their way at once.
constexpr int kMapRounds = (kSelMaxBitmapT / 32 + kSelThreads - 1) / kSelThreads;
__device__ __forceinline__ void load_map(const uint32_t* __restrict__ map, int n_words, uint32_t (&words)[kMapRounds]) {
#pragma unroll
  for (int j = 0; j < kMapRounds; ++j) {
    const int w = j * kSelThreads + threadIdx.x;
    words[j] = 0;
    if (j * kSelThreads < n_words) words[j] = w < n_words ? map[w] : 0u;   // the outer condition is uniform
  }
}

// Lists their tokens (LDS list of up to kSelCandCap, sh.cand_count of them), in no particular order.  Starts from an empty list;
// a barrier has to pass before the list is read.
__device__ __forceinline__ void list_map(SelShared& sh, const uint32_t (&words)[kMapRounds], int n_words, uint32_t* cand) {
  uint32_t n_bits = 0;
#pragma unroll
  for (int j = 0; j < kMapRounds; ++j) n_bits += (uint32_t)__popc(words[j]);
  // one place in the list per wave, shared out by a prefix count
  const uint32_t incl = wave_inclusive_scan(n_bits);
  uint32_t base = 0;
  if ((threadIdx.x & 63) == 63) base = atomicAdd(&sh.cand_count, incl);
  uint32_t slot = last_lane(base) + incl - n_bits;
#pragma unroll
  for (int j = 0; j < kMapRounds; ++j) {
    if (j * kSelThreads < n_words) {   // uniform
      uint32_t bits = words[j];
      while (__ballot(bits != 0u) != 0ull) {
        if (bits) {
          if (slot < (uint32_t)kSelCandCap) cand[slot] = (uint32_t)(j * kSelThreads + threadIdx.x) * 32u + (uint32_t)__builtin_ctz(bits);
          ++slot;
          bits &= bits - 1;
        }
      }
    }
  }
}

// Settles the n_cand listed tokens of an undecided bin: those that are kept join gt_map.  True: all of them.  False: more than
// kSelRankMax share the threshold key; those above it joined, eq_map has its copies, and the first `need` of these are kept.
// `level`: levels of the descent that the bin stands for: 0, or 1 when the keys in it agree in their first digit.  `space`: where the
// list lies, used for histograms once the tokens are in registers.
__device__ __forceinline__ bool settle_listed(SelShared& sh, const float* __restrict__ u, int T, int n_words, uint32_t n_cand, int level,
                                              uint32_t& need, uint32_t* gt_map, uint32_t* eq_map, uint32_t* space) {
  const int tid = threadIdx.x;
  // the listed tokens and their keys, in registers: one round of gathers, all in flight
  constexpr int kHeldCand = kSelCandCap / kSelThreads;
  uint32_t token[kHeldCand], key[kHeldCand];
#pragma unroll
  for (int k = 0; k < kHeldCand; ++k) {
    token[k] = 0;
    if (k == 0 || (uint32_t)(k * kSelThreads) < n_cand)   // uniform
      token[k] = min(space[min((uint32_t)(k * kSelThreads + tid), max(n_cand, 1u) - 1)], (uint32_t)T - 1);   // in range whatever the counts said
  }
#pragma unroll
  for (int k = 0; k < kHeldCand; ++k) {
    key[k] = 0;
    if (k == 0 || (uint32_t)(k * kSelThreads) < n_cand) key[k] = order_key(u[token[k]]);
  }
  auto for_each_listed = [&](auto fn) {
#pragma unroll
    for (int k = 0; k < kHeldCand; ++k)
      if ((uint32_t)(k * kSelThreads + tid) < n_cand) fn(key[k], token[k]);
  };
  if (tid == 0) { sh.cand_count = 0; sh.first_key = key[0]; }
  // keys that agree in their first digit mostly differ in the next, and one copy of its histogram will do (2.9 -> 1.3 us)
  const bool crowded = level == 0 || lanes_crowd((int)(key[0] >> 10 & 2047u));
  for (int i = tid; i < kSelBins; i += kSelThreads) sh.hist()[i] = 0;
  const bool copies = __syncthreads_or(crowded && (uint32_t)(tid | 63) < n_cand) != 0;
  // the list is dead: its space becomes the staging buffer; the list for the ranking starts empty
  uint32_t prefix_mask = level == 0 ? 0u : 0xffe00000u;
  uint32_t prefix = sh.first_key & prefix_mask;   // bits of the threshold key decided so far
  uint32_t n_left = n_cand;
  if (!copies && n_left > (uint32_t)kSelRankMax) {
    for_each_listed([&](uint32_t k, uint32_t) { atomicAdd(&sh.hist()[k >> 10 & 2047u], 1u); });
    __syncthreads();
    find_bin(sh, kSelBins, need, [&](int bin) { return sh.hist()[bin]; });
    n_left = enter_found_bin(sh, 1, prefix, prefix_mask, need);
    level = 2;
  }
#pragma unroll 1
  for (; level < 3 && n_left > (uint32_t)kSelRankMax; ++level)
    n_left = descend_level(sh, space, level, prefix, prefix_mask, need, [&](auto fn) { for_each_listed([&](uint32_t k, uint32_t) { fn(k); }); });
  if (n_left <= (uint32_t)kSelRankMax) {
    for_each_listed([&](uint32_t k, uint32_t t) {
      const uint32_t decided = k & prefix_mask;
      if (decided > prefix) atomicOr(&gt_map[t >> 5], 1u << (t & 31));
      else if (decided == prefix) list_for_ranking(sh, k, t);
    });
    __syncthreads();
    keep_best_listed(sh, min(n_left, sh.cand_count), need, gt_map);   // no more than were listed, whatever the counts said
    __syncthreads();
    return true;
  }
  for (int i = tid; i < n_words; i += kSelThreads) eq_map[i] = 0;
  __syncthreads();
  const uint32_t thr_listed = prefix;
  for_each_listed([&](uint32_t k, uint32_t t) {
    if (k > thr_listed) atomicOr(&gt_map[t >> 5], 1u << (t & 31));
    else if (k == thr_listed) atomicOr(&eq_map[t >> 5], 1u << (t & 31));
  });
  __syncthreads();
  return false;
}

// kCounted: the first-level digits of every segment's scores have already been counted by the scoring launch
// (`counts`: uint32 [segments][kLevel0Bins]); the block takes its histogram from there instead of from a pass over
// the scores, and leaves the counters zero for the next scoring launch.
template <bool kInline, bool kCounted>
__global__ void __launch_bounds__(kSelThreads)
select_kernel(SeqTable tab, InlineOffsets inl, SelRagged ragged, int32_t* __restrict__ offsets, int32_t* __restrict__ idx,
              uint32_t* __restrict__ counts,
              const uint32_t* __restrict__ pre_maps /* per segment [2][pre_words]: written by select_classify_kernel, or null */,
              int pre_words,
              int seg_base, int seg_stride /* global segment = seg_base + sequence * seg_stride + head */,
              int held_limit /* heads of at most this many tokens are left to select_held_kernel */,
              int bitmap_limit /* heads of up to this many tokens use the LDS bitmaps */,
              int bitmap_stage_off /* word offset of the staging buffer in the region */) {
  extern __shared__ __align__(16) unsigned char smem[];
  SelShared& sh = *reinterpret_cast<SelShared*>(smem);
  uint32_t* region = reinterpret_cast<uint32_t*>(smem + sizeof(SelShared));

  const int tid = threadIdx.x;
  const int local_seg = blockIdx.x;
  const int seq = seq_of_unit(tab, local_seg);
  const int lh = local_seg - tab.first[seq];
  const int seg = seg_base + seq * seg_stride + lh;
  // a ragged segment can be no longer than the launch table says (the LDS region is sized by it)
  const int T = ragged.flat != nullptr ? min(ragged.len[seg], tab.T[seq]) : tab.T[seq];
  if (tab.T[seq] <= held_limit) return;
  const float* u = ragged.flat != nullptr ? ragged.flat + ragged.start[seg] : tab.scores[seq] + (size_t)lh * (size_t)T;
  const int off = kInline ? inl.v[seg] : offsets[seg];
  const int budget = (kInline ? inl.v[seg + 1] : offsets[seg + 1]) - off;
  if (kInline && tid == 0) {
    offsets[seg] = off;
    if (local_seg == (int)gridDim.x - 1) offsets[seg + 1] = off + budget;   // the total, by the launch's last block
  }
  int32_t* out = idx + off;
  uint32_t* my_counts = kCounted ? counts + (size_t)seg * kLevel0Bins : nullptr;
  if (budget <= 0 || budget >= T) {   // nothing or everything is kept
    if (kCounted)
      for (int i = tid; i < kLevel0Bins; i += kSelThreads) my_counts[i] = 0;
    if (budget > 0)
      for (int i = tid; i < T; i += kSelThreads) out[i] = i;
    return;
  }
  if (kCounted) {
    for (int i = tid; i < kSelBins; i += kSelThreads) {
      sh.hist()[i] = my_counts[i];
      my_counts[i] = 0;
    }
    __syncthreads();
  }

  uint32_t* copies = region + bitmap_stage_off;   // of a histogram; then the listed tokens, then the staging buffer
  uint32_t prefix = 0;        // bits of the threshold key decided so far
  uint32_t prefix_mask = 0;   // which bits those are
  uint32_t need = (uint32_t)budget;   // rank of the threshold among keys that match the prefix (1-based)

  auto count = [&](auto fn) { for_each_global_key(u, T, [&](uint32_t key, int) { fn(key); }); };
  // The first level leaves one bin undecided: of the radix digits when the scoring launch has counted them, else of
  // linear bins over what four runs of 1024 scores say about the distribution.  When the tokens of that bin are few
  // enough to list (their indices, in the space the emission stages through later), one more pass over the scores settles
  // everything above the bin and collects the list; the rest touches the listed tokens only, their scores in registers.
  uint32_t n_cand;
  LinearBins bins = {0.f, 0.f};
  bool keyed = kCounted;
  uint32_t bin0;
  if (!kCounted) {
    const float first = u[0];
    const float shift = is_finite_score(first) ? first : 0.f;
    float x[4], n = 0.f, sum = 0.f, sq = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = u[(int)(((int64_t)T * k) >> 2) + min(tid, max((T >> 2) - 1, 0))];   // a ragged segment may be short
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool fin = is_finite_score(x[k]);
      const float d = fin ? x[k] - shift : 0.f;
      n += fin ? 1.f : 0.f;
      sum += d;
      sq = fmaf(d, d, sq);
    }
    bins = linear_bins(sh, shift, n, sum, sq);
    bool crowded = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) crowded |= lanes_crowd(bins.bin(x[k]));
    keyed = __syncthreads_or(crowded && (tid | 63) < (T >> 2));
  }
  if (kCounted) {
    n_cand = descend_counted_level(sh, prefix, prefix_mask, need);
    bin0 = prefix >> 21;
  } else if (keyed) {
    n_cand = descend_level(sh, copies, 0, prefix, prefix_mask, need, count);
    bin0 = prefix >> 21;
  } else {
    for_each_global_score(u, T, [&](float s, int) { atomicAdd(&sh.hist()[bins.bin(s)], 1u); });
    __syncthreads();
    find_bin(sh, kSelBins, need, [&](int bin) { return sh.hist()[bin]; });
    n_cand = sh.found_count;
    bin0 = sh.found_bin;
    if (n_cand <= (uint32_t)kSelCandCap && T <= bitmap_limit) need -= sh.found_above;
    __syncthreads();   // found_* and the histogram are rewritten below
  }
  if (T <= bitmap_limit && n_cand <= (uint32_t)kSelCandCap) {
    const int n_words = (T + 31) >> 5;
    uint32_t* gt_map = region;
    uint32_t* eq_map = region + n_words;
    uint32_t* cand = region + bitmap_stage_off;
    if (kCounted && pre_maps != nullptr) {
      // the pass over the scores has been done by the blocks of select_classify_kernel: take its two bitmaps
      // (above the undecided bin / inside it) and list the tokens inside
      const uint32_t* pre_gt = pre_maps + (size_t)seg * 2 * pre_words;
      uint32_t above[kMapRounds], inside[kMapRounds];
      load_map(pre_gt, n_words, above);
      load_map(pre_gt + pre_words, n_words, inside);
      if (tid == 0) sh.cand_count = 0;
#pragma unroll
      for (int j = 0; j < kMapRounds; ++j)
        if (j * kSelThreads + tid < n_words) gt_map[j * kSelThreads + tid] = above[j];
      __syncthreads();
      list_map(sh, inside, n_words, cand);
      __syncthreads();
    } else {
      for (int i = tid; i < n_words; i += kSelThreads) gt_map[i] = 0;
      if (tid == 0) sh.cand_count = 0;
      __syncthreads();
      for_each_global_score(u, T, [&](float s, int i) {
        const uint32_t top = keyed ? order_key(s) >> 21 : (uint32_t)bins.bin(s);
        if (top > bin0) {
          atomicOr(&gt_map[i >> 5], 1u << (i & 31));
        } else if (top == bin0) {
          // (handing out slots per wave with a ballot was measured slower than the plain atomic)
          const uint32_t slot = atomicAdd(&sh.cand_count, 1u);
          if (slot < (uint32_t)kSelCandCap) cand[slot] = (uint32_t)i;
        }
      });
      __syncthreads();
    }
    if (settle_listed(sh, u, T, n_words, n_cand, keyed ? 1 : 0, need, gt_map, eq_map, cand))
      emit_from_bitmaps<false>(sh, T, need, (uint32_t)budget, out, gt_map, eq_map, region + bitmap_stage_off);
    else
      emit_from_bitmaps<true>(sh, T, need, (uint32_t)budget, out, gt_map, eq_map, region + bitmap_stage_off);
    return;
  }
#pragma unroll 1
  for (int level = keyed ? 1 : 0; level < 3; ++level) descend_level(sh, copies, level, prefix, prefix_mask, need, count);
  const uint32_t thr = prefix;   // full 32-bit key of the budget-th largest score; keep `need` of its copies

  if (T <= bitmap_limit) {
    const int n_words = (T + 31) >> 5;
    uint32_t* gt_map = region;
    uint32_t* eq_map = region + n_words;
    for (int i = tid; i < 2 * n_words; i += kSelThreads) region[i] = 0;
    __syncthreads();
    for_each_global_key(u, T, [&](uint32_t key, int i) {
      if (key > thr) atomicOr(&gt_map[i >> 5], 1u << (i & 31));
      else if (key == thr) atomicOr(&eq_map[i >> 5], 1u << (i & 31));
    });
    __syncthreads();
    emit_from_bitmaps<true>(sh, T, need, (uint32_t)budget, out, gt_map, eq_map, region + bitmap_stage_off);
  } else {
    emit_from_keys(sh, T, thr, need, (uint32_t)budget, out, [&](int i) { return order_key(u[i]); });
  }
}


// First half of a top-k whose heads are split over several workgroups (launches over few, long heads: one layer at
// a time).  Needs the first-level counts of the scoring launch.  Every block finds the undecided first-level bin of
// its head from the counts (a 2048-bin scan, repeated in each block rather than communicated) and classifies its
// slice of the scores against it into two global bitmaps: above the bin (kept for certain), and inside it (the
// candidates the remaining two levels choose from).  select_kernel then starts from the bitmaps instead of passing
// over the scores.  The counters are left as they are (select_kernel reads them again and zeroes them).  A head
// whose undecided bin holds more tokens than select_kernel can list is skipped here and takes the unsplit route there.
template <bool kFinish>
__global__ void __launch_bounds__(kSelThreads)
select_classify_kernel(SeqTable tab, const int32_t* __restrict__ offsets, const uint32_t* __restrict__ counts,
                       uint32_t* __restrict__ pre_maps, int pre_words, int seg_base, int seg_stride, int split) {
  __shared__ SelShared sh;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int local_seg = blockIdx.x / split;
  const int part = blockIdx.x - local_seg * split;
  const int seq = seq_of_unit(tab, local_seg);
  const int lh = local_seg - tab.first[seq];
  const int seg = seg_base + seq * seg_stride + lh;
  const int T = tab.T[seq];
  const float* u = tab.scores[seq] + (size_t)lh * (size_t)T;
  const int budget = offsets[seg + 1] - offsets[seg];
  if (budget <= 0 || budget >= T) return;
  const uint32_t* my_counts = counts + (size_t)seg * kLevel0Bins;
  for (int i = tid; i < kSelBins; i += kSelThreads) sh.hist()[i] = my_counts[i];
  __syncthreads();
  uint32_t prefix = 0, prefix_mask = 0, need = (uint32_t)budget;
  const uint32_t n_cand = descend_counted_level(sh, prefix, prefix_mask, need);
  if (n_cand > (uint32_t)kSelCandCap) {
    // too many to list: left to select_kernel, or (kFinish) all that is kept found here, by the head's first block, and nothing left inside
    if constexpr (kFinish) {
      if (part == 0) {
        extern __shared__ __align__(16) uint32_t space[];
        const int n_words = (T + 31) >> 5;
        uint32_t* gt_map = space;
        uint32_t* eq_map = space + n_words;
        uint32_t* copies = space + ((2 * n_words + 3) & ~3);
        auto count = [&](auto fn) { for_each_global_key(u, T, [&](uint32_t key, int) { fn(key); }); };
#pragma unroll 1
        for (int level = 1; level < 3; ++level) descend_level(sh, copies, level, prefix, prefix_mask, need, count);
        const uint32_t thr = prefix;
        for (int i = tid; i < 2 * n_words; i += kSelThreads) space[i] = 0;
        __syncthreads();
        for_each_global_key(u, T, [&](uint32_t key, int i) {
          if (key > thr) atomicOr(&gt_map[i >> 5], 1u << (i & 31));
          else if (key == thr) atomicOr(&eq_map[i >> 5], 1u << (i & 31));
        });
        __syncthreads();
        uint32_t* out_gt = pre_maps + (size_t)seg * 2 * pre_words;
        uint32_t seen = 0;   // copies of the threshold key in earlier words
        for (int w0 = 0; w0 < n_words; w0 += kSelThreads) {   // uniform
          const int w = w0 + tid;
          const uint32_t eq = w < n_words ? eq_map[w] : 0u, n = (uint32_t)__popc(eq);
          const uint32_t incl = wave_inclusive_scan(n);
          if (lane == 63) sh.wave_eq[wave] = incl;
          __syncthreads();
          const uint32_t before = seen + waves_before(sh.wave_eq, wave, lane) + incl - n;
          if (w < n_words) {
            out_gt[w] = gt_map[w] | lowest_set_bits(eq, before < need ? min(n, need - before) : 0u);
            out_gt[pre_words + w] = 0;
          }
          seen += wave_sum(lane < kSelWaves ? sh.wave_eq[lane] : 0u);
          __syncthreads();
        }
      }
    }
    return;
  }
  const uint32_t bin0 = prefix >> 21;
  uint32_t* out_gt = pre_maps + (size_t)seg * 2 * pre_words;
  uint32_t* out_in = out_gt + pre_words;
  // slices of whole 64-token groups (two bitmap words per wave step)
  const int groups = (T + 63) >> 6;
  const int per = (groups + split - 1) / split;
  const int g_lo = part * per, g_hi = min(groups, g_lo + per);
  constexpr int kU = 4;
  for (int g0 = g_lo + wave; g0 < g_hi; g0 += kSelWaves * kU) {
    float v[kU];
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const int i = (g0 + k * kSelWaves) * 64 + lane;
      v[k] = u[i < T ? i : T - 1];
    }
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const int g = g0 + k * kSelWaves;
      const int i = g * 64 + lane;
      const uint32_t top = order_key(v[k]) >> 21;
      const bool in = g < g_hi && i < T;
      const unsigned long long m_gt = __ballot(in && top > bin0);
      const unsigned long long m_in = __ballot(in && top == bin0);
      if (g < g_hi && lane < 2) {
        const int w = 2 * g + lane;
        if (w < pre_words) {
          out_gt[w] = (uint32_t)(m_gt >> (32 * lane));
          out_in[w] = (uint32_t)(m_in >> (32 * lane));
        }
      }
    }
  }
}

// The one launch for longer heads, after select_classify_kernel: every block that copies rows settles the listed tokens of its head for
// itself.  What bounds it: the copy (14 of 30 us for 8 heads of 131072, 105 thousand rows, 256 blocks), the way of the listed scores to each compute unit (4: one
// line for every token or two), the list 2.4, the descent 1.4.  In turn with one block per head that emits and a compaction behind it, the whole call
// with the 256-64-1 scorer: 8 heads of 131072 143.9 -> 138.6 us, 60001 80.7 -> 76.9, 2 heads of 100001 58.5 -> 49.9.
__global__ void __launch_bounds__(kSelThreads)
select_compact_long_kernel(SeqTable tab, const int32_t* __restrict__ offsets, int32_t* __restrict__ idx, uint32_t* __restrict__ counts,
                           const uint32_t* __restrict__ pre_maps, int pre_words, int seg_base, int seg_stride,
                           int map_words, int rows_per_block, uint4* __restrict__ kp, uint4* __restrict__ vp) {
  extern __shared__ __align__(16) unsigned char smem[];
  SelShared& sh = *reinterpret_cast<SelShared*>(smem);
  uint32_t* gt_map = reinterpret_cast<uint32_t*>(smem + sizeof(SelShared));
  uint32_t* eq_map = gt_map + map_words;
  uint32_t* stage = eq_map + map_words;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const SelShare x = block_share(tab, offsets, counts, seg_base, seg_stride, rows_per_block);
  if (x.p0 >= x.p1) return;
  const int T = x.T, p0 = x.p0;
  const int n_rows = x.p1 - p0;
  uint32_t* tokens = stage;   // of the block's rows
  if (x.budget >= T) {   // everything is kept
    for (int i = tid; i < n_rows; i += kSelThreads) tokens[i] = (uint32_t)(p0 + i);
  } else {
    const int n_words = (T + 31) >> 5;
    const uint32_t* pre_gt = pre_maps + (size_t)x.seg * 2 * pre_words;
    uint32_t kept[kMapRounds], inside[kMapRounds];
    load_map(pre_gt, n_words, kept);
    load_map(pre_gt + pre_words, n_words, inside);
    if (tid == 0) sh.cand_count = 0;
    uint32_t above = 0;   // tokens kept for certain
#pragma unroll
    for (int j = 0; j < kMapRounds; ++j) {
      if (j * kSelThreads + tid < n_words) gt_map[j * kSelThreads + tid] = kept[j];
      above += (uint32_t)__popc(kept[j]);
    }
    above = wave_sum(above);
    if (lane == 0) sh.wave_gt[wave] = above;
    __syncthreads();
    list_map(sh, inside, n_words, stage);
    __syncthreads();
    const uint32_t n_cand = min(sh.cand_count, (uint32_t)kSelCandCap);
    uint32_t need = (uint32_t)max(x.budget - (int)wave_sum(lane < kSelWaves ? sh.wave_gt[lane] : 0u), 0);
    __syncthreads();   // the list's counter is used again
    bool ranked = true;
    if (n_cand > 0)
      ranked = settle_listed(sh, tab.scores[x.seq] + (size_t)x.lh * (size_t)T, T, n_words, n_cand, 1, need, gt_map, eq_map, stage);
    // the words of the map, thread t's t, t + 1024, .., and what lies ahead of each: within its wave, then over waves and rounds
    uint32_t* totals = sh.hist();   // of a round and wave
    auto ahead = [&](uint32_t (&n)[kMapRounds]) {   // counts to the number ahead; a barrier on either side of the totals
#pragma unroll
      for (int j = 0; j < kMapRounds; ++j) {
        if (j * kSelThreads < n_words) {   // uniform
          const uint32_t incl = wave_inclusive_scan(n[j]);
          if (lane == 63) totals[j * kSelWaves + wave] = incl;
          n[j] = incl - n[j];
        }
      }
      __syncthreads();
      uint32_t carry = 0;
#pragma unroll
      for (int j = 0; j < kMapRounds; j += 4) {   // 64 totals a lane each
        if (j * kSelThreads < n_words) {
          const uint32_t mine = (j + (lane >> 4)) * kSelThreads < n_words ? totals[j * kSelWaves + lane] : 0u;
          const uint32_t incl = wave_inclusive_scan(mine);
#pragma unroll
          for (int i = 0; i < 4 && j + i < kMapRounds; ++i)
            n[j + i] += carry + (uint32_t)__builtin_amdgcn_readlane((int)(incl - mine), i * kSelWaves + wave);
          carry += last_lane(incl);
        }
      }
    };
    uint32_t word[kMapRounds], before[kMapRounds];
#pragma unroll
    for (int j = 0; j < kMapRounds; ++j) {
      const int w = j * kSelThreads + tid;
      word[j] = j * kSelThreads < n_words && w < n_words ? gt_map[w] : 0u;
    }
    if (!ranked) {   // the first `need` copies of the threshold key join the tokens above it
      uint32_t eq[kMapRounds];
#pragma unroll
      for (int j = 0; j < kMapRounds; ++j) {
        const int w = j * kSelThreads + tid;
        eq[j] = j * kSelThreads < n_words && w < n_words ? eq_map[w] : 0u;
        before[j] = (uint32_t)__popc(eq[j]);
      }
      ahead(before);
#pragma unroll
      for (int j = 0; j < kMapRounds; ++j)
        word[j] |= lowest_set_bits(eq[j], before[j] < need ? min((uint32_t)__popc(eq[j]), need - before[j]) : 0u);
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < kMapRounds; ++j) before[j] = (uint32_t)__popc(word[j]);
    ahead(before);
#pragma unroll
    for (int j = 0; j < kMapRounds; ++j) {
      if (j * kSelThreads < n_words) {   // uniform
        uint32_t bits = word[j];
        int at = (int)before[j] - p0;   // place of the word's first among the block's rows
        if (at >= n_rows || at + __popc(bits) <= 0) bits = 0;
        if (at < 0) {   // the rows of the block before
          bits ^= lowest_set_bits(bits, (uint32_t)-at);
          at = 0;
        }
        if (at + __popc(bits) > n_rows) bits = lowest_set_bits(bits, (uint32_t)(n_rows - at));
        const uint32_t first = (uint32_t)(j * kSelThreads + tid) * 32u;
        for (; bits; bits &= bits - 1) tokens[at++] = first + (uint32_t)__builtin_ctz(bits);
      }
    }
  }
  __syncthreads();
  copy_share(tab, x, tokens, idx, kp, vp);
}

hipError_t select_prepare() {
  const int lds = (int)(sizeof(SelShared) + (size_t)kSelRegionBytes);
  const void* kernels[] = {
      reinterpret_cast<const void*>(select_kernel<false, false>), reinterpret_cast<const void*>(select_kernel<true, false>),
      reinterpret_cast<const void*>(select_kernel<false, true>),  reinterpret_cast<const void*>(select_kernel<true, true>),
#define LKV_HELD_KERNELS(kE)                                                                                             \
  reinterpret_cast<const void*>(select_held_kernel<false, kE>), reinterpret_cast<const void*>(select_held_kernel<true, kE>)
      LKV_HELD_KERNELS(8), LKV_HELD_KERNELS(16), LKV_HELD_KERNELS(kSelMaxHeld),
      reinterpret_cast<const void*>(select_compact_kernel<8>), reinterpret_cast<const void*>(select_compact_kernel<16>),
      reinterpret_cast<const void*>(select_compact_kernel<kSelMaxHeld>), reinterpret_cast<const void*>(select_compact_long_kernel)};
#undef LKV_HELD_KERNELS
  for (const void* k : kernels)
    if (hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds)) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(select_classify_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             kSelRegionBytes);   // its SelShared is static
}

int select_inline_capacity() { return kSelInlineOffsets; }
int select_max_bitmap_tokens() { return kSelMaxBitmapT; }

// Rows of a block of the one-launch top-k and compaction (and the blocks), 0 where the two launches are better.  Heads too long for
// the registers need the scoring launch's counts and room for bitmaps of `pre_words` words; there up to kFuseLongHeads of them (32 heads of
// 36000: 180 -> 177 us, but 185 -> 188 where one block a head has to finish the choice).
int select_compact_rows(const SeqTable& tab, const int32_t* budgets, int seq_stride, int64_t total_rows, const uint32_t* counts,
                        int pre_words, int* blocks) {
  const int segs = tab.first[tab.n];
  if (segs > kFuseMaxHeads || total_rows <= 0) return 0;
  int least = tab.T[0], most = 0;
  for (int i = 0; i < tab.n; ++i) {
    least = tab.T[i] < least ? tab.T[i] : least;
    most = tab.T[i] > most ? tab.T[i] : most;
  }
  if (most > kSelMaxHeldT && (segs > kFuseLongHeads || least <= kSelMaxHeldT || counts == nullptr || most > kSelMaxBitmapT ||
                              (most + 31) / 32 > pre_words))
    return 0;
  return share_rows(budgets, tab.n, seq_stride, segs / tab.n, total_rows, most > kSelMaxHeldT, blocks);
}

static int classify_split(int segs) {
  const int split = kSelSplitTargetBlocks / segs;
  return split > kSelSplitMax ? kSelSplitMax : split;
}

void launch_select_compact(const SeqTable& tab, const int32_t* offsets, int32_t* idx, int seg_base, int seg_stride,
                           int rows_per_block, int blocks, uint32_t* counts, uint32_t* pre_maps, int pre_words, void* kp, void* vp,
                           hipStream_t stream) {
  int most = 0;
  for (int i = 0; i < tab.n; ++i) most = tab.T[i] > most ? tab.T[i] : most;
  if (most > kSelMaxHeldT) {
    const int split = classify_split(tab.first[tab.n]), map_words = (most + 31) / 32;
    const size_t maps = (2 * (size_t)map_words + 3) / 4 * 16;
    hipLaunchKernelGGL(select_classify_kernel<true>, dim3(tab.first[tab.n] * split), dim3(kSelThreads), maps + kSelStageBytes, stream, tab,
                       offsets, counts, pre_maps, pre_words, seg_base, seg_stride, split);
    hipLaunchKernelGGL(select_compact_long_kernel, dim3(blocks), dim3(kSelThreads), sizeof(SelShared) + maps + kSelStageBytes, stream, tab,
                       offsets, idx, counts, pre_maps, pre_words, seg_base, seg_stride, (int)(maps / 8), rows_per_block,
                       static_cast<uint4*>(kp), static_cast<uint4*>(vp));
    return;
  }
  const int map_words = (most + kSelThreads - 1) / kSelThreads * 32;
  const size_t lds = sizeof(SelShared) + 2 * (size_t)map_words * 4 + kSelStageBytes;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kSelThreads), lds, stream, tab, offsets, idx, counts, seg_base, seg_stride, map_words,
                       rows_per_block, static_cast<uint4*>(kp), static_cast<uint4*>(vp));
  };
  if (most > 16 * kSelThreads) launch(select_compact_kernel<kSelMaxHeld>);
  else if (most > 8 * kSelThreads) launch(select_compact_kernel<16>);
  else launch(select_compact_kernel<8>);
}

// `host_offsets` non-null: all n_total_segments + 1 offsets are passed in the kernel arguments
// (n_total_segments < kSelInlineOffsets) and the kernel writes the device array; null: the
// device array has already been filled.
void launch_select(const SeqTable& tab, const int32_t* host_offsets, int n_total_segments, int32_t* offsets,
                   int32_t* idx, int seg_base, int seg_stride, hipStream_t stream, const float* ragged_scores,
                   const int32_t* ragged_start, const int32_t* ragged_len, uint32_t* counts, uint32_t* pre_maps,
                   int pre_words) {
  const int segs = tab.first[tab.n];
  if (segs <= 0) return;
  // heads whose scores fit a workgroup's registers, and longer ones; the LDS of either kernel is sized for the longest
  // sequence of this launch that it takes
  int held_limit = 0, longer = 0, bitmap_limit = 0;
  for (int i = 0; i < tab.n; ++i) {
    const int T = tab.T[i];
    if (T <= kSelMaxHeldT) held_limit = T > held_limit ? T : held_limit;
    else ++longer;
    if (T > kSelMaxHeldT && T <= kSelMaxBitmapT && T > bitmap_limit) bitmap_limit = T;
  }
  const int map_words = (held_limit + kSelThreads - 1) / kSelThreads * 32;
  const size_t held_lds = sizeof(SelShared) + 2 * (size_t)map_words * 4 + kSelStageBytes;
  const size_t bitmap_stage_off = (2 * (size_t)((bitmap_limit + 31) / 32) + 3) & ~(size_t)3;   // two bitmaps, then the staging buffer
  const size_t lds = sizeof(SelShared) + bitmap_stage_off * 4 + kSelStageBytes;
  const SelRagged ragged = {ragged_scores, ragged_start, ragged_len};
  InlineOffsets inl = {};
  if (host_offsets != nullptr)
    for (int i = 0; i <= n_total_segments; ++i) inl.v[i] = host_offsets[i];
  const dim3 grid(segs), block(kSelThreads);
  // Few long heads (a layer at a time): split the pass over the scores of every head over several workgroups first.
  // Needs the first-level counts, room for the two bitmaps, heads too long for the registers and offsets on the device.
  bool split_heads = counts != nullptr && pre_maps != nullptr && host_offsets == nullptr && ragged_scores == nullptr &&
                     held_limit == 0 && bitmap_limit > 0 && segs <= kSelSplitMaxHeads;
  for (int i = 0; i < tab.n && split_heads; ++i)
    if (tab.T[i] > kSelMaxBitmapT || (tab.T[i] + 31) / 32 > pre_words) split_heads = false;
  if (split_heads) {
    const int split = classify_split(segs);
    hipLaunchKernelGGL(select_classify_kernel<false>, dim3(segs * split), block, 0, stream, tab, offsets, counts, pre_maps,
                       pre_words, seg_base, seg_stride, split);
  } else {
    pre_maps = nullptr;
  }
  auto launch = [&](auto inline_tag, auto counted_tag) {
    constexpr bool kInline = decltype(inline_tag)::value, kCounted = decltype(counted_tag)::value;
    auto held = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, block, held_lds, stream, tab, inl, ragged, offsets, idx, counts, seg_base, seg_stride,
                         map_words);
    };
    if (held_limit > 16 * kSelThreads) held(select_held_kernel<kInline, kSelMaxHeld>);
    else if (held_limit > 8 * kSelThreads) held(select_held_kernel<kInline, 16>);
    else if (held_limit > 0) held(select_held_kernel<kInline, 8>);
    if (longer > 0)
      hipLaunchKernelGGL((select_kernel<kInline, kCounted>), grid, block, lds, stream, tab, inl, ragged, offsets, idx, counts,
                         pre_maps, pre_words, seg_base, seg_stride, held_limit, bitmap_limit, (int)bitmap_stage_off);
  };
  if (host_offsets != nullptr) {
    if (counts != nullptr) launch(std::true_type{}, std::true_type{}); else launch(std::true_type{}, std::false_type{});
  } else {
    if (counts != nullptr) launch(std::false_type{}, std::true_type{}); else launch(std::false_type{}, std::false_type{});
  }
}

}  // namespace lkv
