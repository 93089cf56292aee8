// LKV-H at inference time (Sec. 3.3) and the Soft-TopK operator ST_k (Sec. 3.2, Eq. 2, App. A.1;
// its backward pass, App. A.2, further down), in fp64: the ratios decide integer budgets floor(r t).
//
// ST_k(x)_i = f(x_i / tau - lambda), f the Laplace CDF, lambda such that the outputs sum to k.
// With m = #{i : z_i >= lambda}, z = x / tau, App. A.1 gives lambda in closed form from the sums over the head
// and the tail.  No sort is needed for them: taken relative to any trial threshold v,
//   A(v) = 1/2 sum_{z_i >= v} e^{v - z_i},   B(v) = 1/2 sum_{z_i < v} e^{z_i - v},   m(v) = #{z_i >= v}
// (every exponent is <= 0: nothing overflows however small tau is), g(v) = m - A + B - k has the sign of
// lambda - v, and the positive root y of A y^2 + (k - m) y - B = 0 gives the threshold v + log y that this split
// would have.  When no z_i lies between v and v + log y the split is the right one and that is lambda, in closed
// form; otherwise it is the next trial (a Newton step that knows the curvature), kept inside a bracket.
//
// One workgroup per vector.  What bounds it: instruction issue, one exponential per element and trial, so the
// trials are made where they are cheap: a histogram of the inputs finds the value of rank k to a bin's width, one to
// three trials on its bins (two exponentials per thread) come within a few hundredths of the threshold, one or two on fp32
// differences to that centre (one hardware exponential per element) find it to fp32
// accuracy, and only their end point is evaluated in fp64, where one pass both proves the split and yields the sums;
// the exponentials of that pass also give the outputs (e^{v - z} y = e^{lambda - z}).  A trial leaves the cube of its step as error
// (values crossed by the step count with the square of their distance), so a step under a hundredth is the last.
// The trials never pass the threshold (beyond a crossed value the closed form takes more than f does) but cross few
// values each where z is sparse, so they have to begin near rank k: where far values keep the histograms from getting
// there, the value of rank k is found exactly, from the bits.  (256 vectors of 16384, half of them masked with the
// type's lowest: 88 us, 1.5 ms by halving the bracket that such values stretch.)
// fp32 only chooses where fp64 looks: a poor choice costs further fp64 passes, never digits.  The trials on values are summed over
// the waves and told above from below in fp64 all the same (0.25 us): their bracket must not lose the threshold to rounding where
// a vector is long.
// Up to 32768 values the operands stay in registers between passes; longer vectors are read again in every pass
// (they stay in L2).  256 vectors of 16384 fp32 values: 25.5 us (257 us for the LDS sort and
// logarithmic scans this replaces), one vector of 131072: 0.13 ms (2.2 ms for halving a bracket in fp64).  Of the 25: read
// and extremes 4, histogram 2.5, trials 4, fp64 pass 7.5, root 0.7, outputs the rest.  Before that pass fetched its values ahead (7.5
// us, 8.3 with two at a time) and before the trials on bins, values kept in registers up to the trials and the sums over the waves taken
// side by side in the rows of 16 lanes: 30.4 us; 4096 values 15.7 -> 13.7, 8 vectors of 32768 42.6 -> 32.9, 777 values
// 9.2 as before (the call's own price).
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <type_traits>

#include "lkv_bracket.h"
#include "lkv_kernels.h"

namespace lkv {

namespace {

constexpr int kStThreads = 1024;          // workgroup of all but the shortest vectors
constexpr int kStSmallThreads = 256;      // vectors of up to 1024 values: fewer waves to reduce over
constexpr int kStMaxN = 1 << 22;
constexpr int kStLevels = 4;              // histograms at most (a cold temperature spreads the values over many units of z)
constexpr double kStWiden = 1.0 + 1e-6;   // bins this much wider than the span over their number: its upper end falls inside the last one
constexpr double kStEnough = 0.5;         // bin width, in z, from which the fp32 trials converge in two to four steps
constexpr double kStFar = 32.0;           // bin width, in z, up to which the trials still do without an exact start
constexpr int kStSearchSteps = 48;        // fp32 trials at most (bisection alone would need about 30)
constexpr int kStBinSteps = 6;            // trials on the bins at most
constexpr float kStBinsDone = 0.05f;      // step of a trial on bins from which the trials go on with the values
constexpr float kStDone = 0.01f;          // and the step that is the last: it ends within 1e-6 (777 to 131072 values, temperatures of .02 to 1)
constexpr int kStExactSteps = 200;        // fp64 trials at most (bisection alone would need about 60)
constexpr double kStCoarse = 1e15;         // |z| from which fp64 no longer resolves tenths of a unit
constexpr double kStMost = 1e300;         // centre of the search at most: its multiples do not overflow
constexpr double kStTinyProduct = 1e-250; // products of two sums below this have lost digits, or may have
constexpr double kStTiny = 1e-280;        // sums below this have lost (or may have lost) terms to underflow

// In a batched launch block b works on vector b: rows of x, y and info, and its own target sum, which the paper
// keeps strictly inside (0, n) (App. A.1, "Numerical Stability at Boundaries"); the same is enforced here by clamping.
template <typename X>
__device__ inline void select_vector(const X*& x, double*& y, double* __restrict__& info,
                                     double& k, const double* __restrict__ k_vec, int n) {
  if (k_vec == nullptr) return;
  const size_t b = blockIdx.x;
  x += b * n;
  if (y != nullptr) y += b * n;
  if (info != nullptr) info += 2 * b;
  k = fmin(fmax(k_vec[b], 1e-6), (double)n - 1e-6);
}

// ---- reductions over a block, result in every thread, operands combined in a fixed order ----
struct StAdd {
  template <typename V> __device__ __forceinline__ V operator()(V a, V b) const { return a + b; }
};
struct StMin {
  __device__ __forceinline__ float operator()(float a, float b) const { return fminf(a, b); }
  __device__ __forceinline__ double operator()(double a, double b) const { return fmin(a, b); }
};

struct StMax {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
  __device__ __forceinline__ double operator()(double a, double b) const { return fmax(a, b); }
};

template <int kCtrl, typename V>
__device__ __forceinline__ V st_dpp(V x) {
  if constexpr (sizeof(V) == 4) {
    return __builtin_bit_cast(V, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), kCtrl, 0xf, 0xf, true));
  } else {
    const long long u = __builtin_bit_cast(long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, kCtrl, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), kCtrl, 0xf, 0xf, true);
    return __builtin_bit_cast(V, (long long)(((unsigned long long)hi << 32) | lo));
  }
}

// over the 16 lanes of a DPP row
template <typename V, typename Op>
__device__ __forceinline__ V st_row16(V x, Op op) {
  x = op(x, st_dpp<kDppQuadXor1>(x));
  x = op(x, st_dpp<kDppQuadXor2>(x));
  x = op(x, st_dpp<kDppRowHalfMirror>(x));
  return op(x, st_dpp<kDppRowMirror>(x));
}

// x of this lane's row of 16 and of the row beside it (kRows = 16), or of both halves of the wave (32), in either order:
// swaps on the vector ALU, where a shuffle waits for the LDS crossbar
template <int kRows, typename V, typename Op>
__device__ __forceinline__ V st_join(V x, Op op) {
  auto swapped = [](unsigned u) {
    if constexpr (kRows == 16) return __builtin_amdgcn_permlane16_swap(u, u, false, false);
    else return __builtin_amdgcn_permlane32_swap(u, u, false, false);
  };
  if constexpr (sizeof(V) == 4) {
    const u32x2_swap_t a = swapped(__builtin_bit_cast(unsigned, x));
    return op(__builtin_bit_cast(V, (unsigned)a.x), __builtin_bit_cast(V, (unsigned)a.y));
  } else {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const u32x2_swap_t lo = swapped((unsigned)u), hi = swapped((unsigned)(u >> 32));
    return op(__builtin_bit_cast(V, ((unsigned long long)hi.x << 32) | lo.x),
              __builtin_bit_cast(V, ((unsigned long long)hi.y << 32) | lo.y));
  }
}
// over the wave: the rows, then the four rows
template <typename V, typename Op>
__device__ __forceinline__ V st_wave(V x, Op op) {
  return st_join<32>(st_join<16>(st_row16(x, op), op), op);
}

// inclusive prefix sum over the wave: four shifts within the rows of 16 lanes, then the last lane of a row joins those after
template <int kCtrl, int kRows>
__device__ __forceinline__ unsigned st_dpp_add(unsigned x) {
  return x + (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, kRows, 0xf, true);
}
__device__ __forceinline__ unsigned st_scan(unsigned x) {
  x = st_dpp_add<0x111, 0xf>(x);   // row_shr:1, 2, 4, 8 (zeros move in)
  x = st_dpp_add<0x112, 0xf>(x);
  x = st_dpp_add<0x114, 0xf>(x);
  x = st_dpp_add<0x118, 0xf>(x);
  x = st_dpp_add<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
  return st_dpp_add<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
}

// Per-wave results of up to five values; two copies used in turn, so that one barrier per reduction is enough (a wave
// that writes a copy again has passed the barrier after every wave's reads of it).
struct StScratch {
  double v[2][5][16];
  float f[2][3][16];
};

// a value that is the same in every lane, moved to scalar registers (the vector ones are needed for the elements)
__device__ __forceinline__ double st_uniform(double x) {
  const long long u = __builtin_bit_cast(long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(u >> 32));
  return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}

template <int kT>
struct StHist {
  static constexpr int kBins = 2 * kT;
  unsigned bin[kBins];
  unsigned wave_total[kT / 64];
  double above;
  int found;
};

template <int kT, typename Op>
__device__ __forceinline__ double st_collect(const double (&slot)[16], double identity, Op op) {
  const int l = threadIdx.x & 15;
  return st_uniform(st_row16(l < kT / 64 ? slot[l] : identity, op));
}

// The same for up to four sums (minima) at once, one to a row of 16 lanes: result i from lane 16 i.
template <int kT, int kN, typename V, typename Op>
__device__ __forceinline__ V st_collect_rows(const V (*slots)[16], V identity, Op op) {
  const int l = threadIdx.x & 15, r = (threadIdx.x & 63) >> 4;
  return st_row16(l < kT / 64 && r < kN ? slots[r][l] : identity, op);
}
__device__ __forceinline__ double st_lane(double x, int lane) {
  const long long u = __builtin_bit_cast(long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(u >> 32), lane);
  return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ float st_lane(float x, int lane) {
  return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane));
}

// keys whose unsigned order is the numeric order of the values
__device__ __forceinline__ uint32_t st_key(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u >> 31) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ uint64_t st_key(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ float st_value(uint32_t k) { return __uint_as_float((k >> 31) ? (k & 0x7fffffffu) : ~k); }
__device__ __forceinline__ double st_value(uint64_t k) {
  return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}

// x / tau, correctly rounded: one multiplication and a residual correction where x came from fp32 and tau is moderate
// (nothing overflows or loses bits there) and x finite, else the division itself
template <typename X>
__device__ __forceinline__ double st_quotient(X x, double tau, double rtau, bool moderate) {
  const double xd = (double)x;
  if constexpr (sizeof(X) == 4) {
    if (moderate) {
      const double q = xd * rtau;
      return fma(fma(-q, tau, xd), rtau, q);
    }
  }
  return xd / tau;
}

// kE > 0: thread t holds elements t, t + kT, ... (kE of them, n <= kE kT) in registers; kE = 0: any n, re-read in
// every pass.
template <typename X, int kT, int kE>
__global__ void __launch_bounds__(kT)
soft_topk_kernel(const X* x, int n, double k, double tau, double* y /* may alias x */, double* __restrict__ info,
                 int32_t* __restrict__ budgets, double t, const double* __restrict__ k_vec) {
  constexpr bool kHeld = kE > 0;
  constexpr int kR = kHeld ? kE : 1;
  constexpr bool kKeep = kHeld && kE * (int)sizeof(X) <= 32;   // the inputs stay in registers to the end (16 fp32 ones beside the exponentials: spills, 2.4 us slower)
  constexpr double kLog2E = 1.44269504088896340736, kLn2 = 0.693147180559945309417;
  __shared__ StScratch sh;
  __shared__ StHist<kT> hist;
  select_vector(x, y, info, k, k_vec, n);   // batched call: this block's vector and target
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const bool writer = (tid & 63) == 0;
  int turn = 0;
  k = st_uniform(k);
  const double rtau = st_uniform(1.0 / tau);
  bool moderate = tau > 1e-100 && tau < 1e100;

  // ---- where to look: the value of rank k, by histograms of the inputs that narrow to one bin ----
  double lo, hi, zc;   // bracket of the threshold; centre of the search
  int found_bin;       // of the histogram over all values, zc its centre; -1: there is none
  float bin_step = 0.f;   // its width in the units of the search
  X xr[kR];
  {
    if constexpr (kHeld) {
#pragma unroll
      for (int e = 0; e < kR; ++e) xr[e] = x[min(tid + e * kT, n - 1)];   // padding repeats the last value
    }
    for (int i = tid; i < StHist<kT>::kBins; i += kT) hist.bin[i] = 0;
    if (tid == 0) hist.found = -1;
    double least = INFINITY, most = INFINITY;   // min x, min -x
    {
      X small = (X)INFINITY, large = (X)-INFINITY;
      if constexpr (kHeld) {
#pragma unroll
        for (int e = 0; e < kR; ++e) { small = xr[e] < small ? xr[e] : small; large = xr[e] > large ? xr[e] : large; }
      } else {
#pragma unroll 4
        for (int i = tid; i < n; i += kT) { small = x[i] < small ? x[i] : small; large = x[i] > large ? x[i] : large; }
      }
      least = (double)st_wave(small, StMin());
      most = -(double)st_wave(large, StMax());
    }
    auto& v = sh.v[turn];
    if (writer) { v[0][wave] = least; v[1][wave] = most; }
    __syncthreads();
    const double ends = st_collect_rows<kT, 2>(v, (double)INFINITY, StMin());
    least = st_lane(ends, 0);
    most = -st_lane(ends, 16);
    turn ^= 1;
    // g > 0 at lo: every f is at least 1 - e^{-L} / 2 with L >= 1 + log(n / (2 (n - k))), so the sum exceeds
    // n - (n - k) / e > k; g < 0 at hi: every f is at most e^{-U} / 2 with U >= 1 + log(n / (2 k)): sum <= k / e
    // (both in one go: the first row of lanes has least and n - k, the second -most and k)
    moderate = moderate && least > -INFINITY && most < INFINITY;
    const double bound = ends / tau - bracket_margin(n, (tid & 16) == 0 ? (double)n - k : k, [](float x) { return __log2f(x); });
    lo = st_lane(bound, 0);
    hi = -st_lane(bound, 16);
    constexpr int kBins = StHist<kT>::kBins;
    double above = 0.0;   // values in higher bins
    auto for_each = [&](auto visit) {
      if constexpr (kHeld) {
#pragma unroll
        for (int e = 0; e < kR; ++e) visit(xr[e], tid + e * kT < n);
      } else {
#pragma unroll 4
        for (int i = tid; i < n; i += kT) visit(x[i], true);
      }
    };
    auto clear = [&]() {
      __syncthreads();
      for (int i = tid; i < kBins; i += kT) hist.bin[i] = 0;
      if (tid == 0) hist.found = -1;
      __syncthreads();
    };
    // the bin with the value of rank k from the top, or -1; advances `above`
    auto find_bin = [&]() {
      __syncthreads();
      // from the top: thread t owns bins kBins - 1 - 2 t and kBins - 2 - 2 t
      const int top = kBins - 1 - 2 * tid;
      const unsigned c0 = hist.bin[top], c1 = hist.bin[top - 1];
      const unsigned incl = st_scan(c0 + c1);
      if ((tid & 63) == 63) hist.wave_total[wave] = incl;
      __syncthreads();
      const int l = tid & 15;
      const unsigned before = st_row16(l < wave && l < kT / 64 ? hist.wave_total[l] : 0u, StAdd());
      const double e0 = above + (double)(before + incl - c0 - c1);
      if (c0 != 0 && e0 < k && k <= e0 + c0) { hist.found = top; hist.above = e0; }
      if (c1 != 0 && e0 + c0 < k && k <= e0 + c0 + c1) { hist.found = top - 1; hist.above = e0 + c0; }
      __syncthreads();
      const int found = __builtin_amdgcn_readfirstlane(hist.found);
      if (found >= 0) above = st_uniform(hist.above);
      return found;
    };
    double base = least, span = most - least;
    bool looking = span > 0.0 && span < INFINITY;
    found_bin = -1;
    for (int level = 0; level < kStLevels && looking; ++level) {
      if (level > 0) {
        clear();
        found_bin = -1;
      }
      const double width = st_uniform(span * (kStWiden / (double)kBins));
      const float to_bin = 1.f / (float)width;
      auto bin_of = [&](float f) { return (int)fminf(fmaxf(f, 0.f), (float)(kBins - 1)); };
      if (level == 0) {   // every value
        for_each([&](X xv, bool in) {
          if (in) atomicAdd(&hist.bin[bin_of((float)(xv - (X)base) * to_bin)], 1u);
        });
      } else {            // the values of the bin found before
        for_each([&](X xv, bool in) {
          const float f = (float)(xv - (X)base) * to_bin;
          if (in && f >= 0.f && f < (float)kBins) atomicAdd(&hist.bin[bin_of(f)], 1u);
        });
      }
      const int found = find_bin();
      if (found < 0) break;   // rounding moved a value across the bin's edge
      if (level == 0) found_bin = found;
      span = width;
      base = st_uniform(base + found * span);
      looking = span > kStEnough * tau && base + span > base;
    }
    if (__builtin_expect(span <= kStFar * tau, 1)) {
      zc = st_uniform((base + 0.5 * span) / tau);
      if (found_bin >= 0) bin_step = (float)st_uniform(span * rtau * kLog2E);
    } else {
      // Values so far apart (masked with the type's lowest, or infinite) that equal steps do not come down to the rest
      // of them: the value of rank k itself, digit by digit of its ordered bits.
      found_bin = -1;
      using Key = decltype(st_key(X()));
      constexpr int kDigit = kT == 1024 ? 11 : 9;
      static_assert(1 << kDigit == kBins, "a digit per bin");
      Key key = 0;
      above = 0.0;
#pragma unroll 1
      for (int left = 8 * (int)sizeof(Key); left > 0;) {   // bits of the key not yet known
        const int shift = left > kDigit ? left - kDigit : 0;
        clear();
#pragma unroll 4
        for (int i = tid; i < n; i += kT) {
          const Key own = st_key(x[i]);
          if (left == 8 * (int)sizeof(Key) || (own ^ key) >> left == 0)   // agrees in the bits known
            atomicAdd(&hist.bin[(own >> shift) & (Key)((1 << (left - shift)) - 1)], 1u);
        }
        key |= (Key)max(find_bin(), 0) << shift;
        left = shift;
      }
      zc = st_uniform((double)st_value(key) / tau);
    }
    zc = st_uniform(fmin(fmax(zc, -kStMost), kStMost));   // an infinite value of rank k: any threshold beyond the others
    if (!(zc >= lo && zc <= hi)) {
      zc = st_uniform(0.5 * (lo + hi));
      found_bin = -1;
    }
  }

  // ---- search in fp32: w = (z - zc) log2 e ----
  double v;
  {
    const double scale = st_uniform(rtau * kLog2E), shift = st_uniform(-zc * kLog2E);
    float w[kR];
    if constexpr (kHeld) {
#pragma unroll
      for (int e = 0; e < kR; ++e)   // the vector is in the caches by now; padding lies infinitely far down the tail
        w[e] = tid + e * kT < n ? (float)fma((double)xr[e], scale, shift) : -INFINITY;
    }
    float flo = (float)((lo - zc) * kLog2E), fhi = (float)((hi - zc) * kLog2E), fv = 0.f;
    // nothing to search for at a centre that itself rounds to about a unit
    const int n_search = fabs(zc) < kStCoarse ? kStSearchSteps : 0;
    // the threshold that a trial's split would have: d = k - m, af = 2 A, bf = 2 B.  Only a place for the next trial: the hardware's
    // root and reciprocal will do (IEEE ones: 0.5 us)
    auto step_to = [&](float df, float af, float bf) {
      const float root = __builtin_amdgcn_sqrtf(fmaf(df, df, af * bf));
      return fv + __log2f(df >= 0.f ? bf * __builtin_amdgcn_rcpf(df + root) : (root - df) * __builtin_amdgcn_rcpf(af));
    };
    // trials on the bins first, each as many values in its middle, and split where the trial cuts it: in fp32, since the bins
    // are no better
    float c0 = 0.f, c1 = 0.f, w0 = 0.f, w1 = 0.f, per_step = 0.f;
    bool on_bins = found_bin >= 0 && bin_step > 0.f;
    if (on_bins) {
      c0 = (float)hist.bin[2 * tid];
      c1 = (float)hist.bin[2 * tid + 1];
      w0 = (float)(2 * tid - found_bin) * bin_step;
      w1 = (float)(2 * tid + 1 - found_bin) * bin_step;
      per_step = 1.f / bin_step;
    }
#pragma unroll 1
    for (int step = 0; step < n_search; ++step) {
      float head = 0.f, all = 0.f, cnt = 0.f;
      if (on_bins) {   // uniform
        auto visit = [&](float wv, float c) {
          const float d = wv - fv;
          const float e = c * __builtin_amdgcn_exp2f(-fabsf(d));
          const float up = fminf(fmaxf(fmaf(d, per_step, 0.5f), 0.f), 1.f);
          all += e;
          head = fmaf(up, e, head);
          cnt = fmaf(up, c, cnt);
        };
        visit(w0, c0);
        visit(w1, c1);
      } else {
        int n_up = 0;
        auto visit = [&](float wv) {
          const float d = wv - fv;
          const float e = __builtin_amdgcn_exp2f(-fabsf(d));
          const bool up = d >= 0.f;
          all += e;
          head += up ? e : 0.f;
          n_up += up ? 1 : 0;
        };
        if constexpr (kHeld) {
#pragma unroll
          for (int e = 0; e < kR; ++e) visit(w[e]);
        } else {
#pragma unroll 4
          for (int i = tid; i < n; i += kT) visit((float)fma((double)x[i], scale, shift));
        }
        cnt = (float)n_up;
      }
      head = st_wave(head, StAdd());
      all = st_wave(all, StAdd());
      cnt = st_wave(cnt, StAdd());   // exact: whole numbers up to 2^22
      if (on_bins) {
        auto& sf = sh.f[turn];
        if (writer) { sf[0][wave] = head; sf[1][wave] = all; sf[2][wave] = cnt; }
        __syncthreads();
        const float sums = st_collect_rows<kT, 3>(sf, 0.f, StAdd());
        const float af = st_lane(sums, 0);
        turn ^= 1;
        const float next = step_to((float)(k - (double)st_lane(sums, 32)), af, fmaxf(st_lane(sums, 16) - af, 0.f));
        const bool usable = next > flo && next < fhi;
        on_bins = usable && fabsf(next - fv) >= kStBinsDone && step < kStBinSteps;
        if (usable) fv = next;
        continue;
      }
      // the sums over the waves and the side of the trial in fp64
      auto& sv = sh.v[turn];
      if (writer) { sv[0][wave] = head; sv[1][wave] = all; sv[2][wave] = cnt; }
      __syncthreads();
      const double sums = st_collect_rows<kT, 3>(sv, 0.0, StAdd());
      const double a2 = st_lane(sums, 0), b2 = st_lane(sums, 16) - a2;   // 2 A, 2 B
      turn ^= 1;
      const double d = k - st_lane(sums, 32);
      float next = step_to((float)d, (float)a2, (float)fmax(b2, 0.0));
      if (0.5 * (b2 - a2) - d > 0.0) flo = fv; else fhi = fv;   // the threshold lies above, or below, this trial
      if (fabsf(next - fv) < kStDone) {   // an error of its cube is left, below what fp32 resolves
        fv = next;
        break;
      }
      if (d == 0.0 && !(next > flo && next < fhi)) break;   // k values above, and all of them far away: a gap, left to fp64
      if (!(next > flo && next < fhi)) next = 0.5f * (flo + fhi);
      if (!(next > flo && next < fhi)) break;   // down to neighbouring numbers
      fv = next;
    }
    v = fma((double)fv, kLn2, zc);
    if (!(v >= lo && v <= hi)) v = 0.5 * (lo + hi);
    v = st_uniform(v);
  }

  // ---- fp64: prove the split, take the sums ----
  double ex[kR];           // e^{-|z - v|}, negative (or -0) in the tail
  double lambda = v, factor = 1.0;
  int m = 0;
  bool from_held = false;  // the outputs can be formed from ex and factor = e^{lambda - v}
  double blo = lo, bhi = hi;
#pragma unroll 1
  for (int step = 0; step < kStExactSteps; ++step) {
    double a = 0.0, b = 0.0, up = INFINITY, dn = INFINITY;
    int cnt = 0;
    auto visit = [&](double z) {
      const double d = z - v;
      const double e = exp(-fabs(d));
      const bool head = d >= 0.0;
      a += head ? e : 0.0;
      b += head ? 0.0 : e;
      up = fmin(up, head ? d : INFINITY);
      dn = fmin(dn, head ? INFINITY : -d);
      cnt += head ? 1 : 0;
      return head ? e : -e;
    };
    if constexpr (kHeld) {
      int first = tid;
      asm volatile("" : "+v"(first));   // or the compiler keeps indices and quotients from step to step, in scratch memory
      X ahead[kR];
      if constexpr (!kKeep) {
#pragma unroll
        for (int e = 0; e < kR; ++e) ahead[e] = x[min(first + e * kT, n - 1)];
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int e = 0; e < kR; ++e) {
        const int i = first + e * kT;
        const double z = st_quotient(kKeep ? xr[e] : ahead[e], tau, rtau, moderate);
        ex[e] = visit(i < n ? z : -INFINITY);
        if (e & 1) __builtin_amdgcn_sched_barrier(0);   // two exponentials at a time fit the registers
      }
    } else {
#pragma unroll 2
      for (int i = tid; i < n; i += kT) visit(st_quotient(x[i], tau, rtau, moderate));
    }
    a = st_wave(a, StAdd());
    b = st_wave(b, StAdd());
    up = st_wave(up, StMin());
    dn = st_wave(dn, StMin());
    cnt = st_wave(cnt, StAdd());
    auto& sv = sh.v[turn];
    if (writer) { sv[0][wave] = a; sv[1][wave] = b; sv[2][wave] = cnt; sv[3][wave] = up; sv[4][wave] = dn; }
    __syncthreads();
    const double sums = st_collect_rows<kT, 3>(sv, 0.0, StAdd());
    const double gaps = st_collect_rows<kT, 2>(sv + 3, (double)INFINITY, StMin());
    a = 0.5 * st_lane(sums, 0);
    b = 0.5 * st_lane(sums, 16);
    m = (int)st_lane(sums, 32);
    up = st_lane(gaps, 0);
    dn = st_lane(gaps, 16);
    turn ^= 1;
    const double d = k - (double)m;
    double delta;
    if (d == 0.0 && m > 0 && m < n && fmin(a, b) < kStTiny) {
      // A whole target in a gap so wide that the sums underflow: both again, each relative to its own largest term
      double sa = 0.0, sb = 0.0;
      for (int i = tid; i < n; i += kT) {
        const double dz = st_quotient(x[i], tau, rtau, moderate) - v;
        if (dz >= 0.0) sa += exp(up - dz);
        else sb += exp(dn + dz);
      }
      sa = st_wave(sa, StAdd());
      sb = st_wave(sb, StAdd());
      auto& su = sh.v[turn];
      if (writer) { su[0][wave] = sa; su[1][wave] = sb; }
      __syncthreads();
      sa = st_collect<kT>(su[0], 0.0, StAdd());
      sb = st_collect<kT>(su[1], 0.0, StAdd());
      turn ^= 1;
      // (a head or a tail of infinite values only: far enough that the other side's f round to 1 or 0)
      delta = dn == INFINITY ? -746.0 : up == INFINITY ? 746.0 : 0.5 * ((up - dn) + log(sb) - log(sa));
      factor = exp(delta);   // used for the outputs below only where the trial lies near the middle of the gap
    } else {
      // the root without a difference of close numbers; a = 0 (empty head) and b = 0 (empty tail) come out as they should
      const double ab = a * b;
      const double root = ab > kStTinyProduct ? sqrt(fma(d, d, 4.0 * ab)) : hypot(d, 2.0 * sqrt(a) * sqrt(b));
      factor = d >= 0.0 ? 2.0 * b / (d + root) : (root - d) / (2.0 * a);
      delta = log(factor);
    }
    delta = st_uniform(delta);
    factor = st_uniform(factor);
    lambda = v + delta;
    // the split holds when no value lies between v and lambda (values at lambda belong to the head)
    // or the step is lost in rounding v (values beyond 2^53 units of z that tie with the threshold); NaN among the inputs
    // makes every output NaN
    if ((delta >= 0.0 ? delta <= up : -delta < dn) || lambda == v || lambda != lambda) {
      from_held = kHeld && fabs(delta) < 100.0;
      break;
    }
    if ((double)m - k + (b - a) > 0.0) blo = v; else bhi = v;
    double next = lambda;
    if (!(next > blo && next < bhi)) next = 0.5 * (blo + bhi);
    next = st_uniform(next);
    lambda = v;
    if (!(next > blo && next < bhi)) break;   // down to neighbouring numbers: what is inside ties with the root
    v = next;
  }
  if (tid == 0 && info != nullptr) {
    info[0] = lambda;
    info[1] = (double)m;
  }
  auto put = [&](int i, double r) {
    if (y != nullptr) y[i] = r;
    if (budgets != nullptr) budgets[i] = (int32_t)floor(r * t);
  };
  if constexpr (kHeld) {
    if (from_held) {
      const double down = 1.0 / factor;
      int first = tid;
      asm volatile("" : "+v"(first));
#pragma unroll
      for (int e = 0; e < kR; ++e) {
        const bool tail = __double_as_longlong(ex[e]) < 0;
        if (first + e * kT < n) put(first + e * kT, tail ? -0.5 * ex[e] * down : fma(-0.5 * factor, ex[e], 1.0));
      }
      return;
    }
  }
#pragma unroll 2
  for (int i = tid; i < n; i += kT) {
    const double z = st_quotient(x[i], tau, rtau, moderate) - lambda;
    const double half = 0.5 * exp(-fabs(z));
    put(i, z >= 0.0 ? 1.0 - half : half);
  }
}

// Backward of ST_k (App. A.2).  With z_i = x_i / tau - lambda and f'(z) = e^{-|z|} / 2 the implicit
// function theorem gives d lambda / d x_j = f'(z_j) / sum_i f'(z_i) = w_j and d lambda / d k =
// -1 / sum_i f'(z_i), hence for an upstream gradient g = dL/dy
//   dL/dx_j = (f'(z_j) / tau) (g_j - gbar),   dL/dk = gbar = sum_i g_i w_i.
// One workgroup per vector; lambda is read from the forward call's `info`.  One pass takes the exponentials, the two
// sums and the smallest |z|; up to 16384 values the exponentials and g stay in registers for the output, longer
// vectors are read a second time.  Only when the sums underflow (a temperature so cold that every f'(z) does) are
// they taken again relative to the smallest |z|, which still yields the ratios.  Sums in a fixed order.  256 vectors
// of 16384 fp32 values: 18.5 us (34.5 us with three passes over x and two over g); the bytes alone take 14 us.
template <typename X, int kT, int kE>
__global__ void __launch_bounds__(kT)
soft_topk_backward_kernel(const X* __restrict__ x, int n, double tau, const double* __restrict__ info,
                          const double* g, double* dx /* may alias g */, double* __restrict__ dk) {
  constexpr bool kHeld = kE > 0;
  constexpr int kR = kHeld ? kE : 1;
  __shared__ StScratch sh;
  {   // one vector per block
    const size_t b = blockIdx.x;
    x += b * n;
    g += b * n;
    dx += b * n;
    info += 2 * b;
    if (dk != nullptr) dk += b;
  }
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const bool writer = (tid & 63) == 0;
  const double lambda = info[0];
  const double rtau = 1.0 / tau;
  const bool moderate = tau > 1e-100 && tau < 1e100;
  auto distance = [&](X xv) {
    // an infinite (masked) value counts as the type's largest: the quotient's correction would make it NaN
    if constexpr (sizeof(X) == 4) xv = __builtin_amdgcn_fmed3f(xv, -FLT_MAX, FLT_MAX);
    return fabs(st_quotient(xv, tau, rtau, moderate) - lambda);
  };

  double ex[kR], gr[kR];
  double amin = INFINITY, s = 0.0, sg = 0.0;
  if constexpr (kHeld) {
    X xr[kR];
#pragma unroll
    for (int e = 0; e < kR; ++e) {
      xr[e] = x[min(tid + e * kT, n - 1)];
      gr[e] = g[min(tid + e * kT, n - 1)];
    }
#pragma unroll
    for (int e = 0; e < kR; ++e) {
      const double a = distance(xr[e]);
      amin = fmin(amin, a);   // padding repeats the last value
      ex[e] = tid + e * kT < n ? exp(-a) : 0.0;
      s += ex[e];
      sg = fma(gr[e], ex[e], sg);
    }
  } else {
#pragma unroll 2
    for (int i = tid; i < n; i += kT) {
      const double a = distance(x[i]);
      const double e = exp(-a);
      amin = fmin(amin, a);
      s += e;
      sg = fma(g[i], e, sg);
    }
  }
  amin = st_wave(amin, StMin());
  s = st_wave(s, StAdd());
  sg = st_wave(sg, StAdd());
  if (writer) { sh.v[0][0][wave] = amin; sh.v[0][1][wave] = s; sh.v[0][2][wave] = sg; }
  __syncthreads();
  amin = st_collect<kT>(sh.v[0][0], INFINITY, StMin());
  s = st_collect<kT>(sh.v[0][1], 0.0, StAdd());
  sg = st_collect<kT>(sh.v[0][2], 0.0, StAdd());
  if (s < kStTiny) {   // the same in every thread
    s = 0.0;
    sg = 0.0;
    for (int i = tid; i < n; i += kT) {
      const double e = exp(amin - distance(x[i]));
      s += e;
      sg = fma(g[i], e, sg);
    }
    s = st_wave(s, StAdd());
    sg = st_wave(sg, StAdd());
    if (writer) { sh.v[1][0][wave] = s; sh.v[1][1][wave] = sg; }
    __syncthreads();
    s = st_collect<kT>(sh.v[1][0], 0.0, StAdd());
    sg = st_collect<kT>(sh.v[1][1], 0.0, StAdd());
  }
  const double gbar = sg / s;
  if (tid == 0 && dk != nullptr) dk[0] = gbar;
  if constexpr (kHeld) {
#pragma unroll
    for (int e = 0; e < kR; ++e)
      if (tid + e * kT < n) dx[tid + e * kT] = 0.5 * ex[e] * (gr[e] - gbar) * rtau;
  } else {
#pragma unroll 2
    for (int i = tid; i < n; i += kT) dx[i] = 0.5 * exp(-distance(x[i])) * (g[i] - gbar) * rtau;
  }
}

// s = w2 . SiLU(W1 e + b1) (+ b2) for one head per block
__global__ void __launch_bounds__(256)
head_scores_kernel(const float* __restrict__ emb, const float* __restrict__ w1, const float* __restrict__ b1,
                   const float* __restrict__ w2, const float* __restrict__ b2, int d_e, int hidden,
                   double* __restrict__ s) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* part = reinterpret_cast<double*>(smem);   // [hidden]
  const float* e = emb + (size_t)blockIdx.x * d_e;
  for (int j = threadIdx.x; j < hidden; j += blockDim.x) {
    const float* w = w1 + (size_t)j * d_e;
    double z = 0.0;
    for (int q = 0; q < d_e; ++q) z = fma((double)w[q], (double)e[q], z);
    z += (double)b1[j];
    part[j] = (double)w2[j] * (z / (1.0 + exp(-z)));
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double acc = 0.0;
    for (int j = 0; j < hidden; ++j) acc += part[j];
    if (b2 != nullptr) acc += (double)b2[0];
    s[blockIdx.x] = acc;
  }
}

// Which kernel takes a vector of n values: the smallest that holds it in registers (fewer elements per thread, shorter
// passes), one that re-reads it beyond that.  f(tag of the threads, tag of the elements per thread).
template <int kMaxHeld, typename F>
void soft_topk_dispatch(int n, F f) {
  if (n <= 4 * kStSmallThreads) f(std::integral_constant<int, kStSmallThreads>(), std::integral_constant<int, 4>());
  else if (n <= 4 * kStThreads) f(std::integral_constant<int, kStThreads>(), std::integral_constant<int, 4>());
  else if (n <= 16 * kStThreads) f(std::integral_constant<int, kStThreads>(), std::integral_constant<int, 16>());
  else if (n <= kMaxHeld * kStThreads) f(std::integral_constant<int, kStThreads>(), std::integral_constant<int, kMaxHeld>());
  else f(std::integral_constant<int, kStThreads>(), std::integral_constant<int, 0>());
}

template <typename X>
void launch_soft_topk_as(const X* x, int n, double k, double tau, double* y, double* info, int32_t* budgets, double t,
                         hipStream_t stream, int n_vec, const double* k_vec) {
  soft_topk_dispatch<32>(n, [&](auto threads, auto held) {
    hipLaunchKernelGGL((soft_topk_kernel<X, decltype(threads)::value, decltype(held)::value>), dim3(n_vec),
                       dim3(decltype(threads)::value), 0, stream, x, n, k, tau, y, info, budgets, t, k_vec);
  });
}

template <typename X>
void launch_soft_topk_backward_as(const X* x, int n, double tau, const double* info, const double* g, double* dx,
                                  double* dk, hipStream_t stream, int n_vec) {
  soft_topk_dispatch<16>(n, [&](auto threads, auto held) {
    hipLaunchKernelGGL((soft_topk_backward_kernel<X, decltype(threads)::value, decltype(held)::value>), dim3(n_vec),
                       dim3(decltype(threads)::value), 0, stream, x, n, tau, info, g, dx, dk);
  });
}

}  // namespace

int soft_topk_max_n(bool) { return kStMaxN; }
int head_scores_max_hidden() { return 4096; }

// y, info and budgets may each be null; y may alias x when x is fp64.  k_vec != nullptr: n_vec vectors of n values,
// one block each, targets read from the device.
void launch_soft_topk(const void* x, bool is_f64, int n, double k, double tau, double* y, double* info,
                      int32_t* budgets, double t, hipStream_t stream, int n_vec, const double* k_vec) {
  if (is_f64) launch_soft_topk_as(static_cast<const double*>(x), n, k, tau, y, info, budgets, t, stream, n_vec, k_vec);
  else launch_soft_topk_as(static_cast<const float*>(x), n, k, tau, y, info, budgets, t, stream, n_vec, k_vec);
}

void launch_soft_topk_backward(const void* x, bool is_f64, int n, double tau, const double* info, const double* g,
                               double* dx, double* dk, hipStream_t stream, int n_vec) {
  if (is_f64) launch_soft_topk_backward_as(static_cast<const double*>(x), n, tau, info, g, dx, dk, stream, n_vec);
  else launch_soft_topk_backward_as(static_cast<const float*>(x), n, tau, info, g, dx, dk, stream, n_vec);
}

void launch_head_scores(const float* emb, const float* w1, const float* b1, const float* w2, const float* b2,
                        int n_heads, int d_e, int hidden, double* s, hipStream_t stream) {
  hipLaunchKernelGGL(head_scores_kernel, dim3(n_heads), dim3(256), (size_t)hidden * sizeof(double), stream, emb, w1,
                     b1, w2, b2, d_e, hidden, s);
}

}  // namespace lkv
