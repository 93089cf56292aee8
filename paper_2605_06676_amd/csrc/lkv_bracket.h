// Bracket of the Soft-TopK threshold (plain C++).
#pragma once
#include <cstdint>

namespace lkv {

// How far below the least (above the greatest) value the threshold of a target sum can lie: at least 1 + log(n / (2 part)) and at
// least 1, where `part` is n - k (k).  The logarithms are taken in fp32, and a thousandth is added for their rounding; part's
// exponent is taken off before, so that the margin is finite for every part > 0 that fp64 holds.
template <typename Log2>   // float -> float, for arguments in [1, 2^31]
constexpr double bracket_margin(int n, double part, Log2 log2) {
  int exponent = 0;
  if (part < 2.2250738585072014e-308) {   // subnormal
    part *= 18014398509481984.0;          // 2^54
    exponent = -54;
  }
  const uint64_t bits = __builtin_bit_cast(uint64_t, part);
  exponent += (int)(bits >> 52) - 1023;
  const double mantissa = __builtin_bit_cast(double, (bits & 0xfffffffffffffull) | 0x3ff0000000000000ull);
  const float orders = log2((float)n) - 1.f - log2((float)mantissa) - (float)exponent;
  return 1.001 + (orders > 0.f ? (double)(0.693147181f * orders) : 0.0);
}

}  // namespace lkv
