// e^d for d <= 0 (-inf: 0, NaN: NaN) from a base-2 exponential: 2^(d log2 e), with what the product's rounding left out put back as a factor, so
// that it is as good for large -d as for small ones (with an exact 2^p off by 2^-23 of its value at most; without the factor by 33 times that at
// d = -87).  Below -87 the result is 0: no normal number.  No HIP header (constexpr: for host and device), so that it can be run where there is no GPU.
#pragma once

struct ExpParts {
  float x, left;   // the exponential is x + x * left * kExpLn2 (a sum of many may add x and x * left by themselves)
};
constexpr float kExpLn2 = 0.693147180559945f;

template <typename Exp2>
constexpr ExpParts exp_nonpositive_parts(float d, Exp2 exp2_of) {
  constexpr float kLog2e = 1.44269502162933349609f, kLog2eLow = 1.92596299e-8f;
  const float c = d < -87.f ? -200.f : d;   // 2^(-200 log2 e) is 0
  const float p = c * kLog2e;
  return ExpParts{exp2_of(p), __builtin_fmaf(c, kLog2eLow, __builtin_fmaf(c, kLog2e, -p))};
}
template <typename Exp2>
constexpr float exp_nonpositive(float d, Exp2 exp2_of) {
  const ExpParts e = exp_nonpositive_parts(d, exp2_of);
  return __builtin_fmaf(e.x, e.left * kExpLn2, e.x);
}
