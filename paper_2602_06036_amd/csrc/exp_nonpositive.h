// e^d for d <= 0 (-inf: 0, NaN: NaN) from a base-2 exponential: 2^(d log2 e), with what the product's rounding left out put back as a factor, so
// that it is as good for large -d as for small ones (with an exact 2^p off by 2^-23 of its value at most; without the factor by 33 times that at
// d = -87).  Below -87 the result is 0: no normal number.  No HIP header (constexpr: for host and device), so that it can be run where there is no GPU.
#pragma once

template <typename Exp2>
constexpr float exp_nonpositive(float d, Exp2 exp2_of) {
  constexpr float kLog2e = 1.44269502162933349609f, kLog2eLow = 1.92596299e-8f, kLn2 = 0.693147180559945f;
  const float p = d * kLog2e, left = __builtin_fmaf(d, kLog2eLow, __builtin_fmaf(d, kLog2e, -p)), x = exp2_of(p);
  return d < -87.f ? 0.f : __builtin_fmaf(x, left * kLn2, x);
}
