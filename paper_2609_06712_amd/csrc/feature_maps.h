// Branch-free GELU and tanh of the bf16 low-rank kernels. The including file defines MAP_FN (function
// qualifiers), MAP_RCP and MAP_EXP (reciprocal and exponential), so that a host build can check the fits.
//
// Both polynomials are minimax fits in the relative error, which alternates between equal extremes over the
// interval (Chebyshev's criterion: +-1.43e-8 ten times for GELU, +-2.6 to 2.9e-9 for tanh), coefficients rounded
// to fp32. What they replace (erff, tanhf) took a divergent branch per value. On the kernels' own values the fp32 features
// are as far from 64 bits as with those: relative 2-norm 8.2e-8 against 8.1e-8 (GELU), 5.0e-8 against 4.9e-8
// (tanh), projections of unit variance; 6.7e-8 / 6.8e-8 and 4.9e-8 / 4.8e-8 at three times that.
#pragma once

namespace rola {

// GELU x Phi(x) from erfc(z) = t P(t) exp(-z^2), z = |x| / sqrt 2, t = 1 / (1 + 0.4 z): P is of degree 8,
// fitted on z in [0, 5] (relative error 1.5e-8; 7e-7 at z = 6 and 1.5e-5 at 9, where the tail is below 1e-17
// of anything it is added to). In fp32 the lower tail, where 1 + erf cancels, is accurate to
// (16 + 3 z^2) 2^-24: the rounding of z^2 is what the exponential magnifies.
MAP_FN float gelu_fast(float x) {
  const float z = fabsf(x) * 0.70710678118654752f;
  const float t = MAP_RCP(fmaf(0.4f, z, 1.0f));
  float p = 0.02058017541f;
  p = fmaf(p, t, -0.0333637342f);
  p = fmaf(p, t, -0.1531883735f);
  p = fmaf(p, t, 0.3820583653f);
  p = fmaf(p, t, -0.143041639f);
  p = fmaf(p, t, 0.2988953582f);
  p = fmaf(p, t, 0.1714113825f);
  p = fmaf(p, t, 0.2313518033f);
  p = fmaf(p, t, 0.2252966763f);
  const float tail = 0.5f * t * p * MAP_EXP(-z * z);  // 1 - Phi(|x|)
  return x * (x >= 0.f ? 1.0f - tail : tail);
}

// tanh: x + x^3 Q(x^2) (degree 4, 3e-9 relative) up to 0.6, 1 - 2 / (1 + e^2|x|) beyond.
MAP_FN float tanh_fast(float x) {
  const float a = fabsf(x), u = x * x;
  float q = -0.005905868674f;
  q = fmaf(q, u, 0.02080538484f);
  q = fmaf(q, u, -0.05378668365f);
  q = fmaf(q, u, 0.1333195824f);
  q = fmaf(q, u, -0.3333329927f);
  const float small = fmaf(x * u, q, x);
  const float large = 1.0f - 2.0f * MAP_RCP(1.0f + MAP_EXP(2.0f * a));
  return a < 0.6f ? small : copysignf(large, x);
}

}  // namespace rola
