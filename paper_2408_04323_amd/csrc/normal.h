// Normal partial expectation and distribution function on the device, shared
// by the acquisition kernels (Sec. 4.4.1, Eq. 7-8; Sec. 4.4.2, Eq. 9).
//
// G(c) = E[(c - Y)^+] for Y ~ N(mu, sd^2) is sd * h(u), u = (c - mu) / sd,
// h(u) = u Phi(u) + phi(u), and max(0, c - mu) when sd = 0.  h(u) - h(-u) = u,
// so h(u) = max(u, 0) + h(-|u|), and for x >= 0, h(-x) = phi(x) g(x) with
// g(x) = 1 - x M(x), M the Mills ratio P(Z > x) / phi(x).
// * float: g is a rational function P4 / Q6 of s = x / 4 fitted on [0, 14]
//   (coefficients from gen_normal_tail.py: relative error 1e-8 in exact
//   arithmetic, 4e-7 evaluated in float), phi from one exp2; no branches, and
//   1 / sd is formed once per candidate;
// * double: g from one polynomial in 1 / (x + 5), phi from one exp; no branches.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace scoot {

// ---- double ---------------------------------------------------------------
// h(u) = max(u, 0) + phi(x) g(x), x = min(|u|, 39) (phi has underflowed by
// then); phi(0) g(x) = r^2 F(y), r = 1 / (x + 5), F a polynomial of degree 24 in
// y = a r + b, which falls from 1 at x = 0 to -1 at x = 39 (a, b and F from
// gen_normal_tail.py).  y is formed as 1 - (a / 5) x r, and the rounding of
// x + 5 and of x^2 is carried along, so that every step is good to an ulp or
// so: relative error of h below 8e-16 where phi is normal (u > -37).  Bound:
// instruction issue.  The erfc form and its continued fraction below -5, a
// divergent branch, took five to seven times the instructions and lost 1e-13 to
// cancellation near -5: EHVI of 131,072 candidates over 30 strips, workgroups
// of sixteen waves, 88 -> 50 us.
__device__ inline double h_normal(double u) {
  constexpr double F[25] = {  // highest power first
      -1.12101477295085141e-10, 4.86967593605889403e-10, 1.04070605953419851e-09, -6.62835407260708046e-09,
      -3.90281860591476856e-09, 5.62811940502463470e-08, -4.12662223160163691e-09, -4.23639627986858576e-07,
      1.79835609945399103e-07, 3.27089847717067436e-06, -1.39648882979885278e-06, -2.73738152460094199e-05,
      -1.74650752640066872e-06, 2.41709197835505708e-04, 2.95324945408691295e-04, -1.87610033183903467e-03,
      -6.90412138071519466e-03, 1.63158445439290042e-03, 8.50454094687063539e-02, 3.59253524239596278e-01,
      9.32154648213865844e-01, 1.75552344653162984e+00, 2.49687008210205263e+00, 2.61863175536668180e+00,
      1.73271719390637324e+00};
  double x = fabs(u);
  x = x > 39.0 ? 39.0 : x;  // a NaN stays
  const double d = x + 5.0, dl = x - (d - 5.0);  // x + 5 = d + dl
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  r = fma(r, fma(-dl, r, fma(-d, r, 1.0)), r);
  const double y = fma(-2.25641025641025639e+00, x * r, 1.0);
  double p = F[0];
#pragma unroll
  for (int k = 1; k < 25; ++k) p = fma(p, y, F[k]);
  const double q = x * x;
  double e = exp(-0.5 * q);
  e = fma(-0.5 * fma(x, x, -q), e, e);
  return fma(e, p * (r * r), fmax(u, 0.0));
}

// ---- float ------------------------------------------------------------------
// h(u) = max(u, 0) + phi(x) P4(s) / Q6(s), x = min(|u|, 16), s = x / 4.  Past
// x = 14 phi has underflowed to 0 in float (the clamp keeps P and Q finite).
__device__ inline float h_normal(float u) {
  const float x = fminf(fabsf(u), 16.0f);
  const float s = x * 0.25f;
  const float P = fmaf(fmaf(fmaf(fmaf(1.168936206e+00f, s, 3.086232540e+00f), s, 3.946713647e+00f), s,
                            2.790141401e+00f),
                       s, 9.999999897e-01f);
  const float Q =
      fmaf(fmaf(fmaf(fmaf(fmaf(fmaf(1.870267853e+01f, s, 4.938444122e+01f), s, 6.662181372e+01f), s, 5.403020981e+01f),
                     s, 2.706728781e+01f),
                s, 7.803394828e+00f),
           s, 1.0f);
  // phi(x) = exp(-x^2 / 2) / sqrt(2 pi) = 2^(-x^2 log2(e) / 2) / sqrt(2 pi)
  const float phi = 0.39894228040143267794f * __builtin_amdgcn_exp2f(x * x * -0.72134752044448170368f);
  return fmaxf(u, 0.0f) + phi * P * __builtin_amdgcn_rcpf(Q);
}

// G(c) given mu, sd and inv_sd = 1 / sd (inf when sd = 0, then unused).
template <typename T>
__device__ inline T partial_expectation(T c, T mu, T sd, T inv_sd) {
  const T g = sd * h_normal((c - mu) * inv_sd);
  return sd > T(0) ? g : (c - mu > T(0) ? c - mu : T(0));
}
template <typename T>
__device__ inline T reciprocal(T sd) {
  return T(1) / sd;
}

// Phi(u) = P(Z <= u) = erfc(-u / sqrt 2) / 2.
__device__ inline float normal_cdf(float u) { return 0.5f * erfcf(u * -0.70710678118654752440f); }
__device__ inline double normal_cdf(double u) { return 0.5 * erfc(u * -0.70710678118654752440); }

}  // namespace scoot
