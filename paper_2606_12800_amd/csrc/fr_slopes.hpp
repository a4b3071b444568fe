// Multiple-flow-direction weights t_k = (s_k / s_max)^p: in float64, and in
// float32 for cells whose slopes lie outside the range in which the solvers'
// own float32 steps (a reciprocal of s_max, the quotient kept above 2^-126)
// are right.
#pragma once

#include "fr_internal.hpp"

namespace fr {

// Slopes from 2^-60 to 2^60 give quotients of at least 2^-120 and exact
// scalings; below, a drop may be subnormal (its diagonal slope is not exact,
// the reciprocal of s_max is infinite), above, a drop or the reciprocal may
// overflow or be flushed.  An elevation range of 60 binary orders either way
// holds all terrain but flats at elevation 0 raised by single float32 steps
// and cells beside a missing-value mark, so the other branch is rarely taken.
constexpr float SLOPE_LO = 0x1p-60f, SLOPE_HI = 0x1p60f;

// Receivers: bit k of m, at zk[k], over a diagonal where bit k of diag is set.
// Drops, slopes and quotients are float64, which holds all of them; the
// logarithm is taken of the quotient's mantissa, its exponent added.
template <int N>
__device__ __forceinline__ void wide_weights(float zc, const float (&zk)[N], uint32_t m, uint32_t diag, float p,
                                             float (&t)[N]) {
  double s[N], smax = 0.0;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double drop = (double)zc - (double)zk[k];
    s[k] = ((m >> k) & 1u) ? (((diag >> k) & 1u) ? drop * 0x1.6a09e667f3bcdp-1 : drop) : 0.0;
    smax = fmax(smax, s[k]);
  }
  const double ism = smax > 0.0 ? 1.0 / smax : 0.0;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double x = s[k] * ism;  // above 2^-280
    const float l = __builtin_amdgcn_logf((float)__builtin_amdgcn_frexp_mant(x)) +
                    (float)__builtin_amdgcn_frexp_exp(x);
    t[k] = s[k] > 0.0 ? __builtin_amdgcn_exp2f(p * l) : 0.0f;
  }
}

// Powers (s / 2^e)^p in float64, s = drop / (diag ? sqrt 2 : 1), in two steps:
// log2(s / 2^e) as l + ll, from the series of atanh, log2 x = (2 / ln 2)
// atanh((x - 1) / (x + 1)), its quotient and leading term in two doubles; then
// 2^(p (l + ll)) by the series of 2^z on |z| <= 1/2.  The diagonal is half a
// unit of the logarithm, so no slope is rounded; a power is within 0.7 units in
// the last place.  Against pow() on the slopes there are no special cases: the
// peeling solver's float64 MFD takes 2.3 ms against 3.0 on a raw 4096^2 grid
// and 37 against 90 on 12288^2, and its fractions are off by at most 4.3e-16
// against 5.9e-16 (p = 1.1, slopes over 40 binary orders).
__device__ __forceinline__ void slope_log2(double drop, bool diag, int e, double& l, double& ll) {
  double m = __builtin_amdgcn_frexp_mant(drop);  // [1/2, 1)
  int ex = __builtin_amdgcn_frexp_exp(drop) - e;
  if (m < 0x1.6a09e667f3bcdp-1) {  // to [1 / sqrt 2, sqrt 2)
    m *= 2.0;
    ex -= 1;
  }
  // f + fl = (m - 1) / (m + 1); m - 1 is exact.
  const double num = m - 1.0, den = m + 1.0, back = den - 1.0;
  const double denl = (1.0 - (den - back)) + (m - back);
  double r = __builtin_amdgcn_rcp(den);
  r = fma(fma(-den, r, 1.0), r, r);
  r = fma(fma(-den, r, 1.0), r, r);
  const double f = num * r, fl = fma(-f, denl, fma(-f, den, num)) * r, u = f * f;
  // 1/3 + u/5 + ... + u^10/23; |f| <= 0.172.
  double q = 1.0 / 23;
  q = fma(q, u, 1.0 / 21);
  q = fma(q, u, 1.0 / 19);
  q = fma(q, u, 1.0 / 17);
  q = fma(q, u, 1.0 / 15);
  q = fma(q, u, 1.0 / 13);
  q = fma(q, u, 1.0 / 11);
  q = fma(q, u, 1.0 / 9);
  q = fma(q, u, 1.0 / 7);
  q = fma(q, u, 1.0 / 5);
  q = fma(q, u, 1.0 / 3);
  // 2 / ln 2 in two doubles times f + fl, then the rest of the series.
  constexpr double ch = 0x1.71547652b82fep+1, cl = 0x1.777d0ffda0d24p-55;
  const double a = ch * f;
  const double al = fma(a * u, q, fma(ch, f, -a) + fma(ch, fl, cl * f));
  const double whole = (double)ex - (diag ? 0.5 : 0.0);  // 0 or at least |a|
  const double h = whole + a, hl = (a - (h - whole)) + al;
  l = h + hl;
  ll = hl - (l - h);
}
// 2^(p (l + ll)), l below 1; below 2^-1100 it is 0.
__device__ __forceinline__ double slope_exp2(double l, double ll, double p) {
  const double ph = p * l, pl = fma(p, ll, fma(p, l, -ph));
  const double y = ph + pl, n = rint(y);
  const double z = (y - n) + (pl - (y - ph));
  // 2^z = 1 + z ln 2 + (z ln 2)^2 / 2 + ..., 14 terms.
  double w = 0x1.314964d5878a9p-44;
  w = fma(w, z, 0x1.816193166d0f9p-40);
  w = fma(w, z, 0x1.c3bd650fc2986p-36);
  w = fma(w, z, 0x1.e8cac7351bb25p-32);
  w = fma(w, z, 0x1.e4cf5158b8ecap-28);
  w = fma(w, z, 0x1.b5253d395e7c4p-24);
  w = fma(w, z, 0x1.62c0223a5c824p-20);
  w = fma(w, z, 0x1.ffcbfc588b0c7p-17);
  w = fma(w, z, 0x1.430912f86c787p-13);
  w = fma(w, z, 0x1.5d87fe78a6731p-10);
  w = fma(w, z, 0x1.3b2ab6fba4e77p-7);
  w = fma(w, z, 0x1.c6b08d704a0cp-5);
  w = fma(w, z, 0x1.ebfbdff82c58fp-3);
  w = fma(w, z, 0x1.62e42fefa39efp-1);
  return y >= -1100.0 ? ldexp(fma(w, z, 1.0), (int)n) : 0.0;
}

}  // namespace fr
