// Multiple-flow-direction weights t_k = (s_k / s_max)^p in float32 for cells
// whose slopes lie outside the range in which the solvers' own float32 steps
// (a reciprocal of s_max, the quotient kept above 2^-126) are right.
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

}  // namespace fr
