// Exponentials of the rare cells outside the temperature tables, FP64 to a few
// ulp over the whole line: e^x = (1 + p) 2^n, |x - n ln 2| <= ln 2 / 2, p from
// the exponential series. A loop on purpose: the polynomial constants of an
// unrolled exponential would be kept in registers throughout the march (about
// 20 of them, a wavefront per SIMD less). Infinities give the limits, a NaN
// gives NaN.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace iris {

struct ExpParts {
  double p;
  int n;
};
__host__ __device__ __forceinline__ ExpParts exp_parts(double x) {
  const double xc = x < -2000.0 ? -2000.0 : x > 2000.0 ? 2000.0 : x;  // keeps a NaN
  const double n = x == x ? rint(xc * 1.44269504088896340736) : 0.0;
  double r = fma(n, -0x1.62e42fep-1, xc);  // ln 2: 28 bits, then the rest
  r = fma(n, -0x1.f473de6af278fp-30, r);
  double s = 1.0;
#pragma unroll 1
  for (int k = 16; k >= 2; --k) s = fma(r / (double)k, s, 1.0);
  return {r * s, (int)n};
}
__host__ __device__ __forceinline__ double exp_rare(double x) {
  const ExpParts e = exp_parts(x);
  return ldexp(1.0 + e.p, e.n);
}
// Where 2^n is far above 1 the two parts are scaled together: on their own they
// overflow to infinities of opposite sign from x = 711 on where p < 0.
__host__ __device__ __forceinline__ double expm1_rare(double x) {
  const ExpParts e = exp_parts(x);
  if (e.n > 64) return ldexp(1.0 + e.p, e.n);
  return ldexp(e.p, e.n) + (ldexp(1.0, e.n) - 1.0);
}

}  // namespace iris
