// slope.hpp -- the Van Leer limited slope of section 4.3.2 without a branch,
// a reciprocal and a root.  vl_slope (kernels.hpp) skips the quotient when ab <= 0;
// here it is always formed and then selected, so that a wavefront whose lanes
// disagree on the sign does not split, and the compiler can interleave the
// slopes of a face.
#pragma once
#include <hip/hip_runtime.h>

namespace hofks {

// Half the limited slope, ab/(a + b) for ab > 0 and else 0 (b/2 when
// UNLIMITED).  The hardware reciprocal is good to 2^-24.4 (measured over 4e6
// arguments), one Newton step makes that 2^-48, and the correction of the
// quotient by its own remainder leaves the rounding of the last two
// operations: no second step is needed.
template <bool UNLIMITED>
__device__ __forceinline__ double half_slope(double a, double b) {
  if (UNLIMITED) return 0.5 * b;
  const double ab = a * b;
  const double den = a + b;
  double r = __builtin_amdgcn_rcp(den);
  r = fma(fma(-den, r, 1.0), r, r);
  const double q = ab * r;
  const double v = fma(fma(-den, q, ab), r, q);
  return ab > 0.0 ? v : 0.0;
}

// 1/x: two Newton steps, 2^-24.4 -> 2^-48 -> the rounding of the last
// operation (as the division 1/x rounds but for cases within 2^-97 of a tie)
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// n/d with r = rcp_nr(d): the product corrected by its remainder, which rounds
// as the division does
__device__ __forceinline__ double quotient(double n, double d, double r) {
  const double q = n * r;
  return fma(fma(-d, q, n), r, q);
}

// sqrt(x), x > 0 and finite: the hardware reciprocal root (2^-24.2), one
// coupled step for the root and its half reciprocal, and the correction by
// the remainder x - g^2.  (Arguments below the normal range count as its least.)
__device__ __forceinline__ double sqrt_pos(double x) {
  x = fmax(x, 2.2250738585072014e-308);
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double e = fma(-g, h, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  return fma(fma(-g, g, x), h, g);
}

}  // namespace hofks
