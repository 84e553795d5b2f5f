// slope.hpp -- the Van Leer limited slope of section 4.3.2 without a branch.
// vl_slope (kernels.hpp) skips the quotient when ab <= 0; here it is always
// formed and then selected, so that a wavefront whose lanes disagree on the
// sign does not split, and the compiler can interleave the slopes of a face.
// The same quotient: the hardware reciprocal of a + b refined by two Newton
// steps, then 2ab times it with one correction (within a few ulp of the
// IEEE quotient); 0 when ab <= 0; b when unlimited.
#pragma once
#include <hip/hip_runtime.h>

namespace hofks {

__device__ __forceinline__ double vl_slope_sel(double a, double b, int unlimited = 0) {
  const double ab = a * b;
  const double den = a + b;
  double r = __builtin_amdgcn_rcp(den);
  r = fma(fma(-den, r, 1.0), r, r);
  r = fma(fma(-den, r, 1.0), r, r);
  const double q = 2.0 * ab * r;
  const double v = fma(fma(-den, q, 2.0 * ab), r, q);
  return unlimited ? b : (ab > 0.0 ? v : 0.0);
}

// 1/x from the hardware reciprocal refined by two Newton steps (within a
// few ulp of the IEEE quotient, and a shorter dependency chain)
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return r;
}

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

// 1/x: one step of third order, 2^-24.4 -> 2^-73, then the last rounding
__device__ __forceinline__ double rcp3(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

}  // namespace hofks
