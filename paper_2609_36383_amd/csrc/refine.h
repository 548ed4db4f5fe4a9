// refine.h -- FP64 reciprocal and square root of positive normal numbers from hardware
// estimates of relative error 2^-24 at most (measured), to within 0.5 ulp and a few
// thousandths.  Plain arithmetic, so that the host can check it.
#pragma once

#include <math.h>

namespace gmhc {

// 1 / x from r ~ 1 / x, by one third-order step.
__host__ __device__ __forceinline__ double refined_rcp(double x, double r) {
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// sqrt(a) from y ~ 1 / sqrt(a): a third-order step on t = a y, whose two roundings leave up to
// 0.75 ulp, then the exact residual's step.
__host__ __device__ __forceinline__ double refined_sqrt(double a, double y) {
  const double t = a * y;
  const double e = fma(-t, y, 1.0);
  const double s = fma(t * e, fma(e, 0.375, 0.5), t);
  return fma(fma(-s, s, a), 0.5 * y, s);
}

}  // namespace gmhc
