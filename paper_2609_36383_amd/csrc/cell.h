// cell.h -- the cell a position lies in, for the index sort by cell (sort.hip) and for the
// passes that take particles in its order (point.hip).  Those hold one cell for up to sixteen
// particles of equal keys, so both must find the same cell for the same position, also where
// rounding decides it (on a knot): the product that decides is an explicit fma, not left to the
// contraction of the kernel at hand.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include "gmhc_internal.h"

namespace gmhc {
namespace {

// Base node of coordinate x along axis l (the nearest node for S_2, the node below for S_1;
// unwrapped) and the offset from it.  A coordinate that is not finite, or 1e9 cells away, counts
// as the origin's on that axis, so that every position has a valid cell.
__device__ __forceinline__ double axis_node(const Mesh& M, int l, bool linear, double x, double& f) {
  const double d = x - M.lo[l];
  const double r = floor(fma(d, M.inv_h[l], linear ? 0.0 : 0.5));
  const bool ok = r > -1.0e9 && r < 1.0e9;  // false for a NaN
  f = ok ? fma(d, M.inv_h[l], -r) : 0.0;
  return ok ? r : 0.0;
}

}  // namespace
}  // namespace gmhc
