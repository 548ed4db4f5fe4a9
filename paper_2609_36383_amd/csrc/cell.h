// cell.h -- the cell a position lies in, for the index sort by cell (sort.hip) and for the
// passes that take particles in its order (point.hip).  Those hold one cell for up to sixteen
// particles of equal keys, so both must find the same cell for the same position, also where
// rounding decides it (on a knot): the cell coordinate is rounded to FP64 first, not left to the
// contraction of the kernel at hand.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include "gmhc_internal.h"

namespace gmhc {
namespace {

// v as rounded to FP64: its product is not contracted into what follows.
__device__ __forceinline__ double rounded(double v) {
  asm("" : "+v"(v));
  return v;
}

// Base node of coordinate x along axis l (the nearest node for S_2, the node below for S_1;
// unwrapped) and the offset from it.  A coordinate that is not finite, or 1e9 cells away, counts
// as the origin's on that axis, so that every position has a valid cell.
__device__ __forceinline__ double axis_node(const Mesh& M, int l, bool linear, double x, double& f) {
  const double xi = rounded((x - M.lo[l]) * M.inv_h[l]);
  const double r = floor(linear ? xi : xi + 0.5);
  const bool ok = r > -1.0e9 && r < 1.0e9;  // false for a NaN
  f = ok ? xi - r : 0.0;
  return ok ? r : 0.0;
}

}  // namespace
}  // namespace gmhc
