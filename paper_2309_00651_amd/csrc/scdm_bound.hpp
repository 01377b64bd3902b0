// The bound that decides which blocks an SCDM step brings up to date
// (scdm.hip), apart so that a CPU test can check it.
#pragma once

#include <cmath>

#if defined(__HIPCC__)
#define HFX_HD __host__ __device__ __forceinline__
#else
#define HFX_HD inline
#endif

namespace hfx {

// A value that a point's residual norm cannot be below once it is downdated:
// `left` is the norm so far, t = q . a the pick's projection of the point's
// column a (n values, sum of squares a2) on the new unit direction q, which
// the update sums in another order.  Each sum is within n 2^-53 |a| of the
// exact projection (to first order; 2^-52 covers the direction's own norm and
// the higher orders), so the two differ by d at most and their squares by
// d (2 |t| + d); the last term covers the roundings of left - t^2.  The margin
// is absolute: where the direction takes nearly all of the norm, what is left
// may be far below the error of t^2.  Not finite for a non-finite column or
// direction.
HFX_HD double scdm_lower_bound(double left, double t, double a2, int n) {
  const double eps = 2.220446049250313e-16;  // 2^-52
  const double d = 2.0 * n * eps * sqrt(a2);
  return (left - t * t) - (d * (2.0 * fabs(t) + d) + 4.0 * eps * left);
}

}  // namespace hfx
