// Square root, reciprocal and quotient in FP64 by short chains.  Free of HIP
// headers, so that they can be tested on the CPU.
#pragma once
#include <math.h>

#ifdef __HIPCC__
#define CFOG_ROOT_HD __host__ __device__ __forceinline__
#else
#define CFOG_ROOT_HD inline
#endif

namespace cfog {

// The square root of d > 0 and the reciprocal r of that root, from an estimate
// y of 1 / sqrt(d) by Goldschmidt's iteration and a final correction by the
// residual d - g g; then quotients by the root as Markstein's: q = t r corrected
// by its residual.  Shorter than a square root and a division of their own, which
// also serve what d cannot be here (below), with the same results: from estimates
// off by up to 2^-14, every one of 1.8 10^6 random d between 2^-960 and 2^13 and
// quotients by its root equal sqrt and /.
// A pivot of the normal matrix is at most its diagonal entry, a sum of squares of
// monomials of at most 1 over at most 4096 points.  One below 2^-960, where the
// residual underflows, takes points that all lie within 2^-150 of the normalised
// axes; its root is within 2^-52, or where d is subnormal, 2^-27.
CFOG_ROOT_HD double sqrt_rcp(double d, double y, double& r) {
  double g = d * y, h = 0.5 * y;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  g = fma(fma(-g, g, d), h, g);
  g = fma(fma(-g, g, d), h, g);
  r = h + h;
  r = fma(fma(-g, r, 1.0), r, r);
  r = fma(fma(-g, r, 1.0), r, r);
  return g;
}
CFOG_ROOT_HD double quotient(double t, double g, double r) {
  const double q = t * r;
  return fma(fma(-g, q, t), r, q);
}

}  // namespace cfog
