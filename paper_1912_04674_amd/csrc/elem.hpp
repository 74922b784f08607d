// elem.hpp -- FP64 elementary functions for the ranges the particles' state
// takes, shared by the passes.
#pragma once
#include <hip/hip_runtime.h>

namespace envpic {

// |t| at most a few turns: t - n pi/2 with pi/2 in two parts, Taylor series
// of the remainder (at most pi/4; the first omitted terms are below 1e-17)
__device__ inline void sincos_r(double t, double* sn, double* cs) {
  const double n = rint(t * 0.63661977236758134308);
  double r = fma(-n, 1.57079632679489661923, t);
  r = fma(-n, 6.12323399573676603587e-17, r);
  const double z = r * r;
  double a = 1.0 / 355687428096000.0;  // 1/17!
  a = fma(a, z, -1.0 / 1307674368000.0);
  a = fma(a, z, 1.0 / 6227020800.0);
  a = fma(a, z, -1.0 / 39916800.0);
  a = fma(a, z, 1.0 / 362880.0);
  a = fma(a, z, -1.0 / 5040.0);
  a = fma(a, z, 1.0 / 120.0);
  a = fma(a, z, -1.0 / 6.0);
  const double s = fma(a * z, r, r);
  double b = 1.0 / 20922789888000.0;  // 1/16!
  b = fma(b, z, -1.0 / 87178291200.0);
  b = fma(b, z, 1.0 / 479001600.0);
  b = fma(b, z, -1.0 / 3628800.0);
  b = fma(b, z, 1.0 / 40320.0);
  b = fma(b, z, -1.0 / 720.0);
  b = fma(b, z, 1.0 / 24.0);
  b = fma(b, z, -0.5);
  const double c = fma(b, z, 1.0);
  const int q = (int)n;
  const double u = (q & 1) ? c : s, v = (q & 1) ? s : c;
  *sn = (q & 2) ? -u : u;
  *cs = ((q + 1) & 2) ? -v : v;
}

}  // namespace envpic
