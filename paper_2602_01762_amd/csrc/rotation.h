// Rotary angle -> cosine and sine (plain C++, shared by the kernels and a
// host unit test).
#pragma once
#include <math.h>

namespace prism {

// cos and sin of an angle in fp64: the angle less its nearest multiple of
// pi/2, the Taylor sums of sine and cosine on what is left (|r| <= pi/4: the
// terms dropped are below 1e-11), and the quadrant.  The multiple is the low
// bits of the mantissa of 1.5 * 2^52 + it, so it may reach 2^51 quarter turns
// (a base below 1 makes the frequencies grow; past that, fp64 angles have no
// fraction left), and costs fewer instructions than a round and a conversion.
// No branch and no scratch (the library's sincosf keeps a large-argument
// path), but still a few hundred cycles of one wave, so the kernels compute it
// while their first loads are in flight.
__host__ __device__ inline void rotation_cos_sin(double ang, float &c, float &s) {
  const double round = 6755399441055744.0;                      // 1.5 * 2^52
  const double t = fma(ang, 0.63661977236758134, round);        // 2 / pi
  const double q = t - round;
  double r = fma(-q, 1.5707963267948966, ang);                  // pi / 2, high and low words
  r = fma(-q, 6.123233995736766e-17, r);
  const double z = r * r;
  double sn = fma(z, -1.0 / 39916800.0, 1.0 / 362880.0);
  sn = fma(z, sn, -1.0 / 5040.0);
  sn = fma(z, sn, 1.0 / 120.0);
  sn = fma(z, sn, -1.0 / 6.0);
  sn = fma(z * r, sn, r);
  double cs = fma(z, 1.0 / 479001600.0, -1.0 / 3628800.0);
  cs = fma(z, cs, 1.0 / 40320.0);
  cs = fma(z, cs, -1.0 / 720.0);
  cs = fma(z, cs, 1.0 / 24.0);
  cs = fma(z, cs, -0.5);
  cs = fma(z, cs, 1.0);
  const int quad = (int)__builtin_bit_cast(long long, t) & 3;
  const float fs = (float)((quad & 1) ? cs : sn), fc = (float)((quad & 1) ? sn : cs);
  s = (quad & 2) ? -fs : fs;
  c = ((quad + 1) & 2) ? -fc : fc;
}

}  // namespace prism
