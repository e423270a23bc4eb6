// chan_tables.hpp - the channeliser's constants, evaluated at compile time in
// double precision and rounded once to float: the Hamming-windowed sinc
// prototype h[m] = (0.54 - 0.46 cos(2 pi m / (PL - 1))) sinc((m - PL/2) / L),
// m < PL = 4 L, and the twiddles e^{-2 pi i t / L}, t < L/2.  They depend on
// L alone, so they are part of the code object: formerly every call launched
// a kernel that computed them into the caller's scratch (3.5-5 us, half of
// the time of a small call).
#pragma once
#include <hip/hip_runtime.h>

namespace xeng {

constexpr int TAPS = 4;

namespace chan_math {

constexpr double PI = 3.14159265358979323846;

// sin and cos of x in [0, pi/4] by their Taylor series (the first terms left
// out, x^19 / 19! and x^18 / 18!, are below 1e-19 and 3e-18)
constexpr double sin_small(double x) {
  double term = x, sum = x;
  for (int k = 1; k < 9; ++k) {
    term *= -x * x / ((2 * k) * (2 * k + 1));
    sum += term;
  }
  return sum;
}
constexpr double cos_small(double x) {
  double term = 1, sum = 1;
  for (int k = 1; k < 9; ++k) {
    term *= -x * x / ((2 * k - 1) * (2 * k));
    sum += term;
  }
  return sum;
}

// cos(2 pi num / den): the octant is found in integers, so the reduction is exact
constexpr double cos_turn(long long num, long long den) {
  num %= den;
  if (num < 0) num += den;
  const int oct = (int)(8 * num / den);
  const long long rest = 8 * num - oct * den;                            // of the octant, over den
  const double x = (double)(oct % 2 ? den - rest : rest) / (double)den * (PI / 4);  // to the nearest axis
  const bool swap = oct == 1 || oct == 2 || oct == 5 || oct == 6;
  const double v = swap ? sin_small(x) : cos_small(x);
  return oct >= 2 && oct <= 5 ? -v : v;
}
constexpr double sin_turn(long long num, long long den) { return cos_turn(4 * num - den, 4 * den); }

}  // namespace chan_math

template <int L>
struct ChanTables {
  float h[TAPS * L];
  float tw[L / 2][2];
  constexpr ChanTables() : h(), tw() {
    constexpr long long PL = TAPS * L;
    for (int m = 0; m < PL; ++m) {
      const double w = 0.54 - 0.46 * chan_math::cos_turn(m, PL - 1);
      const long long k = 2 * m - PL;  // sinc(k / 2L) = sin(pi k / 2L) / (pi k / 2L)
      const double sinc = k == 0 ? 1.0 : chan_math::sin_turn(k, 4 * L) / (chan_math::PI * (double)k / (2 * L));
      h[m] = (float)(w * sinc);
    }
    for (int t = 0; t < L / 2; ++t) {
      tw[t][0] = (float)chan_math::cos_turn(t, L);
      tw[t][1] = (float)-chan_math::sin_turn(t, L);
    }
  }
};

template <int L>
__device__ const ChanTables<L> chan_tables = ChanTables<L>();

}  // namespace xeng
