// Division by a value known beforehand, without the division.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace lddmm {

// a / h, correctly rounded, with ih = 1 / h rounded: Markstein's theorem ("Computation of
// elementary functions on the IBM RISC System/6000 processor", 1990).  A correction by the
// remainder, which an fma gives exactly, makes the quotient faithful, and a second one, with a
// correctly rounded reciprocal, rounds it as the division does: 5 operations instead of the
// division's dozen.  Holds for the h of div_by_fits and 1e-200 <= |a| < kDivMax, or a = 0; a
// smaller a keeps its sign.  From kDivMax on, infinite and NaN included, the product stands,
// which is at least 1e100, or not finite where the division is.
constexpr double kDivMax = 1e200;

inline bool div_by_fits(double h) { return h >= 1e-100 && h <= 1e100; }

__host__ __device__ __forceinline__ double div_by(double a, double h, double ih) {
  const double q0 = a * ih;
  const double q1 = __builtin_fma(__builtin_fma(-q0, h, a), ih, q0);
  const double q2 = __builtin_fma(__builtin_fma(-q1, h, a), ih, q1);
  return fabs(a) < kDivMax ? q2 : q0;
}

// FITS: div_by_fits(h), else the division itself.
template <bool FITS>
__host__ __device__ __forceinline__ double quotient(double a, double h, double ih) {
  return FITS ? div_by(a, h, ih) : a / h;
}

}  // namespace lddmm
