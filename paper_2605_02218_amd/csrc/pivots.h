// Four pivots of A = L D L^T without exchanges, for counting the negative ones (split.hip).  Plain arithmetic, the same on host and device.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

namespace covspec {

// A pivot that is counted.  Of a matrix of entries up to 1 a pivot p leaves numbers of 1 / p in the rest, which come off again at the next
// ones: the rest is then good to 1e-16 / p.  Where there is none p is taken as -1e-8, which is a matrix 1e-8 away, and good to 1e-8.  (With
// -1e-200, as in a recurrence of quotients, the squares of what it leaves overflow and every pivot behind it counts as negative.)
constexpr double kNoPivot = 1e-30, kPivotInstead = -1e-8;
__host__ __device__ inline double counted_pivot(double p, int& negative) {
  p = fabs(p) > kNoPivot ? p : kPivotInstead;
  negative += p < 0.0 ? 1 : 0;
  return p;
}

// The symmetric 4 x 4 block a = L D L^T: r the reciprocals of D, n the entries of inv(L) below its unit diagonal.
struct CountedBlock {
  double r0, r1, r2, r3, n10, n20, n21, n30, n31, n32;
};
template <typename Reciprocal>
__host__ __device__ inline CountedBlock count_block(double a00, double a10, double a11, double a20, double a21, double a22, double a30, double a31, double a32,
                                                    double a33, Reciprocal reciprocal, int& negative) {
  CountedBlock f;
  f.r0 = reciprocal(counted_pivot(a00, negative));
  const double b11 = fma(-(a10 * a10), f.r0, a11), b21 = fma(-(a20 * a10), f.r0, a21), b31 = fma(-(a30 * a10), f.r0, a31);
  const double b22 = fma(-(a20 * a20), f.r0, a22), b32 = fma(-(a30 * a20), f.r0, a32), b33 = fma(-(a30 * a30), f.r0, a33);
  f.r1 = reciprocal(counted_pivot(b11, negative));
  const double c22 = fma(-(b21 * b21), f.r1, b22), c32 = fma(-(b31 * b21), f.r1, b32), c33 = fma(-(b31 * b31), f.r1, b33);
  f.r2 = reciprocal(counted_pivot(c22, negative));
  f.r3 = reciprocal(counted_pivot(fma(-(c32 * c32), f.r2, c33), negative));
  const double l10 = a10 * f.r0, l20 = a20 * f.r0, l30 = a30 * f.r0, l21 = b21 * f.r1, l31 = b31 * f.r1, l32 = c32 * f.r2;
  f.n10 = -l10;
  f.n20 = fma(l21, l10, -l20);
  f.n21 = -l21;
  f.n31 = fma(l32, l21, -l31);
  f.n30 = -fma(l31, -l10, fma(l32, f.n20, l30));
  f.n32 = -l32;
  return f;
}

}  // namespace covspec
