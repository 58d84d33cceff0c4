// Internal: coefficients of the odd matrix iteration for the polar factor (factor.hip),
//   X <- (a I + b X X^T + c (X X^T)^2) X,
// which maps every singular value x of X to x (a + b x^2 + c x^4).  Pure host arithmetic.
#pragma once
#include <algorithm>
#include <math.h>
#include <utility>

namespace ffsplit {

// x (p0 + p1 x^2 + p2 x^4), its positive critical points in ascending order (their number is returned)
inline double quintic(const double* p, double x) { return x * (p[0] + x * x * (p[1] + x * x * p[2])); }
inline int quintic_extrema(const double* p, double* at) {
  const double disc = 9 * p[1] * p[1] - 20 * p[0] * p[2];
  int n = 0;
  if (disc < 0 || p[2] == 0) return 0;
  for (int sign = -1; sign <= 1; sign += 2) {
    const double x2 = (-3 * p[1] + sign * (p[2] > 0 ? 1 : -1) * sqrt(disc)) / (10 * p[2]);
    if (x2 > 0) at[n++] = sqrt(x2);
  }
  return n;
}

// Odd quintic with the least max |1 - p| on [lo, hi] (lo < hi not too close): the values 1 - e, 1 + e,
// 1 - e, 1 + e at lo, the two interior extrema and hi (Remez exchange).
inline void minimax_quintic(double lo, double hi, double* p) {
  double q = (3 * lo + hi) / 4, r = (lo + 3 * hi) / 4;
  for (int it = 0; it < 40; ++it) {
    const double xs[4] = {lo, q, r, hi};
    double A[4][5];
    for (int i = 0; i < 4; ++i) {
      const double x = xs[i], x2 = x * x;
      A[i][0] = x; A[i][1] = x * x2; A[i][2] = x * x2 * x2; A[i][3] = (i & 1) ? -1 : 1; A[i][4] = 1;
    }
    for (int c = 0; c < 4; ++c) {   // elimination with row exchange
      int best = c;
      for (int i = c + 1; i < 4; ++i)
        if (fabs(A[i][c]) > fabs(A[best][c])) best = i;
      for (int j = 0; j < 5; ++j) std::swap(A[c][j], A[best][j]);
      for (int i = 0; i < 4; ++i)
        if (i != c) {
          const double f = A[i][c] / A[c][c];
          for (int j = c; j < 5; ++j) A[i][j] -= f * A[c][j];
        }
    }
    for (int i = 0; i < 3; ++i) p[i] = A[i][4] / A[i][i];
    double at[2];
    if (quintic_extrema(p, at) < 2) break;
    const double moved = fabs(at[0] - q) + fabs(at[1] - r);
    q = std::max(at[0], lo); r = std::max(at[1], lo);
    if (moved < 1e-10 * hi) break;
  }
}

// Coefficients (a, b, c) of the steps; the singular values start in [1 / (1024 r), 1].  While they may
// reach below 0.15 of the largest: the minimax quintic of [0.15, 1], which multiplies small ones by 3.6
// and keeps the others between 0.52 and 1 of the new largest (the fastest growth, slope 4.2, would map
// some large ones near zero, where they keep their absolute rounding error).  Then the minimax quintic
// of the range itself, and (15 x - 10 x^3 + 3 x^5) / 8 at the end, cubic convergence to 1.  Budget:
// singular values down to 1 / (1024 r) of the Frobenius norm (a square Gaussian Y, r = d_model, has its
// smallest near r^-1.5 of it); a basis direction below that comes out shorter than unit length.
//
// A quintic rises steeply (slope 7 relative to its scale) past the right end of its interval.  Were that
// end the largest value itself, a value there would carry its rounding error on to the next step's end
// seven times larger, and after nine steps of rank 512 leave the range for good (a sketch of rank one
// starts exactly there).  So each interval reaches GROW_ROOM or RANGE_ROOM times as far as the values do:
// everything up to that bound lands at or below the quintic's interior maximum, which is the largest
// value of the next step, and an overshoot within the room is lost instead of amplified.  The extrema
// are those of the coefficients as rounded to fp32.  A last step has slope zero at 1 and needs no room.
// (The room is a hundred times the fp32 error of a step and costs one step more at some ranks.)
constexpr int POLAR_MAX_STEPS = 48;
constexpr double POLAR_GROW_ROOM = 1.01, POLAR_RANGE_ROOM = 1.002;
inline int polar_steps(int r, float (*coef)[3]) {
  double lo = 1.0 / (1024.0 * r), hi = 1.0, grow[3];
  minimax_quintic(0.15, 1.0, grow);
  int n = 0;
  while ((lo < 1.0 - 3e-8 || hi > 1.0 + 3e-8) && n < POLAR_MAX_STEPS) {
    double p[3] = {1.875, -1.25, 0.375}, end = hi;
    if (lo < 0.15 * hi) {
      end = POLAR_GROW_ROOM * hi;
      double s = end;
      for (int i = 0; i < 3; ++i, s *= end * end) p[i] = grow[i] / s;
    } else if (hi - lo > 1e-3) {
      end = POLAR_RANGE_ROOM * hi;
      minimax_quintic(lo, end, p);
    }
    for (int i = 0; i < 3; ++i) p[i] = coef[n][i] = (float)p[i];
    // least and largest value over [lo, end]: at its ends or at a critical point between them
    double at[4] = {lo, end};
    const int m = 2 + quintic_extrema(p, at + 2);
    double least = quintic(p, lo), most = least;
    for (int i = 1; i < m; ++i)
      if (at[i] >= lo && at[i] <= end) {
        least = std::min(least, quintic(p, at[i]));
        most = std::max(most, quintic(p, at[i]));
      }
    lo = least; hi = most;
    ++n;
  }
  return n;
}

}  // namespace ffsplit
