// Internal: coefficients of the odd matrix iteration for the polar factor (polar.hip),
//   X <- (a I + b X X^T + c (X X^T)^2) X,
// which maps every singular value x of X to x (a + b x^2 + c x^4): polar_steps, the steps that take any
// spectrum to 1 (host), and polar_decide, which picks them one by one from what X X^T shows (device).
#pragma once
#include <algorithm>
#include <math.h>
#include <stdint.h>
#include <utility>

#ifdef __HIPCC__
#define FFS_HOST_DEVICE __host__ __device__
#else
#define FFS_HOST_DEVICE
#endif

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

// The same iteration with its steps chosen as it goes.  polar_steps must assume that the least singular
// value is 1 / (1024 r) of the norm; a sketch of a weight matrix has its own far above that (a ratio of 2 to 4 to the
// largest for a flat spectrum, 20 to 400 for spectra that decay like i^-1/2 and 1/i), so that most of its
// steps stretch what needs no stretching: rank 512, 13 steps where 4 do.  Two figures of G = X X^T are enough:
//   before the first step a bound of the largest value (the row sums of |G| and ||G||_F), by which X is
//     scaled: up to 7 times closer than the norm itself;
//   before every later step D = ||G - I||_F^2, the sum of (1 - x^2)^2 over the values x.
// GROW    the minimax quintic of [0.15, 1], until D <= POLAR_BULK r: the bulk of the values is past 0.5 then
//         (or, at the latest, everything is: max_grow steps, those of polar_steps).
// RANGE1, RANGE2   the minimax quintics of [0.5, 1] and of its image: what was past 0.5 ends within 1e-5 of 1.
// FINISH  D now counts the values that were smaller.  The quintics with p(1) = 1, p'(1) = 0 keep the others
//         at 1: slope 2.7 at zero (K) while D > 0.5, that is while a value may be below 0.54, then
//         (15 x - 10 x^3 + 3 x^5) / 8.  Slopes from 2.9 on are not safe: the inner maximum comes
//         too near the repelling fixed point sqrt((a - 1) / (a - 1.5)); 2.7: 1.10 and 1.19.
// The iteration ends with the cubic step that starts from D <= POLAR_DONE: no value is further than 2.3e-3
// from 1 before it, so none further than 3e-8 after it.
//
// A step of FINISH takes a small value up by 2.7 where GROW takes it up by 3.6, and D does not show how small the values
// are that it counts.  So the climbs after j growth steps are numbered: when no more of them are left (climbs[j]) than the
// least value that polar_steps takes to 1 can afford, growth is resumed (regrow[j] steps, which spread the values
// at 1 over [0.5, 1] again), and RANGE1, RANGE2 and one cubic step end it.  max_steps is then at most two more than the
// steps of polar_steps (rank 512: 15 and 13; rank 200: 14 and 12, by climbing alone 16), whatever the spectrum; what was left at
// the end (values smaller still, or zero) is promised nothing, as there.
constexpr float POLAR_BULK = 0.35f, POLAR_DONE = 2e-5f;
constexpr double POLAR_CLIMB_ROOM = 1.12;   // (the climbs' inner maximum is 1.10)
constexpr int POLAR_LEAST_STEPS = 4;   // GROW, RANGE1, RANGE2 and a last one (a fixed plan has more)
constexpr int POLAR_MAX_GROW = 16, POLAR_NO_LIMIT = 15;
enum { POLAR_GROW = 0, POLAR_RANGE2 = 1, POLAR_FINISH = 2, POLAR_ENDED = 3, POLAR_REGROW = 4 };
struct PolarPlan {
  float grow[3], range1[3], range2[3], climb[3], cubic[3];   // grow: for values up to 1, into (0, 1]
  int max_grow, max_steps;
  unsigned long long climbs, regrow;   // four bits for each j below POLAR_MAX_GROW
  int fixed;                          // no choice: the max_steps steps of polar_steps, this launch's is coef
  float coef[3];
};
struct PolarState {
  int mode;
  int grown;    // growth steps; from bit 8 on climbs, or growth steps resumed
  int parity;   // which of the two buffers holds X
  int act;      // the step is carried out
  int last;     // and is the last
};

// Matrices [r, d].  The least value of a flat sketch is 1 - sqrt(r / d) of the largest, and of a square one far below: from
// 10 r > 9 d on the steps of polar_steps are taken, of which there are two fewer.  us a factorisation of two matrices, singular
// values i^0 / i^-1/2 / i^-1, fixed steps and chosen ones: 512 x 1986 rank 456 438 and 371 / 389 / 426, rank 512 493 and 468 / 491 /
// 558; 1024 x 3972 rank 520 797 and 509 / 511 / 596, rank 816 1190 and 775 / 849 / 1068, rank 920 1347 and 951 / 1037 / 1204, rank
// 1024 1680 and 1925; 2048 x 7944 rank 1432 5206 and 2611 / 3268 / 3925, rank 1840 7825 and 4820 / 5319 / 6849, rank 2048 9340 and 10610.
inline PolarPlan polar_plan(int r, int d) {
  PolarPlan p = {};
  if (10 * (int64_t)r > 9 * (int64_t)d) {
    float coef[POLAR_MAX_STEPS][3];
    p.fixed = 1;
    p.max_steps = polar_steps(r, coef);
    return p;
  }
  double q[3], at[2], grow[3], r1[3], r2[3];
  const auto peak = [&](const double* c, double lo, double end) {   // largest value over [lo, end]
    double most = std::max(quintic(c, lo), quintic(c, end));
    const int n = quintic_extrema(c, at);
    for (int i = 0; i < n; ++i)
      if (at[i] >= lo && at[i] <= end) most = std::max(most, quintic(c, at[i]));
    return most;
  };
  minimax_quintic(0.15, 1.0, q);
  const double top = peak(q, 0.0, 1.0);
  for (int i = 0; i < 3; ++i) p.grow[i] = (float)(grow[i] = q[i] / top);
  minimax_quintic(0.5, POLAR_RANGE_ROOM, r1);
  for (int i = 0; i < 3; ++i) p.range1[i] = (float)r1[i];
  const double hi = peak(r1, 0.5, POLAR_RANGE_ROOM);
  minimax_quintic(quintic(r1, 0.5), hi * POLAR_RANGE_ROOM, r2);
  for (int i = 0; i < 3; ++i) p.range2[i] = (float)r2[i];
  const double k[3] = {2.7, -2.9, 1.2}, f[3] = {1.875, -1.25, 0.375};
  for (int i = 0; i < 3; ++i) { p.climb[i] = (float)k[i]; p.cubic[i] = (float)f[i]; }
  // the least value alone, the bulk past 0.5 after j growth steps
  const double g = POLAR_GROW_ROOM, least = 1.0 / (1024.0 * r);
  const auto grown = [&](double x) { return quintic(grow, x / g); };
  for (double x = least; x < 0.5; x = grown(x)) ++p.max_grow;
  p.max_grow = std::min(std::max(p.max_grow, 1), POLAR_MAX_GROW);   // (12 at rank 8192)
  const auto behind = [&](int j, int climbs) {   // j growth steps, both range steps, some climbs
    double x = least;
    for (int i = 0; i < j; ++i) x = grown(x);
    x = quintic(r2, quintic(r1, x));
    for (int i = 0; i < climbs; ++i) x = quintic(k, x);
    return x;
  };
  // steps in all if nothing but climbs follow, for the least value; and one more (D adds up several that are nearly done)
  const auto climbing = [&](int j) {
    double x = behind(j, 0);
    int n = j + 2;
    for (double dev = (1 - x * x) * (1 - x * x); dev > POLAR_DONE / 2; dev = (1 - x * x) * (1 - x * x), ++n)
      x = quintic(dev > 0.5 ? k : f, x);
    return n + 2;
  };
  const auto resumed = [&](int j, int climbs) {   // growth steps after some climbs
    int n = 1;
    for (double x = grown(behind(j, climbs) / POLAR_CLIMB_ROOM); x < 0.5; x = grown(x)) ++n;
    return n;
  };
  p.max_steps = p.max_grow + 3;
  for (int j = 1; j < p.max_grow; ++j) p.max_steps = std::max(p.max_steps, std::min(climbing(j), j + 5 + resumed(j, 0)));
  for (int j = 1; j < p.max_grow; ++j) {
    int c = POLAR_NO_LIMIT, g = 0;
    if (climbing(j) > p.max_steps) {
      for (c = 0; j + 5 + c + 1 + resumed(j, c + 1) <= p.max_steps;) ++c;
      g = resumed(j, c);
    }
    p.climbs |= (unsigned long long)c << (4 * j);
    p.regrow |= (unsigned long long)g << (4 * j);
  }
  return p;
}

// Step `step` (0 .. max_steps - 1) of a matrix of r rows: its coefficients and the state after it.  fig: the
// bound of the largest value before the first step, D before the others.
FFS_HOST_DEVICE inline PolarState polar_decide(const PolarPlan& p, int step, int r, PolarState s, float fig, float (&c)[3]) {
  c[0] = c[1] = c[2] = 0.f;
  if (step > 0 && (s.mode == POLAR_ENDED || s.last)) {
    s.mode = POLAR_ENDED;
    s.act = s.last = 0;
    return s;
  }
  if (step == 0) s.mode = POLAR_GROW, s.grown = 0, s.parity = 0;
  const int j = s.grown & 255, count = s.grown >> 8;
  if (p.fixed) {
    for (int i = 0; i < 3; ++i) c[i] = p.coef[i];
    s.act = 1;
    s.last = step == p.max_steps - 1;
    s.parity ^= 1;
    return s;
  }
  // (the coefficients are picked by value: an address into the plan or an index that is not constant would put a copy of
  // the kernel's arguments in every thread's scratch memory)
  int pick = 4;
  float end = 1.f;
  bool done = false;
  if (s.mode == POLAR_GROW) {
    if (step > 0 && (fig <= POLAR_BULK * (float)r || j >= p.max_grow)) {
      pick = 1;
      s.mode = POLAR_RANGE2;
    } else {
      pick = 0;
      // (a zero matrix has no bound, nor has one with NaN)
      end = (float)POLAR_GROW_ROOM * (step == 0 && fig > 1e-6f && fig < 1.f ? fig : 1.f);
      ++s.grown;
    }
  } else if (s.mode == POLAR_RANGE2) {
    pick = 2;
    s.mode = POLAR_FINISH;
  } else if (s.mode == POLAR_REGROW) {
    if (count >= (int)(p.regrow >> (4 * j) & 15)) {
      pick = 1;
      s.mode = POLAR_RANGE2;
      s.grown = p.max_grow;
    } else {
      pick = 0;
      end = (float)POLAR_GROW_ROOM;
      s.grown += 256;
    }
  } else if (j >= p.max_grow || fig <= POLAR_DONE) {
    done = true;
  } else if (fig > 0.5f) {
    const int most = (int)(p.climbs >> (4 * j) & 15);
    if (most == POLAR_NO_LIMIT || count < most) {
      pick = 3;
      s.grown += 256;
    } else {
      pick = 0;
      end = (float)(POLAR_GROW_ROOM * POLAR_CLIMB_ROOM);
      s.mode = POLAR_REGROW;
      s.grown = j + 256;
    }
  }
  const float e = 1.f / end, e2 = e * e;
  const float scale[3] = {e, e * e2, e * e2 * e2};
  for (int i = 0; i < 3; ++i)
    c[i] = scale[i] * (pick == 0 ? p.grow[i] : pick == 1 ? p.range1[i] : pick == 2 ? p.range2[i] : pick == 3 ? p.climb[i] : p.cubic[i]);
  s.act = 1;
  s.last = done || step == p.max_steps - 1;
  s.parity ^= 1;
  return s;
}

}  // namespace ffsplit
