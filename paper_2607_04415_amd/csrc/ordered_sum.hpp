// A long sum of float64 additions in a fixed order, computed in parallel with
// the same bits.
//
// The sum s = fl(s + x_i), i = 0 .. n-1, is a serial chain by definition.  But
// while s stays inside one binade, [2^e, 2^(e+1)) in magnitude, it is a whole
// multiple m of the binade's spacing U, and fl(s + x) = s + U * r where r
// depends on x / U and, only when x / U lies half way between two whole
// numbers, on whether m is even.  So a run of terms during which s stays in
// its binade adds one amount when it starts at an even m and another one when
// it starts at an odd m, whatever s is: both amounts can be found before s is
// known, all runs at once, by adding the run's terms to two stand-in sums of
// the right binade and parity.  Three steps:
//   outline  each run's plain sum and the range of its partial sums;
//   amounts  from the prefix sums of the outline: where s stays in one binade
//            during the run, with a margin above all rounding errors, the two
//            amounts; else the run is marked open;
//   chain    run by run, s plus the amount of its parity; the terms of an
//            open run one after another.
//
// Plain functions, so that the same lines run on the CPU in a test.
#pragma once

#include <math.h>
#include <stdint.h>
#include <string.h>

#ifdef __HIP__
#define GORIO_HD __host__ __device__ __forceinline__
#else
#define GORIO_HD inline
#endif

namespace gorio {

constexpr uint32_t kSumRun = 256;  // terms per run

// A run's plain sum and the least and greatest of its partial sums (that of
// no terms, 0, included).
struct RunOutline {
  double sum, lo, hi;
};

// What a run adds to a sum whose multiple of the spacing is even / odd.
// even = NaN marks an open run.
struct RunAmount {
  double even, odd;
};

GORIO_HD RunOutline outline_start() { return {0.0, 0.0, 0.0}; }
GORIO_HD void outline_add(RunOutline &o, double x) {
  o.sum += x;
  // a NaN partial sum stays in lo and hi
  o.lo = o.lo < o.sum ? o.lo : o.sum;
  o.hi = o.hi > o.sum ? o.hi : o.sum;
}

GORIO_HD double sum_bits_as_double(uint64_t b) {
  double d;
  memcpy(&d, &b, 8);
  return d;
}
GORIO_HD uint64_t sum_double_bits(double d) {
  uint64_t b;
  memcpy(&b, &d, 8);
  return b;
}

// Bound on |s - plain prefix sum| for every partial sum of n terms whose
// plain partial sums reach at most `most` in magnitude: either order makes at
// most n errors of half a spacing (2^-53 of a value just above `most`), the
// prefix sum of outlines as many again, and the outline's own range two more
// such shares; the factor 8 covers them for n < 2^31.
GORIO_HD double sum_margin(uint64_t n, double most) { return 8.0 * (double)n * 0x1p-53 * most; }

// Stand-in sums for a run that starts near `start` (a plain prefix sum) and
// whose partial sums stay within start + [lo, hi]: false when s may leave its
// binade during the run (or is not a normal number).
GORIO_HD bool run_stand_ins(double start, double lo, double hi, double margin, double &even, double &odd) {
  const double a = start + lo, b = start + hi;
  const double near = fmin(fabs(a), fabs(b)), far = fmax(fabs(a), fabs(b));
  const uint64_t exp = sum_double_bits(near) & 0x7FF0000000000000ull;
  const double floor_ = sum_bits_as_double(exp);  // 2^e
  const double unit = floor_ * 0x1p-52;
  // both ends on one side of zero, and the whole range inside [2^e, 2^(e+1))
  // with the margin and a few units to spare (comparisons fail on NaN)
  const double spare = margin + 8.0 * unit;
  if (!((a > 0.0) == (b > 0.0)) || !(near > 0x1p-900) || !(far < 0x1p900)) return false;
  if (!(near - spare > floor_) || !(far + spare < 2.0 * floor_)) return false;
  even = sum_bits_as_double(sum_double_bits(start) & ~1ull);
  odd = sum_bits_as_double(sum_double_bits(start) | 1ull);
  return true;
}

// Whether a sum is an odd multiple of its binade's spacing.
GORIO_HD bool sum_is_odd(double s) { return (sum_double_bits(s) & 1ull) != 0; }

}  // namespace gorio
