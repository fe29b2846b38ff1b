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
//            amounts; else the run is marked open, with its plain sum where that
//            may serve;
//   chain    run by run, s plus the amount of its parity; an open run's plain
//            sum, or its terms one after another.
//
// Plain functions, so that the same lines run on the CPU in a test.
#pragma once

#include <math.h>
#include <limits.h>
#include <stdint.h>
#include <string.h>

#ifdef __HIP__
#define GORIO_HD __host__ __device__ __forceinline__
#else
#define GORIO_HD inline
#endif

namespace gorio {

constexpr uint32_t kSumRun = 256;  // terms per run

// A run's plain sum, the least and greatest of its partial sums (that of no
// terms, 0, included) and the exponent of the lowest bit set in any term.
struct RunOutline {
  double sum, lo, hi;
  int low;
};

// What a run adds to a sum whose multiple of the spacing is even / odd.  An
// open run has a NaN in `even`; its payload is 0, or kUnitBias + the exponent
// of a unit that divides all its terms and in which its partial sums need no
// more than 53 bits, and then `odd` is the run's plain sum.
struct RunAmount {
  double even, odd;
};
constexpr int kUnitBias = 2048;

// Exponent of a float's lowest set bit (INT_MAX: none).
GORIO_HD int lowest_bit(float x) {
  uint32_t b;
  memcpy(&b, &x, 4);
  uint32_t m = b & 0x7FFFFFu;
  int e = (int)((b >> 23) & 0xFFu);
  if (e) m |= 0x800000u;
  else e = 1;
  return m ? e - 150 + __builtin_ctz(m) : INT_MAX;
}

GORIO_HD RunOutline outline_start() { return {0.0, 0.0, 0.0, INT_MAX}; }
GORIO_HD void outline_add(RunOutline &o, float x) {
  o.sum += (double)x;
  // a NaN partial sum stays in lo and hi
  o.lo = o.lo < o.sum ? o.lo : o.sum;
  o.hi = o.hi > o.sum ? o.hi : o.sum;
  const int e = lowest_bit(x);
  o.low = e < o.low ? e : o.low;
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

// 2^e for e within the normal range.
GORIO_HD double sum_pow2(int e) { return sum_bits_as_double((uint64_t)(e + 1023) << 52); }

// The mark of an open run whose terms are added one after another.
GORIO_HD double sum_open_mark() { return sum_bits_as_double(0x7FF8000000000000ull); }

// The mark of an open run (see RunAmount): with far < 2^e the bound of its
// partial sums, whole multiples of 2^(e - 52) are added without rounding.
GORIO_HD RunAmount run_open(const RunOutline &o, double margin) {
  const uint64_t nan = 0x7FF8000000000000ull;
  const double far = fmax(fabs(o.sum + o.lo), fabs(o.sum + o.hi)) + margin;
  if (far < 0x1p400) {
    const int unit = (int)(sum_double_bits(far) >> 52) - 1023 + 1 - 52;
    if (unit > -1000 && o.low >= unit) return {sum_bits_as_double(nan | (uint64_t)(unit + kUnitBias)), 0.0};
  }
  return {sum_open_mark(), 0.0};
}
// Whether an open run's plain sum can be added to s.
GORIO_HD bool run_is_exact(double s, double mark) {
  const int p = (int)(sum_double_bits(mark) & 0xFFFFull);
  if (p == 0) return false;
  const double t = s * sum_pow2(kUnitBias - p);  // s in units, below 2^53
  return rint(t) == t;
}

// Whether a sum is an odd multiple of its binade's spacing.
GORIO_HD bool sum_is_odd(double s) { return (sum_double_bits(s) & 1ull) != 0; }

}  // namespace gorio
