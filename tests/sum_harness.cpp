// Ordered column sums on the CPU: the library's run arithmetic
// (csrc/ordered_sum.hpp) against a plain sequential loop, bit for bit.
// Usage: sum_harness KIND N SEED; prints "open RUNS equal 0|1".
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <string>
#include <vector>

#include "../paper_2607_04415_amd/csrc/ordered_sum.hpp"

using namespace gorio;

int main(int argc, char **argv) {
  if (argc != 4) return 2;
  const std::string kind = argv[1];
  const size_t n = (size_t)atoll(argv[2]);
  std::mt19937_64 rng((uint64_t)atoll(argv[3]));
  std::normal_distribution<double> gauss(0.0, 1.0);
  std::vector<float> x(n);
  for (size_t i = 0; i < n; ++i) {
    const double g = gauss(rng);
    float v = 0.0f;
    if (kind == "drift") v = (float)(0.006 + 0.1 * g);
    else if (kind == "walk") v = (float)(0.1 * g);
    else if (kind == "fall") v = (float)(-3.0 - g * 1e-3);
    else if (kind == "mixed") v = (float)(g * pow(2.0, (double)(rng() % 60) - 30.0));
    else if (kind == "ties") v = (float)((i < 3 ? 1.0 : 0.0) * 0x1p52) + (float)(0.5 * (double)(rng() % 4));
    else if (kind == "whole") v = (float)(rng() % 256);
    else if (kind == "flip") v = i % 2 ? -1.0f : 1.0f;
    else if (kind == "zeros") v = i == n / 2 ? 1.5f : (i % 3 ? 0.0f : -0.0f);
    else if (kind == "tiny") v = (float)(g * 1e-42);
    else if (kind == "huge") v = (float)(g * 1e38);
    else if (kind == "nan") v = i == n / 2 ? NAN : (float)(1.0 + g);
    else if (kind == "inf") v = i == n / 2 ? INFINITY : (float)(1.0 + g);
    else return 2;
    x[i] = v;
  }
  double plain = 0.0;
  for (float v : x) plain += (double)v;

  const size_t runs = (n + kSumRun - 1) / kSumRun;
  auto end_of = [&](size_t c) { return (c + 1) * kSumRun < n ? (c + 1) * kSumRun : n; };
  std::vector<RunOutline> o(runs);
  std::vector<double> sum(runs);
  for (size_t c = 0; c < runs; ++c) {
    o[c] = outline_start();
    for (size_t i = c * kSumRun; i < end_of(c); ++i) outline_add(o[c], x[i]);
  }
  double start = 0.0, most = 0.0;
  for (size_t c = 0; c < runs; ++c) {
    const double s = o[c].sum, lo = fabs(start + o[c].lo), hi = fabs(start + o[c].hi);
    most = most >= lo ? most : lo;
    most = most >= hi ? most : hi;
    sum[c] = s;
    o[c].sum = start;
    start += s;
  }
  double s = 0.0;
  size_t open = 0;
  for (size_t c = 0; c < runs; ++c) {
    double even, odd;
    if (o[c].lo == 0.0 && o[c].hi == 0.0) continue;
    if (run_stand_ins(o[c].sum, o[c].lo, o[c].hi, sum_margin(n, most), even, odd)) {
      double s0 = even, s1 = odd;
      for (size_t i = c * kSumRun; i < end_of(c); ++i) {
        s0 += (double)x[i];
        s1 += (double)x[i];
      }
      s += sum_is_odd(s) ? s1 - odd : s0 - even;
    } else if (run_is_exact(s, run_open(o[c], sum_margin(n, most)).even)) {
      s += sum[c];
    } else {
      ++open;
      for (size_t i = c * kSumRun; i < end_of(c); ++i) s += (double)x[i];
    }
  }
  const bool equal = s == plain || (s != s && plain != plain);
  printf("open %zu equal %d\n", open, equal ? 1 : 0);
  return 0;
}
