// Host-side check of the rotary angles of a run (csrc/hi_rope.h; compiled and run by test_rope_cpu.py): their fp32 values against those of
// a sincos per position, over positions from 0 to 2^33.
#include <cstdio>
#include <initializer_list>
#include "hi_rope.h"

using namespace hi;

int main() {
  long fails = 0, all = 0;
  for (int64_t from : {0L, 4001L, 131072L, 999983L, 4000000L, 100000001L, 2147483000L, 8589000000L}) {
    long values = 0, differ = 0;
    double worst = 0.0;
    for (double theta : {10000.0, 500000.0})
      for (int i = 0; i < 64; ++i) {
        const double w = pow(theta, -(double)i / 64.0);
        for (int64_t first = from; first < from + 100 * 33; first += 33) {
          RopeRun run(first, w);
          for (int k = 0; k < kRopeRun; ++k) {
            float c, s;
            run.next(c, s);
            double S, C;
            sincos((double)(first + k) * w, &S, &C);
            values += 2;
            differ += (c != (float)C) + (s != (float)S);
            const double x = fabs(c - C), y = fabs(s - S);
            worst = x > worst ? x : worst;
            worst = y > worst ? y : worst;
          }
        }
      }
    // One rounding to fp32: half an ulp of values up to 1, 2^-25.  Values differ only where the middle between two fp32 values lies inside
    // the run's error, 31 products of 1.1e-16: 3.5e-15 / 2^-24 or 6e-8 of them, 0.05 of these 819200 (5 are less likely than 1e-8).
    // Steps of w alone differ in 46 of them at 131 thousand positions, in 270 at a million.
    const bool ok = worst <= 3.0e-8 && differ <= 4;
    if (!ok) ++fails;
    printf("%ld: %ld of %ld differ, worst %.3g%s\n", (long)from, differ, values, worst, ok ? "" : " FAIL");
    all += values;
  }
  printf("%ld values, %ld failures\n", all, fails);
  return fails != 0;
}
