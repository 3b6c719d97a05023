// The kernels divide by multiplication (pf_magic, pf_div): every quotient of the range it is declared exact for, and the
// passes of random launches, against the compiler's division.
#include <cstdio>
#include <cstring>
#include <random>
#include "hi_prefill_part.h"

using namespace hi;

int main() {
  long checks = 0, bad = 0;
  for (uint32_t d = 1; d <= 4096; ++d) {
    const uint32_t x_max = (uint32_t)(((1ull << 32) - 1) / d);
    const uint32_t magic = pf_magic(d, x_max);
    bad += pf_magic(d, (1ull << 32) / d + 1) != 0 || (d > 1 && (uint64_t)x_max * d < (1ull << 32) && !magic);
    for (uint32_t q = x_max / d, i = 0; i < 600; ++i, q = i < 300 ? q - 1 : (i - 300) * 7u)
      for (int e = -1; e <= 1; ++e) {
        const uint64_t x = (uint64_t)q * d + e;
        if (x > x_max) continue;
        ++checks;
        bad += pf_div((uint32_t)x, d, magic) != (uint32_t)x / d;
      }
  }
  std::mt19937 rng(7);
  for (int i = 0; i < 20000; ++i) {
    PfShape s;
    s.split = 1 + (int)(rng() % 64);
    s.nbk = 1 + (int)(rng() % (i & 1 ? 12 : 300));
    s.m = 1 << (rng() % 3);
    s.ta = (int)(rng() % (i % 3 ? 300 : 70000));
    s.tb_all = rng() % 4 ? s.nbk * s.m - (int)(rng() % s.m) : 0;
    s.paired = s.tb_all > 0 && s.nbk >= 2 && rng() % 2;
    s.carried = (int)(rng() % 2);
    PfShape t = s;
    t.by_split = pf_magic((uint32_t)s.split, pf_largest_cut(s));
    t.by_nbk = pf_magic((uint32_t)s.nbk, (uint64_t)s.nbk * s.split);
    for (int j = 0; j < 20; ++j) {
      const int w = (int)(rng() % (unsigned)(s.nbk * s.split));
      for (int which = 0; which < 2; ++which) {
        const PfPass a = pf_pass(s, w, which, 1), b = pf_pass(t, w, which, 1);
        ++checks;
        bad += std::memcmp(&a, &b, sizeof(a)) != 0;
      }
    }
  }
  std::printf("%ld checks, %ld failures\n", checks, bad);
  return bad != 0;
}
