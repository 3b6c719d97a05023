// Host-side check of decode_cut (compiled and run by test_decode_cut.py): whatever the lengths, every head has a partition,
// the table of first workgroups adds up, the number of workgroups stays within the limit where the heads leave room for it,
// partitions hold at least 64 rows, and together they cover every row.
#include <cstdio>
#include <cstdlib>
#include "hi_internal.h"

using namespace hi;

int main() {
  long fails = 0, proportional = 0, same = 0;
  srand(1);
  for (int it = 0; it < 200000; ++it) {
    const int nh = 1 + rand() % kDecodeMaxRagged, max_wgs = rand() % 3 == 0 ? 1 + rand() % 300 : 256;
    DecodeLens lens = {};
    const int64_t top = 1LL << (rand() % 22);
    int64_t longest = 0;
    for (int j = 0; j < nh; ++j) {
      lens.n[j] = rand() % 4 == 0 ? 0 : (uint32_t)((rand() * 32768LL + rand()) % top);
      if (lens.n[j] > longest) longest = lens.n[j];
    }
    int most = 0;
    const int wgs = decode_cut(lens, nh, max_wgs, &most);
    if (lens.rows_per_wg == 0) {
      ++same;
      if (wgs != most * nh || most < 1 || (most > 1 && (wgs > max_wgs || (int64_t)(most - 1) * 64 >= longest))) ++fails;
      continue;
    }
    ++proportional;
    int sum = 0, largest = 0;
    for (int j = 0; j < nh; ++j) {
      const int p = decode_parts(lens.n[j], lens.rows_per_wg);
      if (lens.first[j] != sum || p < 1 || (int64_t)p * lens.rows_per_wg < lens.n[j]) ++fails;
      sum += p;
      if (p > largest) largest = p;
    }
    for (int j = nh; j < kDecodeMaxRagged; ++j) fails += lens.first[j] != 0xffff;
    if (sum != wgs || largest != most || lens.rows_per_wg < 64 || (wgs > max_wgs && max_wgs >= 2 * nh)) ++fails;
  }
  printf("%ld failures, %ld cut in proportion, %ld alike\n", fails, proportional, same);
  return fails || !proportional || !same;
}
