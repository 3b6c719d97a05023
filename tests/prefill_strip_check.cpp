// Host-side check of blocks of positions of one height (PrefillLaunch::strip; compiled and run by test_prefill_strip_cpu.py): such a
// unit has no launch that runs the wide form, its blocks cover the chunk, each has a row, and over the unit's launches every
// block sweeps the past tiles and its own ones up to that of its last row exactly once.
#include <cstdio>
#include <set>
#include <vector>
#include "hi_internal.h"
#include "hi_prefill_part.h"

using namespace hi;

static long fails = 0, units = 0;
#define CHECK(cond, ...) do { if (!(cond)) { if (fails < 20) { printf("FAIL %d: ", __LINE__); printf(__VA_ARGS__); printf("\n"); } ++fails; } } while (0)

static void run(int G, int C, int nh, int variant, long past, long slice) {
  const PrefillLaunch unit = prefill_unit_shape(G, C, nh, variant, past, slice, 1L << 33, nh);
  if (!unit.deep || unit.strip == 0) return;
  ++units;
  const int full = 2 * prefill_strip(G);
  CHECK(!(variant & (16 | 128)) && !prefill_is_wide(variant, unit.split, past + C), "a form that takes full blocks");
  CHECK(unit.strip % 16 == 0 && unit.strip < full && (long)unit.nbk * unit.strip >= C && (long)(unit.nbk - 1) * unit.strip < C &&
        unit.nbk == ceil_div(C, full), "%d blocks of %d for %d rows", unit.nbk, unit.strip, C);
  std::vector<std::multiset<long>> seen(unit.nbk), want(unit.nbk);
  const int launches = past > 0 && slice > 0 ? (int)ceil_div(past, slice) : 1;
  for (int l = 0; l < launches; ++l) {
    const int last = l == launches - 1;
    const long na = launches == 1 ? past : (past - l * slice < slice ? past - l * slice : slice);
    const PrefillLaunch pl = prefill_launch_of(unit, last, last);
    CHECK(pl.strip == unit.strip, "one height for the unit");
    PfShape s;
    s.nbk = pl.nbk; s.m = pl.strip / 64; s.strip = pl.strip; s.split = pl.split; s.paired = pl.paired; s.carried = l > 0;
    s.ta = (int)((na + 63) / 64); s.tb_all = last ? (C + 63) / 64 : 0;
    for (int w = 0; w < pl.nbk * pl.split; ++w)
      for (int which = 0; which < 2; ++which) {
        const PfPass p = pf_pass(s, w, which, last);
        if (!p.run) continue;
        for (int t = p.a0; t < p.a1; ++t) seen[p.bx].insert(1000000L * (l + 1) + t);
        for (int t = p.b0; t < p.b1; ++t) seen[p.bx].insert(t);
      }
    for (int b = 0; b < pl.nbk; ++b) {
      for (int t = 0; t < s.ta; ++t) want[b].insert(1000000L * (l + 1) + t);
      const long end = (long)(b + 1) * unit.strip < C ? (long)(b + 1) * unit.strip : C;
      for (long t = 0; last && t < (end + 63) / 64; ++t) want[b].insert(t);
    }
  }
  for (int b = 0; b < unit.nbk; ++b) CHECK(seen[b] == want[b], "block %d of G=%d C=%d nh=%d past=%ld slice=%ld", b, G, C, nh, past, slice);
}

int main() {
  for (int G : {1, 2, 4, 8}) for (int C : {65, 77, 96, 129, 140, 150, 257, 300, 333, 520, 700, 1100, 1300, 2500}) for (int nh : {1, 2, 8, 32})
    for (int variant : {0, 3, 4, 8, 16, 64, 128, 3 + 8}) for (long past : {0L, 100L, 3001L, 20000L, 100003L, 1000000L}) for (long slice : {0L, 1024L, 32768L})
      run(G, C, nh, variant, past, slice);
  CHECK(units > 500, "%ld units", units);
  printf("%ld units, %ld failures\n", units, fails);
  return fails != 0;
}
