// Host-side check of prefill_unit_shape (compiled and run by test_prefill_unit_shape.py): the launches of a unit with
// the split and pairing chosen for it are replayed on sets of tile ids, as partition_check.cpp does for the default
// shape - every block of positions must have seen each of its tiles exactly once, no image may lie outside the
// capacity, and the closed form of pf_contributors must agree with counting.
#include <algorithm>
#include <cstdio>
#include <set>
#include <vector>
#include "hi_internal.h"
#include "hi_prefill_part.h"

using namespace hi;

static long fails = 0;
#define CHECK(cond, ...) do { if (!(cond)) { if (fails < 20) { printf("FAIL %s:%d: ", __FILE__, __LINE__); printf(__VA_ARGS__); printf("\n"); } ++fails; } } while (0)

struct Image { int block = -1; std::multiset<long> tiles; };

// Units of the 4-wave kernel: the ranges of every block, swept launch by launch, are the ranges of one launch over everything,
// each swept in order; a range loads its image exactly where an earlier launch has begun it; no image lies beyond the row.
static long narrow = 0, narrow_most = 0;
static void run_narrow(int G, int C, int nh, int variant, long past, long slice, long capacity, int all_heads) {
  const PrefillLaunch unit = prefill_unit_shape(G, C, nh, variant, past, slice, capacity, all_heads);
  if (unit.deep || unit.split == 1) return;
  ++narrow;
  if (unit.split > narrow_most) narrow_most = unit.split;
  const int strip = prefill_strip(G), blocks = (int)ceil_div(C, strip), rows = prefill_grid_y(G) * nh;
  CHECK(unit.carry_bytes <= capacity && unit.carry_bytes == (long)rows * blocks * unit.split * kWgThreads * kCarryFloatsPerLane * 4, "images");
  CHECK(unit.img_row == blocks * unit.split && unit.merge && unit.past_tiles == (past + 63) / 64, "shape");
  for (int h = 1; h <= all_heads; ++h)
    for (long sl : {0L, 64L, 1024L}) {
      const PrefillLaunch other = prefill_unit_shape(G, C, h, variant, past, sl, capacity, all_heads);
      CHECK(prefill_launch_shape(G, C, h, variant, 1, 1).deep || other.split == unit.split, "split of %d heads: %d, not %d", h, other.split, unit.split);
    }
  std::vector<std::vector<int>> swept(unit.img_row);
  const int launches = slice > 0 ? (int)ceil_div(past, slice) : 1;
  for (int l = 0; l < launches; ++l) {
    const int last = l == launches - 1, tile0 = launches == 1 ? 0 : (int)(l * slice / 64);
    const long na = launches == 1 ? past : (past - l * slice < slice ? past - l * slice : slice);
    const PrefillLaunch pl = prefill_launch_of(unit, last, last);
    CHECK(pl.merge == last && pl.split == unit.split && pl.img_row == unit.img_row, "launch");
    std::set<int> numbers;
    for (int x = 0; x < unit.img_row; ++x) {
      const int w = pf_wg_index(x, unit.img_row, pl.xcd), k = w / blocks, bx = blocks - 1 - w % blocks;
      CHECK(w >= 0 && w < unit.img_row && numbers.insert(w).second, "workgroup number");
      const int own = ((C < (bx + 1) * strip ? C : (bx + 1) * strip) + 63) / 64;
      const PfRange r = pf_narrow_range(unit.past_tiles, own, k, unit.split, tile0, (int)((na + 63) / 64), last);
      if (r.lo >= r.hi) continue;
      std::vector<int>& seq = swept[k * blocks + bx];
      CHECK(r.fresh == (int)seq.empty(), "range %d of block %d: fresh %d after %zu tiles", k, bx, r.fresh, seq.size());
      CHECK(r.lo >= tile0 && (r.hi <= tile0 + (na + 63) / 64 || last), "tiles outside the launch");
      for (int t = r.lo; t < r.hi; ++t) seq.push_back(t);
    }
  }
  for (int bx = 0; bx < blocks; ++bx) {
    const int own = ((C < (bx + 1) * strip ? C : (bx + 1) * strip) + 63) / 64;
    int at = 0;
    for (int k = 0; k < unit.split; ++k) {
      const PfRange whole = pf_narrow_range(unit.past_tiles, own, k, unit.split, 0, unit.past_tiles, 1);
      const std::vector<int>& seq = swept[k * blocks + bx];
      CHECK(whole.fresh && whole.lo == at && whole.hi > whole.lo && (int)seq.size() == whole.hi - whole.lo, "range %d of block %d", k, bx);
      for (size_t i = 0; i < seq.size(); ++i) CHECK(seq[i] == whole.lo + (int)i, "order");
      at = whole.hi;
    }
    CHECK(at == unit.past_tiles + own, "block %d ends at tile %d of %d", bx, at, unit.past_tiles + own);
  }
}

static void run_unit(int G, int C, int nh, int variant, long past, long slice, long capacity, int* split_out) {
  const PrefillLaunch unit = prefill_unit_shape(G, C, nh, variant, past, slice, capacity);
  const PrefillLaunch base = prefill_launch_shape(G, C, nh, variant, 1, 1);
  CHECK(unit.carry_bytes <= capacity || unit.carry_bytes == base.carry_bytes, "capacity");
  *split_out = unit.split;
  if (!unit.deep) return;
  const int m = 2 * prefill_strip(G) / 64, launches = past > 0 && slice > 0 ? (int)ceil_div(past, slice) : 1;
  std::vector<Image> img(unit.img_row);
  std::vector<std::multiset<long>> out(unit.nbk);
  std::vector<int> written(unit.nbk, 0);
  PfShape sh{};
  for (int l = 0; l < launches; ++l) {
    const int last = l == launches - 1;
    const PrefillLaunch pl = prefill_launch_of(unit, last, last);
    const long na = launches == 1 ? past : (past - l * slice < slice ? past - l * slice : slice);
    sh.nbk = pl.nbk; sh.m = m; sh.ta = (int)((na + 63) / 64); sh.tb_all = last ? (C + 63) / 64 : 0;
    sh.split = pl.split; sh.paired = pl.paired; sh.carried = l > 0;
    const int n = pl.nbk * pl.split;
    std::vector<Image> next = img;
    std::set<int> numbers, stored;
    for (int x = 0; x < n; ++x) {
      const int w = pf_wg_index(x, n, pl.xcd);
      CHECK(w >= 0 && w < n && numbers.insert(w).second, "workgroup number %d of %d", w, n);
      for (int which = 0; which < 2; ++which) {
        const PfPass ps = pf_pass(sh, w, which, last);
        if (ps.init || (ps.run && ps.store >= 0)) {
          CHECK(ps.store >= 0 && ps.store < unit.img_row && stored.insert(ps.store).second, "store to image %d of %d", ps.store, unit.img_row);
          if (ps.store < 0 || ps.store >= unit.img_row) return;
          next[ps.store] = Image();
          next[ps.store].block = ps.bx;
        }
        if (!ps.run) continue;
        std::multiset<long> acc;
        if (ps.load >= 0) {
          CHECK(ps.load < unit.img_row && img[ps.load].block == ps.bx && (ps.load == ps.store || ps.store < 0), "load of image %d", ps.load);
          if (ps.load < unit.img_row) acc = img[ps.load].tiles;
        }
        for (int t = ps.a0; t < ps.a1; ++t) acc.insert(1000000L * (l + 1) + t);
        for (int t = ps.b0; t < ps.b1; ++t) acc.insert(t);
        if (ps.store >= 0) next[ps.store].tiles = acc;
        else { CHECK(last && !written[ps.bx]++, "block %d written early or twice", ps.bx); out[ps.bx] = acc; }
      }
    }
    img = next;
  }
  for (int b = 0; b < unit.nbk; ++b) {
    int n_e, n_x;
    pf_block_images(sh, b, n_e, n_x);
    const bool direct = n_e + n_x == 1 && unit.split == 1;
    CHECK(direct == (written[b] > 0), "block %d", b);
    CHECK(direct || unit.merge, "no merge");
    for (int i = 0; !direct && i < n_e + n_x; ++i) {
      const int id = i < n_e ? pf_image_e(sh, b, i) : pf_image_x(sh, b, i - n_e);
      CHECK(id < unit.img_row && img[id].block == b, "merge of block %d reads image %d", b, id);
      if (id < unit.img_row) out[b].insert(img[id].tiles.begin(), img[id].tiles.end());
    }
    std::multiset<long> want;
    for (int l = 0; l < launches; ++l) {
      const long na = launches == 1 ? past : (past - l * slice < slice ? past - l * slice : slice);
      for (long t = 0; t < (na + 63) / 64; ++t) want.insert(1000000L * (l + 1) + t);
    }
    const long end = std::min<long>((long)(b + 1) * 64 * m, C);        // the block's rows see own tiles up to that of its last row
    for (int t = 0; t < (end + 63) / 64; ++t) want.insert(t);
    CHECK(out[b] == want, "block %d of G=%d C=%d nh=%d variant=%d past=%ld slice=%ld split=%d paired=%d", b, G, C, nh, variant, past, slice, unit.split, unit.paired);
  }
}

int main() {
  long cases = 0, uneven = 0, most = 0;
  for (int G : {1, 2, 4, 8}) for (int C : {1, 33, 64, 77, 129, 600, 1500, 2400}) for (int nh : {1, 3, 8}) for (int variant : {0, 3, 4, 8, 1})
    for (long past : {0L, 1L, 100L, 3001L, 20000L}) for (long slice : {0L, 512L, 4096L}) for (long extra : {0L, 60L << 20}) {
      if ((long)C * nh > 8000) continue;
      int split = 0;
      run_unit(G, C, nh, variant, past, slice, prefill_carry_bound(G, C, nh) + extra, &split);
      ++cases;
      if (split & (split - 1)) ++uneven;
      if (split > most) most = split;
    }
  CHECK(uneven > 0 && most > 8, "splits that are no power of two: %ld, largest %ld", uneven, most);
  for (int G : {1, 2, 4, 8}) for (int C : {1, 33, 64, 77, 300, 512, 960}) for (int nh : {1, 2, 8}) for (int variant : {0, 4, 8, 64})
    for (long past : {0L, 100L, 1536L, 2049L, 3001L, 20000L, 131072L, 1000003L}) for (long slice : {0L, 512L, 4096L, 65536L}) for (long room : {1L, 8L, 64L})
      run_narrow(G, C, nh, variant, past, slice, prefill_carry_bound(G, C, 8) + room * (1L << 20), 8);
  CHECK(narrow > 1000 && narrow_most > 40, "%ld units of the 4-wave kernel cut, into %ld at most", narrow, narrow_most);
  // launches whose workgroups sweep 640 tiles and more run the wide form, also where the chunk does not fill its last block
  struct { int G, C, nh; long past; } longs[] = {{1, 1300, 32, 60000}, {1, 2100, 32, 300000}, {1, 3590, 32, 200000}, {4, 77, 8, 1000000}, {1, 200, 32, 1 << 20}};
  for (const auto& u : longs) {
    const PrefillLaunch pl = prefill_unit_shape(u.G, u.C, u.nh, 0, u.past, 0, 1L << 40, u.nh);
    CHECK(pl.deep && prefill_is_wide(0, pl.split, u.past + u.C), "%d rows behind %ld: split %d", u.C, u.past, pl.split);
    CHECK(!prefill_is_wide(0, pl.split, 640L * 64 * pl.split - 1) && !prefill_is_wide(16, 1, 1L << 30) && !prefill_is_wide(64, 1, 1L << 30) &&
          prefill_is_wide(128, pl.split, 64), "rule");
  }
  // the units of test_gpu_prefill_sweep.py that have a merge launch, and those that have none, whatever room they find
  struct { int G, H, nh; long past; int C, merge; } merged[] = {{1, 17, 16, 3000, 150, 1}, {4, 8, 8, 3001, 77, 1}, {8, 9, 7, 1500, 130, 1}, {4, 3, 1, 4000, 33, 1},
                                                                {1, 2, 2, 2500, 1, 1}, {4, 8, 8, 64, 1000, 0}, {1, 5, 3, 100, 40, 0}};
  for (const auto& u : merged) for (long room : {0L, 1L << 40})
    CHECK(prefill_unit_shape(u.G, u.C, u.nh, 0, u.past, 0, prefill_carry_bound(u.G, u.C, u.H) + room, u.H).merge == u.merge, "%d rows behind %ld: merge", u.C, u.past);
  for (int nbk : {2, 3, 7, 10}) for (int m : {1, 2, 4}) for (int ta : {0, 1, 5, 47, 200}) for (int split : {1, 2, 3, 5, 11, 40}) for (int clip : {0, 1}) {
    PfShape s{nbk, m, ta, nbk * m - clip, split, 1, 0};
    for (int p = 0; p < nbk / 2; ++p) for (int sw = 0; sw < 2; ++sw) {
      const int deep = nbk - 1 - p, nr = 2 * split, Td = ta + pf_own_tiles(s, deep), L = Td + ta + pf_own_tiles(s, p);
      int seen = 0;
      for (int k = 0; k <= nr; ++k) {
        int before, total, all = 0;
        for (int kk = 0; kk < nr; ++kk) {
          const int x0 = (int)((long)L * kk / nr), x1 = (int)((long)L * (kk + 1) / nr);
          all += x1 > x0 && (sw ? x1 > Td : x0 < Td);
        }
        if (k == nr) break;
        pf_contributors(s, deep, p, nr, sw, k, before, total);
        CHECK(total == all && before == seen, "contributors nbk=%d m=%d ta=%d split=%d k=%d: %d/%d, counted %d/%d", nbk, m, ta, split, k, before, total, seen, all);
        const int x0 = (int)((long)L * k / nr), x1 = (int)((long)L * (k + 1) / nr);
        seen += x1 > x0 && (sw ? x1 > Td : x0 < Td);
      }
    }
  }
  printf("%ld units replayed, %ld failures, %ld with a split that is no power of two, largest split %ld\n", cases, fails, uneven, most);
  return fails ? 1 : 0;
}
