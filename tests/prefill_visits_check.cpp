// Host-side replay of what the 4-wave prefill kernels visit (csrc/hi_prefill_visits.h; compiled and run by test_prefill_sweep_cpu.py), from
// the definitions alone: the streams fetch every visit's rows from where they lie and stay inside the buffers, also behind the last visit;
// over its visits a query row sees every key it should exactly once and no other; visits that are taken as seen in full are; a chunk's rows
// enter the store where they belong, and the workgroups that read what they replace are the ones that are counted.
#include <algorithm>
#include <cstdio>
#include <map>
#include <random>
#include <set>
#include <vector>
#include "hi_internal.h"

using namespace hi;

static long checks = 0, bad = 0, rides = 0, waits = 0;
#define CHECK(c) do { ++checks; if (!(c)) { if (++bad < 10) std::printf("line %d: %s\n", __LINE__, #c); } } while (0)

static const char* const kPast = (const char*)(1ll << 40);       // the past segment, or the store
static const char* const kOwn = (const char*)(2ll << 40);

// A stream of the kernels: row r of the present tile lies at rows[r] rows behind w.base.
struct Stream : PfLoads { int64_t rows[64]; };

static void narrow(std::mt19937_64& rng, int i) {
  auto pick = [&](int64_t n) { return (int64_t)(rng() % (uint64_t)n); };
  const int G = 1 << pick(4), strip = prefill_strip(G);
  const int C = 1 + (int)pick(i % 2 ? 200 : 900), past = i % 5 == 0 ? 0 : 1 + (int)pick(1200);
  const int split = i % 3 == 0 ? 1 : 1 + (int)pick(6);
  const int launches = past > 0 ? 1 + (int)pick(3) : 1;
  const int past_tiles = (past + 63) / 64, blocks = (C + strip - 1) / strip;
  const int bx = (int)pick(blocks), own = (std::min(C, bx * strip + strip) + 63) / 64;
  // what each query row of the block has seen, over ranges and launches
  std::map<int, std::vector<int>> seen;
  for (int k = 0; k < split; ++k) {
    int tile0 = 0;
    for (int l = 0; l < launches; ++l) {
      const int last = l == launches - 1, left = past_tiles - tile0;
      const int tiles = last ? left : std::min(left, (int)pick(left + 1));
      const int na = std::max(0, std::min(past - 64 * tile0, 64 * tiles)), nb = last ? C : 0;
      if (na + nb == 0) { tile0 += tiles; continue; }
      const int jump = split > 1 && tiles > 1 && pick(2) ? 1 + (int)pick(tiles - 1) : 0;
      const int64_t far = jump ? 256 * (1 + pick(1000)) : 0;
      PfNarrow n;
      n.na = na; n.nb = nb; n.a0 = n.b0 = 0; n.jump_tile = jump; n.jump_bytes = far;
      if (split > 1) {
        const PfRange r = pf_narrow_range(past_tiles, own, k, split, tile0, tiles, last);
        if (r.lo >= r.hi) { tile0 += tiles; continue; }
        n.a0 = r.lo - tile0;
        n.b0 = r.lo > past_tiles ? r.lo - past_tiles : 0;
        n.ta = std::max((r.hi < past_tiles ? r.hi : past_tiles) - r.lo, 0);
        n.T = r.hi - r.lo;
      } else {
        n.ta = (na + 63) / 64;
        n.T = n.ta + (std::min(nb, bx * strip + strip) + 63) / 64;
      }
      CHECK(n.T >= 1);
      Stream w;
      w.v = w.usual = 0;
      auto meet = [&]() {
        int rows;
        if (pf_narrow_meet(w, n, kPast, kOwn, rows))
          for (int r = 0; r < 64; ++r) w.rows[r] = r < rows ? r : rows - 1;
      };
      meet();
      for (int v = 0; v < n.T + 2; ++v) {        // the K stream runs two visits ahead
        const int at = v < n.T ? v : n.T - 1;
        const bool in_b = at >= n.ta;
        const int tile = in_b ? n.b0 + at - n.ta : n.a0 + at, seg = in_b ? nb : na;
        for (int r = 0; r < 64; ++r) {
          const char* const p = w.base + 256 * w.rows[r];
          if (v < n.T) {
            const int row = std::min(64 * tile + r, seg - 1);
            CHECK(p == (in_b ? kOwn : kPast) + 256ll * row + (!in_b && jump && tile >= jump ? far : 0));
          } else {                               // any rows that are there
            const int64_t o = p - (p >= kOwn ? kOwn : kPast), edge = 16384ll * jump;
            CHECK(p >= kOwn ? o >= 0 && o + 256 <= 256ll * nb
                            : o >= 0 && (!jump ? o + 256 <= 256ll * na : o + 256 <= edge || (o >= edge + far && o - far + 256 <= 256ll * na)));
          }
        }
        if (v < n.T)
          for (int wave = 0; wave < strip / 32; ++wave) {
            const int i0 = bx * strip + 32 * wave;
            const PfOpen open = pf_narrow_open(n, i0);
            const bool masked = !(v < open.a || (v >= n.ta && v < open.b));
            for (int q = i0; q < i0 + 32; ++q) {
              const uint64_t bits = masked ? pf_narrow_seen(n, v, q) : ~0ull;
              if (!masked) CHECK(pf_narrow_seen(n, v, q) == ~0ull);
              for (int r = 0; r < 64; ++r)
                if (bits >> r & 1) seen[q].push_back(in_b ? past + 64 * tile + r : 64 * (tile0 + tile) + r);
            }
          }
        if (pf_loads_next(w, n.T)) meet();
      }
      tile0 += tiles;
    }
  }
  for (int q = bx * strip; q < std::min(C, bx * strip + strip); ++q) {
    std::vector<int>& s = seen[q];
    std::sort(s.begin(), s.end());
    CHECK((int)s.size() == past + q + 1);
    for (int j = 0; j < (int)s.size(); ++j) if (s[j] != j) { CHECK(s[j] == j); break; }
  }
}

static void window(std::mt19937_64& rng, int i) {
  auto pick = [&](int64_t n) { return (int64_t)(rng() % (uint64_t)n); };
  const int G = 1 << pick(4), strip = prefill_strip(G);
  const int sink = i % 4 == 0 ? 0 : i % 4 == 1 ? 64 * (int)pick(4) : (int)pick(300);
  const int recent = 1 + (int)pick(i % 3 ? 150 : 1500);
  const int C = 1 + (int)pick(i % 2 ? 300 : 1500);
  const int64_t P = i % 6 == 0 ? 0 : i % 6 == 1 ? pick(sink + 2) : i % 6 == 2 ? sink + pick(recent + 2) : pick(4000);
  const int store_rows = sink + recent;
  auto place = [&](int64_t token) { return token < sink ? token : sink + (token - sink) % recent; };
  // the store as a program leaves it: which token is in which row
  std::vector<int64_t> store(store_rows, -1);
  for (int64_t t = 0; t < P; ++t)
    if (t < sink || t >= P - recent) store[place(t)] = t;
  const PfWindow a = pf_window_of(P, C, sink, recent);
  PrefillWindowUpdate u;
  const int heads = 1 + (int)pick(40);
  const bool ride = window_update(G, C, P, sink, recent, heads, &u);
  const PfStoreRows& rows = u.rows;
  const int strips = (C + strip - 1) / strip;
  // the rows the chunk puts into the store, and what the store then holds
  std::map<int, int64_t> put;
  for (int64_t t = P; t < P + C; ++t)
    if (t < sink || t >= P + C - recent) put[(int)place(t)] = t;
  std::set<int> replaced;                        // rows that held something
  for (auto& e : put) if (store[e.first] >= 0) replaced.insert(e.first);
  long n_put = 0;
  for (int c = 0; c < C; ++c) {
    if (!(c < rows.cs || (c >= rows.u0 && c < rows.u0 + rows.cr))) continue;
    const auto it = put.find(pf_store_row(rows, sink, recent, c));
    CHECK(it != put.end() && it->second == P + c);
    ++n_put;
  }
  CHECK(n_put == (long)put.size() && n_put == rows.cs + rows.cr);
  const auto ordered = [&](int s) { return s < 3 || s >= strips - 2 || s % 5 == 0; };
  int last_reader = -1;
  for (int s = 0; s < strips; ++s) {
    const int i_lo = s * strip, i_hi = i_lo + strip - 1;
    const PfWindowTiles t = pf_window_tiles(a, i_lo, i_hi);
    CHECK(t.T >= 1);
    const bool in_full = ordered(s);
    Stream w;
    w.v = w.usual = 0;
    auto meet = [&]() {
      int n, row0;
      if (!pf_window_meet(w, a, t, kPast, kOwn, n, row0)) return;
      for (int r = 0; r < 64; ++r) w.rows[r] = n ? (r < n ? r : n - 1) : pf_window_row(a, std::min(row0 + r, a.ns + a.m - 1));
    };
    meet();
    std::map<int, std::vector<int64_t>> seen;
    for (int v = 0; v < t.T + 2; ++v) {
      for (int r = 0; r < 64; ++r) {
        const char* const p = w.base + 256 * w.rows[r];
        const bool own = p >= kOwn;
        const int64_t o = p - (own ? kOwn : kPast);
        CHECK(o >= 0 && o % 256 == 0 && o / 256 < (own ? C : store_rows));
        if (!own && replaced.count((int)(o / 256))) last_reader = s;
      }
      if (v < t.T) {
        bool in_b;
        const int j0 = pf_window_locate(t, v, in_b) * 64;
        for (int wave = 0; wave < strip / 32 && in_full; ++wave) {
          const int i0 = i_lo + 32 * wave;
          const PfSeenVisits open = pf_window_open(a, t, i0);
          const bool masked = !((uint32_t)(v - open.first) < (uint32_t)open.n) && !pf_window_full(a, in_b, j0, i0);
          for (int q = i0; q < i0 + 32; ++q) {
            const uint64_t bits = pf_window_seen(a, in_b, j0, q);
            if (!masked && q < C) CHECK(bits == ~0ull);
            for (int r = 0; r < 64; ++r) {
              if (!(bits >> r & 1)) continue;
              const int64_t at = (w.base + 256 * w.rows[r] - (in_b ? kOwn : kPast)) / 256;
              CHECK(in_b ? at < C : at < store_rows);
              seen[q].push_back(in_b ? P + at : store[at]);
            }
          }
        }
      }
      if (pf_loads_next(w, t.T)) meet();
    }
    for (int q = i_lo; q <= i_hi && q < C && in_full; ++q) {
      std::vector<int64_t> want, &got = seen[q];
      for (int64_t j = 0; j <= P + q; ++j)
        if (j < sink || P + q - j < recent) want.push_back(j);
      std::sort(got.begin(), got.end());
      CHECK(got == want);
    }
  }
  CHECK(last_reader < rows.readers);             // nobody reads a row behind the workgroups that are counted
  const long workgroups = (long)strips * (G == 8 ? 2 : 1) * heads;
  CHECK(ride == (rows.readers == 0 || (2 * rows.readers <= strips && rows.cs + rows.cr <= (workgroups > 1024 ? 512 : 256))));
  if (ride && rows.readers > 0) ++rides;
  if (!ride) ++waits;
}

int main() {
  std::mt19937_64 rng(5);
  for (int i = 0; i < 12000; ++i) narrow(rng, i);
  for (int i = 0; i < 1500; ++i) window(rng, i);
  CHECK(rides > 200 && waits > 200);
  // the rule's edges: half of the strips, one row more than 256 and 512, one strip more than 1024 workgroups
  PrefillWindowUpdate u;
  CHECK(window_update(4, 192, 4000, 64, 65, 1, &u) && u.rows.readers == 2 && window_update(4, 160, 4000, 64, 65, 1, &u));
  CHECK(!window_update(4, 96, 4000, 64, 65, 1, &u) && u.rows.readers == 2);
  CHECK(window_update(4, 5000, 9000, 0, 256, 1, &u) && u.rows.readers > 0 && !window_update(4, 5000, 9000, 0, 257, 1, &u));
  CHECK(!window_update(4, 8192, 9000, 0, 512, 4, &u) && window_update(4, 8193, 9000, 0, 512, 4, &u) && !window_update(4, 8193, 9000, 0, 513, 4, &u));
  CHECK(window_update(4, 5000, 0, 0, 4000, 1, &u) && u.rows.readers == 0);
  std::printf("%ld checks, %ld rides, %ld launches of their own, %ld failures\n", checks, rides, waits, bad);
  return bad != 0;
}
