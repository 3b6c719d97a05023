// The loads of prefill_kernel_deep16, replayed pass by pass (csrc/hi_prefill_part.h): the tiles that a pass asks for ahead are
// the right ones, and no load - nor the ones behind a pass's last tile - leaves the rows that the launch was given.  And its
// runs of steady tiles: all other tiles take their maxima.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
#include "hi_prefill_part.h"

using namespace hi;

static long checks = 0, bad = 0, runs = 0;
#define CHECK(c) do { ++checks; if (!(c)) { if (++bad < 10) std::printf("line %d: %s\n", __LINE__, #c); } } while (0)

int main() {
  std::mt19937_64 rng(11);
  auto pick = [&](int64_t n) { return (int64_t)(rng() % (uint64_t)n); };
  for (int i = 0; i < 30000; ++i) {
    PfShape s;
    s.split = 1 + (int)pick(i % 3 ? 5 : 64);
    s.m = 1 << pick(3);
    const int64_t nb = i % 5 == 0 ? 0 : 1 + pick(i % 2 ? 700 : 3000);
    const int64_t na = nb == 0 ? 1 + pick(4000) : (i % 7 ? pick(4000) : 0);
    const int64_t C = nb ? nb : 1 + pick(1000);
    s.nbk = (int)((C + 64 * s.m - 1) / (64 * s.m));
    s.ta = (int)((na + 63) / 64);
    s.tb_all = (int)((nb + 63) / 64);
    s.paired = nb > 0 && s.nbk >= 2 && pick(2);
    s.carried = 0;
    const int jump = na > 128 && pick(3) == 0 ? 1 + (int)pick((na - 1) / 64) : 0;
    // the past rows in one or two pieces, and the own rows, far apart
    const char* const past = (const char*)(1ll << 40);
    const char* const own = (const char*)(2ll << 40);
    const int64_t far = jump ? 256 * pick(100000) + 256 : 0;
    auto inside = [&](const char* p, int64_t rows) {
      if (p >= own) return p + rows * 256 <= own + nb * 256;
      const int64_t at = p - past, edge = jump ? 16384ll * jump : na * 256;
      if (at < 0) return false;
      if (at < edge) return at + rows * 256 <= edge && at + rows * 256 <= na * 256;
      return jump && at >= edge + far && at - far + rows * 256 <= na * 256;
    };
    for (int b = 0; b < s.nbk && nb; ++b) {             // a block's last row sees the chunk's rows up to itself
      const int64_t last = std::min<int64_t>((b + 1) * 64 * s.m, C) - 1;
      CHECK(pf_own_tiles(s, b) == (int)(last / 64) + 1);
    }
    for (int j = 0; j < 6; ++j) {
      const int w = (int)pick((int64_t)s.nbk * s.split);
      for (int which = 0; which < 2; ++which) {
        const PfPass ps = pf_pass(s, w, which, 1);
        if (!ps.run) continue;
        PfSweep sw;
        const char* const p0 = past + pf_sweep_of(sw, ps, na, nb, jump, far);
        CHECK(sw.T == ps.a1 - ps.a0 + ps.b1 - ps.b0 && sw.T >= 1);
        auto where = [&](int t) -> const char* {           // first row of sweep tile t, from the pass's own numbers
          if (t >= ps.a1 - ps.a0) return own + 16384ll * (ps.b0 + t - (ps.a1 - ps.a0));
          const int tile = ps.a0 + t;
          return past + 16384ll * tile + (jump && tile >= jump ? far : 0);
        };
        for (int t = 0; t < sw.T; ++t) {
          CHECK((t >= sw.ta ? own : p0) + pf_tile_offset(sw, t) == where(t));
          CHECK(pf_tile_rows(sw, t) >= 1 && inside(where(t), pf_tile_rows(sw, t)));
          CHECK(pf_tile_rows(sw, t) == 64 || !inside(where(t), pf_tile_rows(sw, t) + 1));
        }
        // tiles that need no maximum, searched tile by tile: groups of four in runs over the past (up to a jump, and from two
        // tiles before it on) and over the own rows, each entered where eight tiles are left of it
        const int pos = ps.bx * 64 * s.m, ta = sw.ta;
        std::vector<char> steady(sw.T, 0);
        {
          int t = 1;
          auto search = [&](int64_t end, int from) {
            if (end - std::max(t, from) < 8) return;
            while (t % 4 || t < from) ++t;
            for (; t + 4 <= end; t += 4) std::fill_n(steady.begin() + t, 4, 1);
          };
          const int64_t full = sw.na / 64;
          if (sw.jr < ta) {
            search(std::min<int64_t>(full, sw.jr) - 3, 0);
            search(full - 3, sw.jr - 2);
          } else {
            search(full - 3, 0);
          }
          t = std::max(t, ta);
          search(std::min<int64_t>(std::min<int64_t>((pos + 1) / 64, nb / 64 - 3) - ps.b0 + ta, sw.T - 3), 0);
        }
        std::vector<char> found(sw.T, 0);
        PfStream st[2];                                     // V(t + 2), K(t + 3)
        for (int j = 0; j < 2; ++j) pf_stream_start(st[j], sw, 3 + j, p0, own);
        for (int t = 1, piece = 0;;) {
          const PfRun run = pf_next_run(sw, piece, t, pos);
          CHECK(run.begin >= t && run.end <= sw.T);
          auto asked = [&](const PfStream& x, int u) {
            CHECK(inside(x.p, x.rows));
            if (u < sw.T) CHECK(x.p == where(u) && x.rows == pf_tile_rows(sw, u));
          };
          auto meet = [&](PfStream& x, int u) { if (x.left == 0) pf_stream_meet(x, sw, u, p0, own); };
          for (; t < run.begin; ++t)
            for (int j = 0; j < 2; ++j) {
              asked(st[j], t + 2 + j);
              st[j].p += st[j].step;
              --st[j].left;
              meet(st[j], t + 3 + j);
            }
          if (t >= sw.T) break;
          ++runs;
          CHECK(run.begin % 4 == 0 && run.end % 4 == 0 && run.end > run.begin && run.end <= sw.T - 3);
          for (int j = 0; j < 2; ++j) CHECK(st[j].left >= run.end - run.begin && st[j].rows == 64);
          for (; t < run.end; ++t) {
            found[t] = 1;
            CHECK(pf_tile_rows(sw, t) == 64 && (t < ta || 64 * (t + sw.own0) + 63 <= pos));
            for (int j = 0; j < 2; ++j) {
              asked(st[j], t + 2 + j);
              st[j].p += 16384;
            }
          }
          for (int j = 0; j < 2; ++j) {
            st[j].left -= run.end - run.begin;
            meet(st[j], t + 2 + j);
          }
        }
        CHECK(found == steady);
      }
    }
  }
  CHECK(runs > 1000);
  std::printf("%ld checks, %ld failures, %ld runs\n", checks, bad, runs);
  return bad != 0;
}
