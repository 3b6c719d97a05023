// The loads of prefill_kernel_deep16, replayed pass by pass (csrc/hi_prefill_part.h): the tiles that a pass asks for ahead are
// the right ones, and no load - nor the ones behind a pass's last tile - leaves the rows that the launch was given.
#include <algorithm>
#include <cstdio>
#include <random>
#include "hi_prefill_part.h"

using namespace hi;

static long checks = 0, bad = 0;
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
    if (pick(2)) {                                     // blocks of one height, a multiple of 16 positions
      const int even = (int)(((C + s.nbk - 1) / s.nbk + 15) / 16 * 16);
      if ((s.nbk - 1) * even < C) s.strip = even;
    }
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
      const int64_t last = std::min<int64_t>((b + 1) * (s.strip ? s.strip : 64 * s.m), C) - 1;
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
        for (int ahead = 3; ahead >= 2; --ahead) {          // K(t + 3), V(t + 2)
          PfStream st;
          pf_stream_start(st, sw, 1 + ahead, p0, own);
          for (int t = 1; t < sw.T; ++t) {
            const int u = t + ahead;
            CHECK(inside(st.p, st.rows));
            if (u < sw.T) CHECK(st.p == where(u) && st.rows == pf_tile_rows(sw, u));
            st.p += st.step;
            if (--st.left == 0) pf_stream_meet(st, sw, u + 1, p0, own);
          }
        }
      }
    }
  }
  std::printf("%ld checks, %ld failures\n", checks, bad);
  return bad != 0;
}
