// How one launch of the 8-wave prefill kernel divides its work among workgroups (pure integer arithmetic, shared by
// the kernel, the merge kernel, the launcher and the host-side tests; no HIP call).
//
// A launch covers, for every block of query positions b (nbk blocks of `strip` positions, m = strip / 64 tiles
// each), a sequence of 64-row K/V tiles: the `ta` tiles of the past rows the launch was given, then the
// o(b) = min(tb_all, (b + 1) m) tiles of the chunk's own rows at or below the block's causal boundary (Eq. 3: row p
// sees keys 0..p).  Deep blocks have up to tb_all more tiles than shallow ones.  Two partitions:
//   * on its own (`paired` = 0): the sequence of block b is cut into `split` equal ranges, one workgroup each; with
//     split = 1 a workgroup owns its block.  All blocks are equally long when the launch has no own rows.
//   * paired (`paired` = 1, launches that include the chunk's own rows): block nbk-1-p (deep) and block p (shallow)
//     form a unit whose tiles are laid out [deep past | deep own | shallow own | shallow past] and cut into
//     2 * split equal ranges - every workgroup sweeps the same number of tiles whatever its position in the causal
//     triangle, and range k covers the same past rows in every unit, so the workgroups of a range still walk the
//     past in step.  A range may hold tiles of both blocks: the workgroup makes one pass per block.
// Each pass accumulates a softmax state (m, l, O) for one block over a set of tiles; the states of one block are
// merged at the end (any subset of keys in any order gives a valid partial state).  Images of the states:
//   E(b, j), j < split: the j-th contributor of block b - carried from launch to launch of a unit;
//   X(b, j - split):    contributors beyond `split` in a paired launch (fresh states).
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define HI_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define HI_HD inline
#endif

namespace hi {

struct PfShape {
  int nbk;      // blocks of query positions per head
  int m;        // 64-row tiles of own rows a block adds: strip / 64
  int ta;       // past tiles of this launch
  int tb_all;   // tiles of the chunk's own rows (0: the launch has none)
  int split;    // workgroups per block
  int paired;   // balanced partition over (deep, shallow) pairs of blocks
  int carried;  // the images E hold states of earlier launches of the unit
  uint32_t by_split = 0, by_nbk = 0;    // pf_magic of split and nbk (0: divide)
};

// x / d as one multiplication: the kernels divide by split and nbk before they can ask for their first byte, and the
// compiler's division is about 40 dependent instructions of a lone wavefront (0.3 us each: 3 us of a 57 us launch of 600 rows
// behind 3000 went to this arithmetic).  With magic = floor(2^32 / d) + 1 the quotient is exact for x d < 2^32; pf_magic gives
// 0, and pf_div divides, where x can be larger.
HI_HD uint32_t pf_magic(uint32_t d, uint64_t x_max) {
  return d > 1 && x_max * d < (1ull << 32) ? (uint32_t)((1ull << 32) / d + 1) : 0;
}
HI_HD uint32_t pf_div(uint32_t x, uint32_t d, uint32_t magic) {
  return magic ? (uint32_t)(((uint64_t)x * magic) >> 32) : d == 1 ? x : x / d;
}
// the largest number that pf_pass divides by split (the ranges' boundaries) in a launch of this shape
HI_HD uint64_t pf_largest_cut(const PfShape& s) { return 2ull * ((uint64_t)s.ta + s.tb_all) * (2ull * s.split) + 2ull * s.nbk * s.split; }

struct PfPass {
  int run;      // 1: tiles to process
  int init;     // 1: nothing to process, but image `store` must receive an empty state
  int bx;       // block of positions
  int a0, a1;   // past tiles [a0, a1) of the launch
  int b0, b1;   // own tiles [b0, b1) of the chunk
  int load;     // image to start from, -1: empty state
  int store;    // image to store the state to, -1: normalise and write the output rows
};

// images per grid row (one head, one quad of query heads): E then X
HI_HD int pf_images_per_row(int nbk, int split) { return 2 * nbk * split; }
HI_HD int pf_image_e(const PfShape& s, int b, int j) { return j * s.nbk + b; }
HI_HD int pf_image_x(const PfShape& s, int b, int j) { return s.nbk * s.split + b * s.split + j; }

// boundary k of the nr equal ranges a sequence of L tiles is cut into (L * nr < 2^32)
HI_HD int pf_cut(int L, int k, int nr) { return (int)((uint32_t)L * (uint32_t)k / (uint32_t)nr); }

// Workgroup number of grid position x in a grid row of n workgroups.  xcd: the hardware deals workgroups to the 8 XCDs
// in turn; position x takes number (x % 8) (n / 8) + x / 8, so that an XCD's workgroups have consecutive numbers - those
// of one range of K/V rows, which its L2 then fetches once (n is a multiple of 8).
HI_HD int pf_wg_index(int x, int n, int xcd) { return xcd ? (x & 7) * (n >> 3) + (x >> 3) : x; }

HI_HD int pf_own_tiles(const PfShape& s, int b) {
  const int o = (b + 1) * s.m;
  return o < s.tb_all ? o : s.tb_all;
}

// the unit block b belongs to: its deep block, its shallow block (-1: on its own), the number of ranges
HI_HD void pf_unit_of_block(const PfShape& s, int b, int& deep, int& shallow, int& nr) {
  const int pairs = s.paired ? s.nbk / 2 : 0;
  if (b < pairs) { deep = s.nbk - 1 - b; shallow = b; nr = 2 * s.split; }
  else if (b >= s.nbk - pairs) { deep = b; shallow = s.nbk - 1 - b; nr = 2 * s.split; }
  else { deep = b; shallow = -1; nr = s.split; }
}

// contributors of block b (ranges of its unit that hold at least one of its tiles), and how many of them come
// before range k
HI_HD void pf_contributors(const PfShape& s, int deep, int shallow, int nr, int is_shallow, int k, int& before, int& total) {
  const int Td = s.ta + pf_own_tiles(s, deep);
  const int L = Td + (shallow >= 0 ? s.ta + pf_own_tiles(s, shallow) : 0);
  before = total = 0;
  if (L >= nr) {
    // no range is empty: the ranges that start before Td hold deep tiles, those that end after it shallow ones
    const uint32_t u = (uint32_t)nr, l = (uint32_t)L, td = (uint32_t)Td;
    const int kd = (int)((td * u + l - 1) / l);              // first k with cut(k) >= Td
    const int ks = (int)(((td + 1) * u + l - 1) / l) - 1;    // first k with cut(k + 1) > Td
    if (is_shallow) { total = nr - ks; before = k > ks ? k - ks : 0; }
    else { total = kd < nr ? kd : nr; before = k < total ? k : total; }
    return;
  }
  for (int kk = 0; kk < nr; ++kk) {
    const int x0 = pf_cut(L, kk, nr), x1 = pf_cut(L, kk + 1, nr);
    const bool hit = x1 > x0 && (is_shallow ? x1 > Td : x0 < Td);
    if (hit) {
      ++total;
      if (kk < k) ++before;
    }
  }
}

// Pass `which` (0: the unit's deep block, 1: its shallow block) of workgroup w (0 .. nbk * split - 1) of a grid row.
HI_HD PfPass pf_pass(const PfShape& s, int w, int which, int last) {
  PfPass g;
  g.run = g.init = 0; g.bx = 0; g.a0 = g.a1 = g.b0 = g.b1 = 0; g.load = g.store = -1;
  int deep, shallow, nr, k;
  const int pairs = s.paired ? s.nbk / 2 : 0;
  if (w < pairs * 2 * s.split) {
    const int p = (int)(pf_div((uint32_t)w, (uint32_t)s.split, s.by_split) >> 1);
    deep = s.nbk - 1 - p; shallow = p; nr = 2 * s.split; k = w - p * nr;
  } else {
    // blocks on their own: the deepest first, range z of every block before range z + 1 of any (of pairs, one is left or none)
    const int singles = s.nbk - 2 * pairs;
    const int v = w - pairs * 2 * s.split;
    k = pairs ? v : (int)pf_div((uint32_t)v, (uint32_t)s.nbk, s.by_nbk);
    deep = s.nbk - pairs - 1 - (v - k * singles); shallow = -1; nr = s.split;
  }
  if (which == 1 && shallow < 0) return g;
  const int od = pf_own_tiles(s, deep), ob = shallow >= 0 ? pf_own_tiles(s, shallow) : 0;
  const int Td = s.ta + od;
  const int L = Td + (shallow >= 0 ? s.ta + ob : 0);
  const int half = shallow >= 0 ? 1 : 0;        // nr = split << half: boundary k is floor(L k / split) >> half
  const int x0 = (int)(pf_div((uint32_t)L * (uint32_t)k, (uint32_t)s.split, s.by_split) >> half);
  const int x1 = (int)(pf_div((uint32_t)L * (uint32_t)(k + 1), (uint32_t)s.split, s.by_split) >> half);
  auto clampi = [](int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); };
  if (which == 0) {
    g.bx = deep;
    g.a0 = clampi(x0, 0, s.ta); g.a1 = clampi(x1, 0, s.ta);
    g.b0 = clampi(x0 - s.ta, 0, od); g.b1 = clampi(x1 - s.ta, 0, od);
  } else {
    g.bx = shallow;
    g.b0 = clampi(x0 - Td, 0, ob); g.b1 = clampi(x1 - Td, 0, ob);
    g.a0 = clampi(x0 - Td - ob, 0, s.ta); g.a1 = clampi(x1 - Td - ob, 0, s.ta);
  }
  const bool nonempty = g.a1 > g.a0 || g.b1 > g.b0;
  int j = k, nc = nr;                 // a block on its own: range z keeps image z in every launch of the unit
  if (shallow >= 0) pf_contributors(s, deep, shallow, nr, which, k, j, nc);
  if (!nonempty) {
    if (shallow < 0 && !s.carried) { g.init = 1; g.store = pf_image_e(s, g.bx, k); }
    return g;
  }
  g.run = 1;
  if (j < s.split) {
    const int e = pf_image_e(s, g.bx, j);
    g.load = s.carried ? e : -1;
    g.store = (last && s.split == 1 && nc == 1) ? -1 : e;
  } else {
    g.store = pf_image_x(s, g.bx, j - s.split);
  }
  return g;
}

// The images the merge of block b has to combine after the unit's last launch: n_e images E(b, 0..n_e-1), then n_x
// images X(b, 0..n_x-1).  n_e + n_x == 1 with split == 1 means the block was written directly by its only pass.
HI_HD void pf_block_images(const PfShape& s, int b, int& n_e, int& n_x) {
  int deep, shallow, nr;
  pf_unit_of_block(s, b, deep, shallow, nr);
  if (shallow < 0) { n_e = s.split; n_x = 0; return; }
  int before, nc;
  pf_contributors(s, deep, shallow, nr, b == shallow ? 1 : 0, 0, before, nc);
  n_e = s.carried ? s.split : (nc < s.split ? nc : s.split);
  n_x = nc > s.split ? nc - s.split : 0;
}

// The 4-wave kernel: the tiles of a block of positions - all past tiles of the UNIT, then the own tiles up to the block's
// causal boundary - are cut into `split` ranges, whatever the launches the unit comes in.  A launch that was given past tiles
// [tile0, tile0 + ta) of the unit, and the own tiles if it is the last one, works on [lo, hi) of range k (in tiles of the
// unit; empty: not this workgroup's turn).  Every range is swept in one order from an empty state, so the result does not
// depend on where the launches end.
struct PfRange { int lo, hi; int fresh; };
HI_HD PfRange pf_narrow_range(int past_tiles, int own_tiles, int k, int split, int tile0, int ta, int last) {
  const int total = past_tiles + own_tiles;
  const int x0 = pf_cut(total, k, split), x1 = pf_cut(total, k + 1, split);
  const int end = last ? total : tile0 + ta;
  PfRange r;
  r.lo = x0 > tile0 ? x0 : tile0;
  r.hi = x1 < end ? x1 : end;
  r.fresh = x0 >= tile0;
  return r;
}

// The tiles of one pass of prefill_kernel_deep16, in the order in which it sweeps them: past tiles [0, ta), of which [0, full_a)
// are full, then own tiles; tile t >= ta is tile t + own0 of the chunk's own rows.  A past segment in two pieces: its tiles
// from jr on lie `jump` bytes further on.
constexpr int kPfSweepRows = 64;
constexpr int64_t kPfSweepBytes = 16384;
struct PfSweep {
  int ta, T, full_a, own0, own_full, jr;      // own_full: end of the full own tiles of the sweep
  int64_t na, nb, jump;                       // rows of the past part; rows of the chunk
};
// fills w; returns the byte offset of the pass's first past tile in the launch's past segment
HI_HD int64_t pf_sweep_of(PfSweep& w, const PfPass& ps, int64_t na, int64_t nb, int jump_tile, int64_t jump_bytes) {
  const bool behind = jump_tile > 0 && jump_tile <= ps.a0;         // the whole pass lies behind the jump
  w.jr = jump_tile > 0 && !behind ? jump_tile - ps.a0 : 0x7fffffff;
  w.jump = jump_bytes;
  int64_t end = (int64_t)ps.a1 * kPfSweepRows;
  if (end > na) end = na;
  w.na = end - (int64_t)ps.a0 * kPfSweepRows;
  w.nb = nb;
  w.ta = (int)((w.na + kPfSweepRows - 1) / kPfSweepRows);
  w.full_a = (int)(w.na / kPfSweepRows);
  w.T = w.ta + ps.b1 - ps.b0;
  w.own0 = ps.b0 - w.ta;
  const int64_t full = nb / kPfSweepRows - w.own0;
  w.own_full = (int)(full < w.T ? full : w.T);
  return (int64_t)ps.a0 * kPfSweepBytes + (behind ? jump_bytes : 0);
}
// byte offset of tile t behind the pass's past rows (t < ta) or the chunk's own rows, and its rows
HI_HD int64_t pf_tile_offset(const PfSweep& w, int t) {
  return t >= w.ta ? (int64_t)(t + w.own0) * kPfSweepBytes : (int64_t)t * kPfSweepBytes + (t >= w.jr ? w.jump : 0);
}
HI_HD int pf_tile_rows(const PfSweep& w, int t) {
  const int64_t left = t >= w.ta ? w.nb - (int64_t)(t + w.own0) * kPfSweepRows : w.na - (int64_t)t * kPfSweepRows;
  return left < kPfSweepRows ? (int)left : kPfSweepRows;
}

// A stream of tile loads, one tile after the other: the next one lies at p and has `rows` rows (the lanes' addresses are clamped
// to them).  The caller goes on with p += step; --left, and calls pf_stream_meet with the next tile's number when left is 0:
// there the stream meets the next piece of the past, the own rows, a partial tile, or the pass's end.  At the end it stays at
// its last tile, which then lands in ring slots that nobody reads any more.
struct PfStream { const char* p; int64_t step; int left, rows; };
HI_HD void pf_stream_to(PfStream& s, const PfSweep& w, int u, const char* past, const char* own) {
  s.rows = pf_tile_rows(w, u);
  s.p = (u >= w.ta ? own : past) + pf_tile_offset(w, u);
  if (s.rows == kPfSweepRows) {
    s.step = kPfSweepBytes;
    s.left = (u >= w.ta ? w.own_full : u < w.jr && w.jr < w.ta && w.jr < w.full_a ? w.jr : w.full_a) - u;
  } else {
    s.step = 0;
    s.left = 1;
  }
}
HI_HD void pf_stream_meet(PfStream& s, const PfSweep& w, int u, const char* past, const char* own) {
  if (u < w.T) { pf_stream_to(s, w, u, past, own); return; }
  s.p -= s.step;
  s.step = 0;
  s.left = 0x7fffffff;
}
// the stream in front of tile u of a pass that has one tile at least
HI_HD void pf_stream_start(PfStream& s, const PfSweep& w, int u, const char* past, const char* own) {
  pf_stream_to(s, w, u < w.T ? u : w.T - 1, past, own);
  if (u >= w.T) {
    s.step = 0;
    s.left = 0x7fffffff;
  }
}

// The runs of steady tiles of a pass: [begin, end), whole groups of four that begin at a multiple of four, every tile full and seen
// in full from position `pos` (the block's first) on, and so are the tiles that it asks for ahead, all on one side of a jump.
// All other tiles take their maxima, and a run is worth its entry from eight tiles on.  pf_next_run gives the first run that
// begins at tile t or behind it (or T, T); piece: 0 before the first call, where the search goes on.
struct PfRun { int begin, end; };
HI_HD PfRun pf_next_run(const PfSweep& w, int& piece, int t, int pos) {
  while (piece < 3) {
    const bool two = w.jr < w.ta;
    int lo = t, end = w.full_a - 3;
    if (piece == 0 && two && w.jr - 3 < end) end = w.jr - 3;
    if (piece == 1) {
      if (!two) end = 0;
      if (w.jr - 2 > lo) lo = w.jr - 2;
    }
    if (piece == 2) {
      const int seen = (pos + 1) / kPfSweepRows - w.own0;
      end = w.own_full - 3 < seen ? w.own_full - 3 : seen;
      if (w.ta > lo) lo = w.ta;
    }
    ++piece;
    if (end - lo < 8) continue;
    const int begin = (lo + 3) & ~3;
    return {begin, begin + ((end - begin) & ~3)};
  }
  return {w.T, w.T};
}

}  // namespace hi
