// What the workgroups of the 4-wave prefill kernels visit (pure integer arithmetic, shared by the kernels, their launchers and the
// host-side tests; no HIP call): the 64-row tiles of each workgroup in their order, the rows of a tile that a query row sees, the
// streams that load them, and the rows of a chunk that enter a streaming head's store.
#pragma once
#include "hi_prefill_part.h"

namespace hi {

// Rows [0, n) of a tile as a bit mask.
HI_HD uint64_t pf_rows_below(int n) { return n <= 0 ? 0 : n >= 64 ? ~0ull : (1ull << n) - 1; }

// The loads of K tiles, or of V tiles, as a stream: visit v's rows lie at `base`, row r of a tile at the stream's offset for r behind it
// (those of 64 rows in a row if `usual`), and up to visit `until` the next tile is the next 16 KiB with the same offsets.  Behind the
// last visit (T of them) come its rows again, which nobody reads.
struct PfLoads { const char* base; int v, until, usual; };
// the next visit; true: the stream has come to rows it does not know yet
HI_HD bool pf_loads_next(PfLoads& w, int T) {
  w.base += kPfSweepBytes;
  if (++w.v != w.until) return false;
  if (w.v < T) return true;
  w.base -= kPfSweepBytes;
  w.until = w.v + 1;
  return false;
}

// ---- prefill_kernel: visit v is past tile a0 + v up to visit ta, then the chunk's own tile b0 + v - ta.
struct PfNarrow {
  int na, nb;            // rows of the past segment, own rows
  int ta, T;             // past tiles, and all tiles of the workgroup (at least 1)
  int a0, b0;
  int jump_tile;         // past tiles from this one on lie jump_bytes further on (0: in one piece)
  int64_t jump_bytes;
};
// The stream has come to visit w.v: the rows `past` or `own` begins with.  True: it takes offsets of its own, row min(r, rows - 1) for r.
HI_HD bool pf_narrow_meet(PfLoads& w, const PfNarrow& n, const char* past, const char* own, int& rows) {
  const bool in_b = w.v >= n.ta;
  const int na = n.na, nb = n.nb, segment = in_b ? nb : na;      // (picked from memory, the compiler keeps them there)
  const int tile = in_b ? n.b0 + w.v - n.ta : n.a0 + w.v, whole = segment / kPfSweepRows;
  const bool jumped = !in_b && n.jump_tile > 0 && tile >= n.jump_tile;
  const bool usual = tile < whole;
  int end = whole;                              // the run of tiles that follow each other
  if (!in_b && n.jump_tile > 0 && !jumped && n.jump_tile < end) end = n.jump_tile;
  w.until = w.v + (usual ? end - tile : 1);
  if (!in_b && w.until > n.ta) w.until = n.ta;
  w.base = (in_b ? own : past) + (int64_t)tile * kPfSweepBytes;
  if (jumped) w.base += n.jump_bytes;
  rows = usual ? kPfSweepRows : segment - tile * kPfSweepRows;
  const bool anew = !(usual && w.usual);
  w.usual = usual;
  return anew;
}
// Visits [0, a) and [ta, b) show all their rows to the 32 query rows from i0 on: the others are a segment's last rows, or own rows
// behind a query's position.
struct PfOpen { int a, b; };
HI_HD PfOpen pf_narrow_open(const PfNarrow& n, int i0) {
  const int whole_a = n.na / kPfSweepRows, whole_b = n.nb / kPfSweepRows, seen = (i0 + 1) / kPfSweepRows;
  return {whole_a - n.a0 < n.ta ? whole_a - n.a0 : n.ta, n.ta + (seen < whole_b ? seen : whole_b) - n.b0};
}
// the rows of visit v that query row i sees
HI_HD uint64_t pf_narrow_seen(const PfNarrow& n, int v, int i) {
  const bool in_b = v >= n.ta;
  const int j0 = (in_b ? n.b0 + v - n.ta : n.a0 + v) * kPfSweepRows, na = n.na, nb = n.nb;
  const int end = (in_b ? nb : na) - j0, own = in_b ? i + 1 - j0 : kPfSweepRows;
  return pf_rows_below(end < own ? end : own);
}

// ---- prefill_window_kernel: A is what a streaming head's store holds of the past (its sink rows, then the ring's rows in token order),
// B the chunk's own rows.
struct PfWindow {
  int C, n_sink, n_recent;
  int ns;                 // sink rows of the past: min(P, n_sink)
  int m;                  // recent rows of the past held by the ring: tokens t0 .. P-1, t0 = max(n_sink, P-n_recent+1)
  int ring0;              // ring slot of token t0
  int lo0;                // index in A of the first recent row visible to chunk row 0 (row i: lo0 + i); may be < ns
  int sink_b;             // chunk rows that are sink tokens: clamp(n_sink - P, 0, C)
};
HI_HD PfWindow pf_window_of(int64_t P, int C, int n_sink, int n_recent) {
  const int64_t t0 = P - n_recent + 1 > n_sink ? P - n_recent + 1 : n_sink;
  PfWindow w;
  w.C = C; w.n_sink = n_sink; w.n_recent = n_recent;
  w.ns = (int)(P < n_sink ? P : n_sink);
  w.m = (int)(P > t0 ? P - t0 : 0);
  w.ring0 = w.m > 0 ? (int)((t0 - n_sink) % n_recent) : 0;
  w.lo0 = (int)(P - n_recent - t0 + 1) + w.ns;       // token P - n_recent + 1 as an index into A
  w.sink_b = (int)(n_sink > P ? (n_sink - P < C ? n_sink - P : C) : 0);
  return w;
}
// The tiles of a workgroup over query positions [i_lo, i_hi]: A [0, a1) and [a2, ta), then B [0, b1) and [b2, tb); nAv of them in A.
struct PfWindowTiles { int ta, tb, a1, a2, b1, b2, nAv, T; };
HI_HD PfWindowTiles pf_window_tiles(const PfWindow& a, int i_lo, int i_hi) {
  PfWindowTiles t;
  t.ta = (a.ns + a.m + kPfSweepRows - 1) / kPfSweepRows;
  const int nb_vis = a.C < i_hi + 1 ? a.C : i_hi + 1;
  t.tb = (nb_vis + kPfSweepRows - 1) / kPfSweepRows;
  t.a1 = (a.ns + kPfSweepRows - 1) / kPfSweepRows;
  if (t.a1 > t.ta) t.a1 = t.ta;
  const int loA = a.lo0 + i_lo;
  t.a2 = loA <= 0 ? 0 : loA / kPfSweepRows;
  t.a2 = t.a2 < t.a1 ? t.a1 : (t.a2 > t.ta ? t.ta : t.a2);
  t.b1 = (a.sink_b + kPfSweepRows - 1) / kPfSweepRows;
  if (t.b1 > t.tb) t.b1 = t.tb;
  const int loB = i_lo - a.n_recent + 1;
  t.b2 = loB <= 0 ? 0 : loB / kPfSweepRows;
  t.b2 = t.b2 < t.b1 ? t.b1 : (t.b2 > t.tb ? t.tb : t.b2);
  t.nAv = t.a1 + (t.ta - t.a2);
  t.T = t.nAv + t.b1 + (t.tb - t.b2);            // >= 1: the tile holding the workgroup's first row
  return t;
}
// visit v -> (sequence, tile)
HI_HD int pf_window_locate(const PfWindowTiles& t, int v, bool& in_b) {
  in_b = v >= t.nAv;
  if (!in_b) return v < t.a1 ? v : t.a2 + (v - t.a1);
  const int w = v - t.nAv;
  return w < t.b1 ? w : t.b2 + (w - t.b1);
}
// Where the store keeps row u of A.
HI_HD int pf_window_row(const PfWindow& a, int u) {
  if (u < a.ns) return u;
  int x = a.ring0 + (u - a.ns);
  if (x >= a.n_recent) x -= a.n_recent;
  return a.n_sink + x;
}
// The stream has come to visit w.v.  True: it takes offsets of its own, row min(r, rows - 1) for r; rows = 0: rows of A from `row0` on,
// through the ring, behind the store's first row.  Tiles follow each other inside the chunk, among the sink rows, and in the ring up to
// where it wraps.  With offsets formed for every tile of the ring, twice now that K and V are streams of their own, four one-query heads of
// 4000 rows behind 4000 took 58.4 us at a window of 64 + 1500 where one set for both planes had taken 51.2; in runs they take 43.9.
HI_HD bool pf_window_meet(PfLoads& w, const PfWindow& a, const PfWindowTiles& t, const char* store, const char* own, int& rows, int& row0) {
  bool in_b;
  const int tile = pf_window_locate(t, w.v, in_b);
  row0 = tile * kPfSweepRows;
  int run, at = row0;                           // tiles that follow each other, and the first one's row
  if (in_b) {
    const int whole = a.C / kPfSweepRows, end = tile >= t.b1 ? t.tb : t.b1;
    run = (end < whole ? end : whole) - tile;
  } else if (row0 < a.ns) {
    run = a.ns / kPfSweepRows - tile;
  } else {
    at = pf_window_row(a, row0);
    const int wraps = a.n_sink + a.n_recent - at, left = a.ns + a.m - row0;
    run = (wraps < left ? wraps : left) / kPfSweepRows;
  }
  const bool usual = run > 0;                   // else the chunk's last rows, rows on both sides of an edge of the ring or of the sink rows
  w.until = w.v + (usual ? run : 1);
  w.base = in_b ? own : store;
  if (usual || in_b) w.base += (int64_t)at * (kPfSweepBytes / kPfSweepRows);
  rows = usual ? kPfSweepRows : in_b ? a.C - row0 : 0;
  const bool anew = !(usual && w.usual);
  w.usual = usual;
  return anew;
}
// Visits [first, first + n) of the recent rows of B show all their rows to the 32 query rows from i0 on.
struct PfSeenVisits { int first, n; };
HI_HD PfSeenVisits pf_window_open(const PfWindow& a, const PfWindowTiles& t, int i0) {
  const int from = i0 + 31 - a.n_recent + 1, last = i0 < a.C - 1 ? i0 : a.C - 1;
  int t0 = from <= 0 ? 0 : (from + kPfSweepRows - 1) / kPfSweepRows;
  if (t0 < t.b2) t0 = t.b2;
  const int t1 = (last + 1) / kPfSweepRows;
  return {t.nAv + t.b1 + t0 - t.b2, t1 > t0 ? t1 - t0 : 0};
}
// Does another tile, the one that begins with row j0 of its sequence, show all its rows to them?
HI_HD bool pf_window_full(const PfWindow& a, bool in_b, int j0, int i0) {
  const int end = j0 + kPfSweepRows - 1;
  return in_b ? end <= (i0 < a.C - 1 ? i0 : a.C - 1) && end < a.sink_b
              : end <= a.ns + a.m - 1 && (end < a.ns || j0 >= a.lo0 + i0 + 31);
}
// The rows of that tile that query row i sees: those up to hi, of which sink rows (below sk) and rows from lo on.
HI_HD uint64_t pf_window_seen(const PfWindow& a, bool in_b, int j0, int i) {
  const int hi = (in_b ? (i < a.C - 1 ? i : a.C - 1) : a.ns + a.m - 1) - j0;
  const int sk = (in_b ? a.sink_b : a.ns) - j0;
  const int lo = (in_b ? i - a.n_recent + 1 : a.lo0 + i) - j0;
  return pf_rows_below(hi + 1) & (pf_rows_below(sk) | ~pf_rows_below(lo));
}

// ---- The chunk's rows on their way into the store: rows [0, cs) to rows s0 .., rows u0 + i (i < cr) to ring slots (slot0 + i) mod n_recent.
// The workgroups of a head's first `readers` strips of positions read ring rows, which these replace: those in the tiles of A behind the
// sink rows (or in the last sink rows' tile, which every strip visits).
struct PfStoreRows { int cs, s0, u0, cr, slot0, readers; };
HI_HD PfStoreRows pf_store_rows(const PfWindow& a, int64_t P, int strip) {
  PfStoreRows r;
  r.cs = a.sink_b;
  r.s0 = (int)P;
  r.u0 = a.C - a.n_recent > r.cs ? a.C - a.n_recent : r.cs;
  r.cr = a.C - r.u0;
  r.slot0 = r.cr > 0 ? (int)((P + r.u0 - a.n_sink) % a.n_recent) : 0;
  const int64_t strips = ((int64_t)a.C + strip - 1) / strip, past = ((int64_t)a.ns + a.m + kPfSweepRows - 1) / kPfSweepRows * kPfSweepRows - a.lo0;
  int64_t readers = a.m == 0 ? 0 : a.ns % kPfSweepRows != 0 ? strips : past <= 0 ? 0 : (past + strip - 1) / strip;
  r.readers = (int)(readers < strips ? readers : strips);
  return r;
}
// The place of chunk row u in the store.
HI_HD int pf_store_row(const PfStoreRows& r, int n_sink, int n_recent, int u) {
  if (u < r.cs) return r.s0 + u;
  const int slot = r.slot0 + (u - r.u0);
  return n_sink + (slot >= n_recent ? slot - n_recent : slot);
}
// Whether the attention launch should write them: without readers by every workgroup; else by the last reader while the others still run,
// so it has to come early, and what it writes has to take no longer than the launch of its own that it saves.  That launch costs 2.4 us
// for any number of rows (calls back to back), one workgroup's copy 1 us per 100 - and where all workgroups run at once, two on
// each of 256 compute units, nobody is left to hide it.  Gain of riding, microseconds of a call behind 3000 rows, for 64 / 128 / 256 / 384 /
// 512 / 900 rows: 60 to 376 workgroups 2.4 / 1.6 / 0.2 / -1.3 / -2.8 / -8 (240, two heads to an XCD: -12 at 900); 480, of 8 heads, 4.0 / 3.4 /
// 2.7 / 1.1 / 0.1 / -1.5; 564 2.0 / 0.6 / -1.5 / -4.7 / -6.6 / -13; 1024 3.8 / 2.3 / 0.7 / -0.3 / -2.1 / -4.2; more than two rounds, 1128 4.1 /
// 4.0 / 4.2 / 3.4 / 3.7 / 2.5, 2048 3.6 / 3.0 / 2.0 / 1.3 / 0.3 / -2.  Of 328 shapes this line picks the slower way in
// 28: by 1.5 us at most where it rides, by 5.9 of 159 where it does not.
HI_HD bool pf_store_rides(const PfStoreRows& r, int64_t strips, int64_t workgroups) {
  return r.readers == 0 || (2 * r.readers <= strips && r.cs + r.cr <= (workgroups > 1024 ? 512 : 256));
}

}  // namespace hi
