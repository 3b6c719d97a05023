// Internal declarations shared by the host-side sources of the library (not part of the ABI).
#pragma once
#include <cstdint>
#include <cstddef>
#include "headinfer.h"
#include "hi_prefill_part.h"
#include "hi_prefill_visits.h"

namespace hi {

constexpr int kHeadDim = 128;
constexpr int kRowBytes = kHeadDim * 2;          // one K (or V) row of one head, bf16
constexpr int kLinkRowBytes4 = kHeadDim / 2 + 4 * (kHeadDim / 32);   // a row as 4-bit codes + bf16 scale/zero per 32 channels
constexpr int kWgThreads = 256;                  // 4 wavefronts of 64
constexpr int kCarryFloatsPerLane = 68;          // 64 O^T accumulators + running maxima + row-sum shares (one of each
                                                 // in the 32x32x16 kernels, two in the 16x16x32 kernel)
constexpr int kPartialFloats = kHeadDim + 2;     // O[128], m, l of one (partition, query head)

void set_last_error(const char* fmt, ...);

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

// query positions covered by one prefill workgroup, and the grid's second dimension, for a GQA group size
inline int prefill_strip(int G) { return 32 * (4 / (G < 4 ? G : 4)); }
inline int prefill_grid_y(int G) { return G > 4 ? G / 4 : 1; }

// The 8-wave prefill kernel covers 2 * strip positions per workgroup.  When a chunk gives it fewer workgroups than
// would fill the chip, `split` workgroups share each block of positions and divide the tiles of every launch
// between them (their states are merged after the unit's last launch).  prefill_split and prefill_launch_shape are the
// choice by the chunk alone, which sizes the plan's workspace: the 8-wave kernel when workgroups * split reaches
// kPrefillDeepMinWorkgroups, the 4-wave kernel otherwise.  What a unit runs is prefill_unit_shape's choice.
constexpr int kPrefillFillWorkgroups = 192;
constexpr int kPrefillDeepMinWorkgroups = 128;
constexpr int kPrefillMaxSplit = 8;
inline int prefill_split(int G, int64_t chunk_len, int n_heads = 1) {
  const int64_t wgs = ceil_div(chunk_len, 2 * prefill_strip(G)) * prefill_grid_y(G) * n_heads;
  int split = 1;
  while (wgs * split < kPrefillFillWorkgroups && split < kPrefillMaxSplit) split *= 2;
  return split;
}
// What one launch of a prefill unit looks like (host side; the kernels derive the rest from these numbers).
// variant: low two bits 0 = pick the kernel by chunk length, 1 = 4-wave kernel, 3 = 8-wave kernel; + 4: pair deep and
// shallow blocks in every last launch that has two blocks, + 8: never pair (measurement); + 16: the 8-wave kernel in
// its 32x32x16 MFMA form instead of the 16x16x32 one; + 64 / + 128: the 16x16x32 kernel with 8 wavefronts of 32 query rows
// (prefill_kernel_deep16) / with 4 wavefronts of 64 (prefill_kernel_wide) whatever the launch's length (by default the
// second for launches whose workgroups sweep kPrefillWideMinTiles tiles and more).
constexpr int kPrefillWideMinTiles = 640;
constexpr int kPdLanes = 512;                   // lanes of an 8-wave workgroup
constexpr int kPrefillPairMinTiles = 4;         // pair when it saves the deepest workgroup at least this many tiles
struct PrefillLaunch {
  int deep;            // 8-wave kernel (else the 4-wave one)
  int split;           // workgroups per block of positions
  int paired;          // balanced partition over (deep, shallow) pairs of blocks
  int nbk;             // blocks of positions per head (8-wave kernel)
  int merge;           // a merge launch follows
  int64_t carry_bytes; // state images the launches of this unit address in the carry
  int img_row;         // state images of one grid row (a head, a quad of query heads)
  int xcd;             // the workgroups of a grid row are numbered so that neighbours share an XCD (pf_wg_index)
  int past_tiles;      // 4-wave kernel, split > 1: tiles of the unit's cached rows
};
inline PrefillLaunch prefill_launch_shape(int G, int64_t chunk_len, int n_heads, int variant, int last, int has_own) {
  PrefillLaunch p;
  const int strip = prefill_strip(G), gy = prefill_grid_y(G), base = variant & 3;
  p.split = prefill_split(G, chunk_len, n_heads);
  p.nbk = (int)ceil_div(chunk_len, 2 * strip);
  p.deep = base == 3 || (base == 0 && (int64_t)p.nbk * gy * n_heads * p.split >= kPrefillDeepMinWorkgroups);
  p.paired = p.merge = p.xcd = p.past_tiles = 0;
  p.img_row = pf_images_per_row(p.nbk, p.split);
  if (p.deep) {
    // tiles the workgroups of the deepest block sweep beyond the average (the causal triangle), which pairing removes
    const int64_t saved = (int64_t)(2 * strip / 64) * (p.nbk - 1) / (2 * p.split);
    p.paired = last && has_own && p.nbk >= 2 && !(variant & 8) && ((variant & 4) || saved >= kPrefillPairMinTiles);
    p.merge = last && (p.split > 1 || p.paired);
    p.carry_bytes = (int64_t)2 * p.nbk * p.split * gy * n_heads * kPdLanes * kCarryFloatsPerLane * 4;
  } else {
    p.split = 1;
    p.carry_bytes = ceil_div(chunk_len, strip) * gy * n_heads * kWgThreads * kCarryFloatsPerLane * 4;
  }
  return p;
}

// Does a launch of the 8-wave kernel over this many K/V rows run its wide form?
inline bool prefill_is_wide(int variant, int split, int64_t rows) {
  if (variant & 16) return false;
  return (variant & 128) != 0 || ((variant & 64) == 0 && rows / 64 >= (int64_t)kPrefillWideMinTiles * split);
}

constexpr int kPrefillUnitMaxSplit = 64;
constexpr int kPrefillCus = 256;

// Ranges the 4-wave kernel cuts a unit's tiles into, where the chunk alone would pick that kernel (few blocks of positions):
// fixed in tiles of the unit and chosen without regard to the launches the unit comes in or to the heads of the call, so
// that offloaded and resident results, and those of different head groups, agree bit for bit.  The least time by this model,
// in microseconds: 4 to start, load and store the state, 1.3 per tile with one workgroup per compute unit, 1.9 with two; the
// merge 5 + 0.03 per image; for the largest group this kernel serves at this chunk length (all_heads: heads of a layer).
// Measured, uncut -> cut (the 8-wave kernel at its best split): 30 rows of 8 heads behind 100 thousand 1795 -> 104 us (127),
// 64 rows 1788 -> 141 (134), 64 rows behind 5000 107 -> 25 (36); one head: 512 rows behind 1536 48 -> 23, 900 rows behind 20
// thousand 389 -> 63 (71), behind 60 thousand 1093 -> 139 (124).  Error against 64 bits over 24 shapes (mean of the relative
// 2-norms): 0.00122 -> 0.00099 (0.00110).
inline int prefill_narrow_split(int G, int64_t C, int64_t past, int64_t capacity, int all_heads) {
  const int strip = prefill_strip(G), gy = prefill_grid_y(G);
  int64_t heads = (kPrefillDeepMinWorkgroups / kPrefillMaxSplit - 1) / (ceil_div(C, 2 * strip) * gy);
  if (heads > all_heads) heads = all_heads;
  if (heads < 1) heads = 1;
  const int64_t blocks = ceil_div(C, strip) * gy * heads, image = (int64_t)kWgThreads * kCarryFloatsPerLane * 4;
  const int64_t past_tiles = ceil_div(past, 64), tiles = past_tiles + ceil_div(C, 64);
  int best = 1;
  double best_us = 1e30;
  for (int split = 1; split <= kPrefillUnitMaxSplit && (split == 1 || 4 * (int64_t)split <= past_tiles); ++split) {
    const int64_t wgs = blocks * split, full = wgs / (2 * kPrefillCus), rest = wgs % (2 * kPrefillCus);
    if (split > 1 && wgs * image > capacity) break;
    const double range = (double)ceil_div(tiles, split);
    double us = (double)full * (4.0 + 1.9 * range);
    if (rest) us += 4.0 + (rest > kPrefillCus ? 1.9 : 1.3) * range;
    if (split > 1) us += 5.0 + 0.03 * (double)wgs;
    if (us < best_us) {
      best_us = us;
      best = split;
    }
  }
  return best;
}

// The split and the pairing of one unit, chosen for what the unit sweeps: `past` cached rows in launches of up to
// `slice` of them (0: one launch), then the chunk's own rows.  capacity: bytes the state images may take (the plan's
// carry holds what prefill_launch_shape asks for; the decode partials behind it are idle while a prefill unit runs).
// The result is that of the unit's last launch; prefill_launch_of gives the others.
//
// The candidate with the least time by this model wins, in microseconds, fitted to sweeps of split and pairing over 17
// shapes (1 to 32 heads, chunks of 30 to 4096 rows, 0 to 100 thousand cached rows; it picks a split within 6 % of the best
// one in all of them).  A workgroup of the 8-wave kernel, one per compute unit: 10 to start, load and store its state;
// 1.9 per tile for its first 14 tiles (ring fill, masked and alignment tiles), then 1.1 per tile while at most 190 run and
// up to 1.45 on a full chip (power).  A paired launch makes two passes (12 more).  The merge: 5 + 0.035 per image.  The
// 4-wave kernel: 4 + 1.3 per tile with one workgroup per compute unit, 1.9 with two.
// (The constants were fitted to an 8-wave kernel that began 2.5 us later and took 2.6 us for a tile that takes its maximum, where
// it takes 2.3 now.  Constants re-fitted to a faster form of it - 8 to start, 0.35 more for each of four tiles, 1.15 to 1.5 per
// tile, 8 a second pass - chose worse splits, 0.79 to 1.02 times as fast over 23 shapes: the model has one fill for all
// workgroups and knows nothing of rows that neighbours share in an L2, which the old constants happen to cover.)
// What it replaces sized the split by the chunk alone, in powers of two up to 8: 77 rows of 8 heads behind 100 thousand ran
// on 128 workgroups (302 us, now 178), 600 rows behind 3000 in two rounds of workgroups (92 -> 70), 2400 rows behind 5000
// likewise (333 -> 277).  Chunks that the rule by the chunk alone gives to the 4-wave kernel stay there, cut into ranges.
inline PrefillLaunch prefill_launch_of(PrefillLaunch unit, int last, int has_own) {
  if (unit.deep && !(last && has_own)) unit.paired = 0;
  if (unit.paired) unit.xcd = 0;           // pairs are numbered range by range already
  if (!last) unit.merge = 0;
  return unit;
}
inline PrefillLaunch prefill_unit_shape(int G, int64_t C, int n_heads, int variant, int64_t past, int64_t slice,
                                        int64_t capacity, int all_heads = 0) {
  PrefillLaunch best = prefill_launch_shape(G, C, n_heads, variant, 1, 1);
  const int strip = prefill_strip(G), rows = prefill_grid_y(G) * n_heads, base = variant & 3;
  if (!best.deep) {
    best.split = 1;
    if (base == 1) return best;
    const int strips = (int)ceil_div(C, strip);
    best.split = prefill_narrow_split(G, C, past, capacity, all_heads > n_heads ? all_heads : n_heads);
    best.merge = best.split > 1;
    best.img_row = strips * best.split;
    best.carry_bytes *= best.split;
    best.past_tiles = (int)ceil_div(past, 64);
    best.xcd = best.img_row % 8 == 0;
    return best;
  }
  const int64_t launches = past > 0 && slice > 0 ? ceil_div(past, slice) : 1;
  const double tiles_past = (double)ceil_div(past, 64) / (double)launches;       // of one launch
  const int64_t own = ceil_div(C, 64), m = 2 * strip / 64, image = (int64_t)kPdLanes * kCarryFloatsPerLane * 4;
  const double deepest = (double)(own < best.nbk * m ? own : best.nbk * m), average = 0.5 * (deepest + (double)m);
  auto workgroup = [](double tiles, int64_t running) {
    const double tile = running > 194 ? 1.45 * (double)running / kPrefillCus : 1.1;
    return 10.0 + (tiles < 14.0 ? tiles * 1.9 : 14.0 * 1.9 + (tiles - 14.0) * tile);
  };
  // wgs workgroups of `first` tiles in the first round (the deepest), `others` in the rounds after it
  auto rounds = [&](int64_t wgs, double first, double others) {
    const int64_t full = wgs / kPrefillCus, rest = wgs % kPrefillCus;
    if (full == 0) return workgroup(first, rest);
    return workgroup(first, kPrefillCus) + (double)(full - 1) * workgroup(others, kPrefillCus) + (rest ? workgroup(others, rest) : 0.0);
  };
  auto cost = [&](int split, int paired) {
    const int64_t wgs = (int64_t)best.nbk * rows * split;
    auto range = [&](double tiles) { return (double)(int64_t)(tiles / split + 0.999); };
    double us = (double)(launches - 1) * rounds(wgs, range(tiles_past), range(tiles_past));
    if (paired) us += rounds(wgs, range(tiles_past + average), range(tiles_past + average)) + 12.0 * (double)ceil_div(wgs, kPrefillCus);
    else us += rounds(wgs, range(tiles_past + deepest), range(tiles_past + average));
    if (split > 1 || paired) us += 5.0 + (double)wgs * 0.035;
    return us;
  };
  double best_us = 0.97 * cost(best.split, best.paired);     // a clear gain, or stay with the default
  if (base != 3 && !(variant & (4 | 8 | 16 | 64 | 128))) {       // (those flags name forms of the 8-wave kernel)
    const int64_t wgs = ceil_div(C, strip) * rows;
    const double us = (double)launches * ((double)ceil_div(wgs, 2 * kPrefillCus) *
                                          (4.0 + (tiles_past + (double)own) * (wgs > kPrefillCus ? 1.9 : 1.3)));
    if (us < best_us) {
      best_us = us;
      best.deep = best.paired = best.merge = 0;
      best.split = 1;
      best.carry_bytes = wgs * kWgThreads * kCarryFloatsPerLane * 4;
    }
  }
  const int64_t fewest = past > 0 ? (past < slice || slice <= 0 ? past : slice) / 64 : own;   // tiles of a full launch
  for (int split = 1; split <= kPrefillUnitMaxSplit; ++split) {
    if (split > 1 && split > fewest) break;
    for (int paired = 0; paired < 2; ++paired) {
      if (paired && (best.nbk < 2 || (variant & 8))) continue;
      if (!paired && best.nbk >= 2 && (variant & 4)) continue;
      const int64_t images = (int64_t)(paired ? 2 : 1) * best.nbk * split;
      if (images * rows * image > capacity) continue;
      const double us = cost(split, paired);
      if (us >= best_us) continue;
      best_us = us;
      best.deep = 1; best.split = split; best.paired = paired;
      best.merge = split > 1 || paired;
      best.img_row = (int)images;
      best.carry_bytes = images * rows * image;
    }
  }
  // neighbours in the numbering read the same K/V rows: let them share an XCD's L2 when one round of workgroups holds all
  best.xcd = best.deep && best.split > 1 && best.nbk * best.split % 8 == 0 &&
             (int64_t)best.nbk * rows * best.split <= kPrefillCus;
  return best;
}

// the largest carry any launch of chunks up to C rows over groups of up to n_heads heads can address, whatever the
// kernel variant (both kernels' image counts are step functions of the chunk length with steps at multiples of strip)
inline int64_t prefill_carry_bound(int G, int64_t C, int n_heads) {
  const int strip = prefill_strip(G);
  int64_t worst = 0;
  for (int64_t len = strip; ; len += strip) {
    const int64_t l = len < C ? len : C;
    for (int nh = 1; nh <= n_heads; ++nh)
      for (int variant = 0; variant <= 3; ++variant) {
        if (variant == 2) continue;
        const int64_t need = prefill_launch_shape(G, l, nh, variant, 1, 1).carry_bytes;
        if (need > worst) worst = need;
      }
    if (len >= C) break;
  }
  return worst;
}

// floats of decode partials one head can produce (one launch per staging slice, n_split partials each; a head of
// a group has 1/n of the slice and 1/n of the partitions, up to rounding - hence the factor 2): the distance
// between the heads' partials in the workspace
inline int64_t decode_part_head_stride(int64_t max_context, int64_t slice_tokens, int n_split, int G) {
  return 2 * (ceil_div(max_context, slice_tokens) + 1) * n_split * G * kPartialFloats;
}

hi_status validate_problem(const hi_problem* p);

// Appendix E head roles: is (layer, head) a streaming head?  (the mask if given, else the last streaming_heads heads)
inline bool head_is_streaming(const hi_problem& p, const uint8_t* mask, int layer, int head) {
  if (mask) return mask[(int64_t)layer * p.n_kv_heads + head] != 0;
  return head >= p.n_kv_heads - p.streaming_heads;
}
// streaming heads of all layers
inline int64_t count_streaming(const hi_problem& p) {
  if (!p.streaming_mask) return (int64_t)p.n_layers * p.streaming_heads;
  int64_t n = 0;
  for (int64_t i = 0; i < (int64_t)p.n_layers * p.n_kv_heads; ++i) n += p.streaming_mask[i] != 0;
  return n;
}

// ---- kernel launchers (defined in the .hip files) ------------------------------------------------------
// done: an event (hipEvent_t) that marks the end of the last kernel launched, see launch_kernel; null: none
struct PrefillSegment {
  const void* k;      // device, [n][128] bf16 (first head of a group)
  const void* v;
  int64_t n;          // rows
  int causal;         // 1: rows are the chunk's own (row j visible to query i iff j <= i)
  int64_t head_stride = 0;   // bytes from one head's K (V) rows to the next head's, for launches over a head group
  // A past segment may consist of two pieces (two staging slots in one launch): rows [0, jump_rows) start at k / v,
  // the rows after them jump_bytes further on than they would in one piece.  jump_rows is a multiple of 64; 0: one
  // piece.  The 16x16x32 kernels and the 4-wave kernel with split > 1 take such a segment.
  int64_t jump_rows = 0;
  int64_t jump_bytes = 0;
  int64_t tile0 = 0;         // past segment: its first tile, counted over the unit's cached rows
};

// Rows [heads][rows][128] of K and of V to the heads' places in an HBM cache, head_stride bytes apart: in a launch of its own, or
// along with a unit's merge launch (the unit reads the cache only before those rows).
struct PrefillAppend {
  const void* k_new; const void* v_new;
  void* k_dst; void* v_dst;
  int64_t rows;
  int heads;
  int64_t head_stride;
};

// One launch of the prefill kernel over up to two KV segments.  first: start from an empty softmax state
// instead of loading the carry; last: normalise and write `out` instead of storing the carry.
// variant: as at prefill_launch_shape (+ 32: the queries are pre-scaled, see softmax_scale_log2); shape: the unit's, from
// prefill_unit_shape; every launch of one unit must use the same variant and shape (the carry layouts differ).
// carry_bytes: size of the carry buffer (checked against what the launch will use).
// n_heads > 1: one launch over a group of KV heads; q is [n_heads][G][chunk_len][128], out likewise, the causal
// segment's rows [n_heads][chunk_len][128], the other segment's heads head_stride bytes apart.
hi_status launch_prefill(void* stream, const void* q, int G, int chunk_len, const PrefillSegment& a,
                         const PrefillSegment& b, int first, int last, void* carry, void* out, int out_fp32,
                         int variant, const PrefillLaunch& unit, int n_heads, int64_t carry_bytes,
                         const PrefillAppend* append = nullptr, void* done = nullptr);
hi_status launch_kv_append(void* stream, const PrefillAppend& append, void* done = nullptr);

// The factor between a query-key dot product and the base-2 exponent of its softmax weight: log2(e) / sqrt(128) for
// the q of Eq. 3, 1 for queries that already carry that factor (hi_problem.q_prescaled).
inline float softmax_scale_log2(bool q_prescaled) { return q_prescaled ? 1.0f : 1.4426950408889634f / 11.313708498984761f; }

// rows per head of a decode launch whose heads differ in length (passed to the kernels by value)
constexpr int kDecodeMaxRagged = 64;
// A head is cut into ceil(n / rows_per_wg) partitions (at least one): every workgroup of the launch reads about as many rows,
// whatever head it works for - or, with lengths close together, into the same number.
struct DecodeLens {
  uint32_t n[kDecodeMaxRagged];         // rows (of an HBM-resident head: far below 2^31)
  uint32_t rows_per_wg;                 // 0: the same number of partitions for every head
  uint16_t first[kDecodeMaxRagged];     // workgroup that starts each head (0xffff behind the last head)
};
constexpr int kDecodeMaxCut = 16384;    // workgroups of such a launch
constexpr int decode_parts(uint32_t n, uint32_t rows_per_wg) {           // (constexpr: host and device)
  return n <= rows_per_wg ? 1 : (int)((n + rows_per_wg - 1) / rows_per_wg);
}
// Cuts heads of lens.n[0 .. n_heads) rows into partitions of at least 64 rows, for at most max_wgs workgroups where the heads
// are no more than that.  Returns the number of workgroups; most: the largest number of partitions any head has.
// With the same number for every head the longest head's workgroups are left alone at the end: in proportion, 8 sequences of
// 8 heads spread evenly up to 60 thousand rows take 175 us instead of 207 (6.3 TB/s), one of 60 thousand beside 63 heads of 50
// rows 20 instead of 176.  But finding its head costs a workgroup about 1 us: worth it where the longest head's workgroups
// would read at least 160 rows more than the average (at 250 the gain is 0.8 us, at 330 2 us).
constexpr int kDecodeCutMinRows = 160;
inline int decode_cut(DecodeLens& lens, int n_heads, int max_wgs, int* most) {
  const uint32_t* n = lens.n;
  if (max_wgs > kDecodeMaxCut) max_wgs = kDecodeMaxCut;
  int64_t total = 0, longest = 0;
  for (int j = 0; j < n_heads; ++j) {
    total += n[j];
    if (n[j] > longest) longest = n[j];
  }
  const int64_t alike = max_wgs / n_heads > 0 ? max_wgs / n_heads : 1, need = ceil_div(longest, 64);
  const int64_t same = need < alike ? need : alike;
  lens.rows_per_wg = 0;
  *most = (int)(same > 0 ? same : 1);
  if (longest / *most - total / max_wgs < kDecodeCutMinRows) return *most * n_heads;
  // half a workgroup per head lost to rounding is what to expect, a whole one the worst case
  for (int lost = n_heads / 2; ; lost = n_heads) {
    const int64_t each = ceil_div(total, max_wgs - lost > 1 ? max_wgs - lost : 1);
    lens.rows_per_wg = (uint32_t)round_up(each > 64 ? each : 64, 16);
    int wgs = 0;
    *most = 1;
    for (int j = 0; j < n_heads; ++j) {
      const int p = decode_parts(n[j], lens.rows_per_wg);
      lens.first[j] = (uint16_t)wgs;
      wgs += p;
      if (p > *most) *most = p;
    }
    for (int j = n_heads; j < kDecodeMaxRagged; ++j) lens.first[j] = 0xffff;
    if (wgs <= max_wgs || lost == n_heads) return wgs;
  }
}

// The combine step carried by the partial launch itself (see decode_partial_kernel): the arguments launch_decode_combine
// takes, and one counter per head of the launch, zero between launches.
constexpr int kTailMaxParts = 16;            // partitions of a head that one workgroup combines
constexpr int kTailMaxHeads = 128;           // KV heads of such a launch
struct DecodeTail {
  const void* k_new; const void* v_new;
  void* out; int out_fp32;
  void* k_append; void* v_append; int64_t append_head_stride;
  int* counters;
};

// Counters for one context (kTailMaxHeads ints of the current device, zero for work enqueued on `stream` from now on; the
// stream is not being captured): null when all slots are taken.  They are given back with the hipEvent_t that marks the end
// of the context's last launch that used them, which is then theirs.
// tail_counters_prepare does what only the first taking on a device has to do.
void tail_counters_prepare();
int* tail_counters_take(void* stream, int* slot);
void tail_counters_give(int slot, void* busy_until);

// Split-KV decode over rows [0, n) of one slice: writes n_split partials starting at partial index part0.
// n_heads > 1: q is [n_heads][G][128], the heads' K (V) rows kv_head_stride bytes apart, their partials
// part_head_stride floats apart.
// skip_row >= 0: that row takes no part (the row of a streaming head's store that the token replaces).
hi_status launch_decode_partial(void* stream, const void* q, int G, const void* k, const void* v, int64_t n,
                                int n_split, void* partials, int part0, bool q_prescaled, int n_heads = 1,
                                int64_t kv_head_stride = 0,
                                int64_t part_head_stride = 0, int64_t skip_row = -1, const DecodeLens* lens = nullptr,
                                const DecodeTail* tail = nullptr, int n_wgs = 0, void* done = nullptr);
// tail != null (part0 = 0, n_split <= kTailMaxParts): the launch combines its partials too.
// lens != null: head h has lens->n[h] rows instead of n (n = the largest of them), n_split is the largest number of
// partitions of a head and n_wgs that of all workgroups (decode_cut), and launch_decode_combine appends
// head h's row at row lens->n[h] behind k_append / v_append (which then point at row 0 of the first head)
// Merge n_part partials with the token's own row and write out[G][128]; if k_append/v_append are not null the
// token's K/V row is also copied there (device rows of an HBM-resident cache; heads append_head_stride bytes
// apart).  n_heads > 1: q and out are [n_heads][G][128], k_new / v_new [n_heads][128].
hi_status launch_decode_combine(void* stream, const void* q, int G, const void* k_new, const void* v_new,
                                const void* partials, int n_part, void* out, int out_fp32, void* k_append,
                                void* v_append, bool q_prescaled, int n_heads = 1, int64_t part_head_stride = 0,
                                int64_t append_head_stride = 0, const DecodeLens* lens = nullptr, void* done = nullptr);

// Streaming heads (Appendix E): a head that keeps n_sink initial and n_recent recent tokens in an HBM store of
// n_sink + n_recent rows (sink token j at row j; token j >= n_sink at row n_sink + (j - n_sink) mod n_recent).
constexpr int64_t kStreamMaxRows = 1 << 22;
// One chunk of such a head (a group of n_heads, their stores store_head_stride bytes apart): row past_len + i
// sees key j iff j <= past_len + i and (j < n_sink or past_len + i - j < n_recent); the past comes from the
// store, the chunk's own rows from k_new / v_new.  Layouts of q, k_new, v_new, out as in launch_prefill.
// update: the launch takes the chunk's rows into the store itself (window_update says which, and whether it should: pf_store_rides;
// counters: one int per head if there are readers).
struct PrefillWindowUpdate { PfStoreRows rows; int* counters; };
inline bool window_update(int G, int chunk_len, int64_t past_len, int n_sink, int n_recent, int n_heads, PrefillWindowUpdate* w) {
  const int strip = prefill_strip(G);
  w->rows = pf_store_rows(pf_window_of(past_len, chunk_len, n_sink, n_recent), past_len, strip);
  w->counters = nullptr;
  const int64_t strips = ceil_div(chunk_len, strip);
  return pf_store_rides(w->rows, strips, strips * prefill_grid_y(G) * n_heads);
}
hi_status launch_prefill_window(void* stream, const void* q, int G, int chunk_len, const void* store_k,
                                const void* store_v, int64_t store_head_stride, const void* k_new, const void* v_new,
                                int64_t past_len, int n_sink, int n_recent, void* out, int out_fp32, int n_heads,
                                bool q_prescaled, const PrefillWindowUpdate* update = nullptr, void* done = nullptr);
// The chunk's rows enter the store (run it after the chunk's attention, on the same stream).
hi_status launch_stream_store_update(void* stream, const void* k_new, const void* v_new, int chunk_len,
                                     int64_t past_len, int n_sink, int n_recent, void* store_k, void* store_v,
                                     int64_t store_head_stride, int n_heads, void* done = nullptr);

// 4-bit rows of the host link: `planes` planes of `rows` rows each, plane p at base + p * pitch on either side
// (bf16 rows of 256 bytes <-> encoded rows of kLinkRowBytes4 bytes).
hi_status launch_kv_quant(void* stream, const void* src, int64_t src_pitch, void* dst, int64_t dst_pitch,
                          int64_t rows, int planes);
hi_status launch_kv_dequant(void* stream, const void* src, int64_t src_pitch, void* dst, int64_t dst_pitch,
                            int64_t rows, int planes);

}  // namespace hi
