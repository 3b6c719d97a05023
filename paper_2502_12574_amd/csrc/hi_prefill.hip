// K1: chunked-prefill attention of one (chunk, KV head) unit for gfx950.
//
// Algorithm 1, prefill phase: the chunk's G*C query rows attend over the head's past rows [0, P) (streamed into
// HBM staging) and, causally, over the chunk's own rows (Eq. 3 / Eq. 9).  The evaluation is the usual tiled
// online softmax with fp32 running max / sum / output, built for 64-wide wavefronts and the 32x32x16 bf16 MFMA:
//
//   * The transposed product S^T = K Q^T is computed, so a query row lives in ONE lane column (lane % 32):
//     its running max and sum are per-lane scalars, rescaling O is a per-lane multiply, and the fp32 scores a
//     lane holds are already laid out as the B operand of the second product O^T += V^T P^T once rounded to
//     bf16 - no cross-lane shuffles between the two contractions.
//   * The V^T operand comes from LDS transpose reads (ds_read_b64_tr_b16) of the row-major V tile.
//   * K/V tiles of 64 rows go HBM -> LDS by direct-to-LDS 128-bit loads, swizzled for conflict-free operand
//     reads.
//   * The G query heads at the same positions share a workgroup (for G = 4), so all its waves share the causal
//     boundary and sweep the same K/V tiles.
//   * Workgroups of a unit sweep the K/V rows in near lock-step, so each tile is pulled from HBM about once per
//     XCD and served to the other compute units from that XCD's L2.
//
// Two kernels share this arithmetic: prefill_kernel (4 waves, 2 LDS stages, two workgroups per compute unit, one
// barrier per tile: short chunks) and prefill_kernel_deep (8 waves, one workgroup per compute unit, the two waves of
// a SIMD alternating between a matrix phase and a softmax phase: long chunks, the fast one).
//
// The softmax state (m, l, O) can be carried across launches (one launch per staging slice) in a register-image
// workspace, which is how a unit is computed while later slices of its past are still on the host link.
#include <mutex>
#include <type_traits>
#include "hi_device.h"
#include "hi_internal.h"
#include "hi_prefill_part.h"
#include "hi_prefill_visits.h"

namespace hi {

constexpr int kPfTileRows = 64;
constexpr int kPfTileBytes = kPfTileRows * kRowBytes;   // 16 KiB of K (or V)
constexpr int kPfStageBytes = 2 * kPfTileBytes;         // K tile then V tile
constexpr int kPfStages = 2;
constexpr int kPfLdsBytes = kPfStages * kPfStageBytes;  // 64 KiB: two workgroups per compute unit

struct PrefillArgs {
  const uint16_t* q;      // [G][C][128]
  const char* ka; const char* va; int64_t na;   // past segment (not causal)
  const char* kb; const char* vb; int64_t nb;   // the chunk's own rows (causal)
  float* carry;           // [n_wg][66][256]
  void* out;              // [G][C][128]
  int G, C, first, last, out_fp32;
  float c;                // log2(e) / sqrt(d)
  int split;              // workgroups per block of positions (they divide the block's tile sequence)
  int gy;                 // grid y per head; blockIdx.y / gy is the head of a group launch
  int64_t a_head_stride;  // bytes between the heads' rows in the past segment
  int paired;             // 8-wave kernel: deep and shallow blocks of the causal triangle share their tiles
  int nbk;                // 8-wave kernel: blocks of positions per head
  int img_row;            // state images per grid row (8-wave kernel; 4-wave kernel with split > 1)
  int xcd;                // see pf_wg_index
  int tile0, past_tiles;  // 4-wave kernel with split > 1: first tile of the past segment in the unit, past tiles of the unit
  uint32_t by_split, by_nbk;       // 8-wave kernel: see pf_magic
  int a_jump_tile;        // the past segment's tiles from this one on lie a_jump_bytes further on (0: one piece)
  int64_t a_jump_bytes;
};

// Group launches: point the arguments at this workgroup's head; returns blockIdx.y within the head.
__device__ __forceinline__ int pf_select_head(PrefillArgs& a) {
  const int head = blockIdx.y / a.gy;
  const int64_t rows = (int64_t)head * a.C;
  a.q += rows * a.G * kHeadDim;
  a.out = (char*)a.out + rows * a.G * kHeadDim * (a.out_fp32 ? 4 : 2);
  a.ka += head * a.a_head_stride;
  a.va += head * a.a_head_stride;
  a.kb += rows * kRowBytes;
  a.vb += rows * kRowBytes;
  return blockIdx.y - head * a.gy;
}

// The launch's shape as the work partition takes it (strip: positions per block).
__host__ __device__ __forceinline__ PfShape pf_shape_of(const PrefillArgs& a, int strip) {
  PfShape sh;
  sh.nbk = a.nbk; sh.m = strip / kPfTileRows;
  sh.ta = (int)((a.na + kPfTileRows - 1) / kPfTileRows);
  sh.tb_all = (int)((a.nb + kPfTileRows - 1) / kPfTileRows);
  sh.split = a.split; sh.paired = a.paired; sh.carried = !a.first;
  sh.by_split = a.by_split; sh.by_nbk = a.by_nbk;
  return sh;
}

__device__ __forceinline__ int swz_k(int row) { return row & 15; }
__device__ __forceinline__ int swz_v(int row) { return ((row & 3) << 2) | (row & 2); }

// combine a value with the one held by lane ^ 32 (the other 32 K/V rows of the same query row)
__device__ __forceinline__ float max_halves(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Per-lane constants of the tile traffic, computed once per kernel.
struct PfLaneConst {
  uint32_t gk[2];    // 8-wave kernel: global byte offset inside a 64-row K tile of this lane's 2 load instructions
  uint32_t gv;       // same for V (the second instruction adds 1024)
  uint32_t koff[8];  // LDS byte offset of the K operand read for contraction step kk (sub-block 1 adds 8192)
  uint32_t voff[4];  // LDS byte offset of the V^T transpose read for dim block db (+2048 next 4 rows of the
                     // pair, +4096 second 16-row group, +8192 second sub-block)
};

// x, formed anew where this stands: what the compiler derives from it is not kept in registers across the loop around it
__device__ __forceinline__ int formed_here(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// One tile's K loads (or V loads) by the whole workgroup of 8 wavefronts, two instructions each.
// Full tiles need no vector ALU work at all; the last tile of a segment clamps its row indices (rows past the
// end re-read the last row and are masked by the caller).  lds_tile is the LDS byte address of the 16 KiB tile.
__device__ __forceinline__ void pf_issue_k(const char* kt, int rows, uint32_t lds_tile, int wave, int lane,
                                           const PfLaneConst& lc) {
  const uint32_t ldk = lds_tile + wave * 2048;
  if (rows >= kPfTileRows) {
    g2lds16_s<0>(kt, lc.gk[0], ldk);
    g2lds16_s<0>(kt, lc.gk[1], ldk + 1024);
  } else {
    lane = formed_here(lane);
    const int r_in = lane >> 4;
    const int cpos = lane & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (wave * 2 + i) * 4 + r_in;
      const int rc = r < rows ? r : rows - 1;
      g2lds16_s<0>(kt, (uint32_t)(rc * kRowBytes + ((cpos ^ swz_k(r)) << 4)), ldk + i * 1024);
    }
  }
}

__device__ __forceinline__ void pf_issue_v(const char* vt, int rows, uint32_t lds_tile, int wave, int lane,
                                           const PfLaneConst& lc) {
  const uint32_t ldv = lds_tile + wave * 2048;
  if (rows >= kPfTileRows) {
    g2lds16_s<0>(vt, lc.gv, ldv);
    g2lds16_s<1024>(vt, lc.gv, ldv);     // the immediate advances the global AND the LDS address
  } else {
    lane = formed_here(lane);
    const int r_in = lane >> 4;
    const int cpos = lane & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (wave * 2 + i) * 4 + r_in;
      const int rc = r < rows ? r : rows - 1;
      g2lds16_s<0>(vt, (uint32_t)(rc * kRowBytes + ((cpos ^ swz_v(r)) << 4)), ldv + i * 1024);
    }
  }
}

typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

struct PfState {
  f32x16 o[4];
  float m, l;
};

// Normalise one query row's accumulators and write out[g][i][:]: register r of block db is dim
// 32*db + 8*(r/4) + 4*hl + r%4; l is this half-wave's part of the row sum.
__device__ __forceinline__ void pf_write_row(void* out, int out_fp32, int C, int g, int i, int hl,
                                             const f32x16 (&o)[4], float l) {
  const float inv = 1.0f / sum_halves(l);
  if (i >= C) return;
  const int64_t base = ((int64_t)g * C + i) * kHeadDim;
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      const int dim = 32 * db + 8 * rq + 4 * hl;
      const float x0 = o[db][4 * rq] * inv, x1 = o[db][4 * rq + 1] * inv;
      const float x2 = o[db][4 * rq + 2] * inv, x3 = o[db][4 * rq + 3] * inv;
      if (out_fp32) {
        *(float4*)((float*)out + base + dim) = make_float4(x0, x1, x2, x3);
      } else {
        *(uint2*)((uint16_t*)out + base + dim) = make_uint2(pack_bf16(x0, x1), pack_bf16(x2, x3));
      }
    }
}

// S^T = K Q^T for one 64-row K tile at kt: register r of sub-block sb is tile row 32*sb + 8*(r/4) + 4*hl + r%4
// (query row = lane % 32).  The two sub-blocks' accumulation chains alternate, so consecutive MFMAs never
// depend on each other.  The first tile of a 4-wave kernel; those behind it come out of pf_tile4.
__device__ __forceinline__ void pf_scores(lds_char* kt, const PfLaneConst& lc, const bf16x8 (&qf)[8],
                                          f32x16 (&s)[2]) {
  constexpr int A = 4;           // operands read ahead: left to itself the compiler keeps two in flight and the MFMAs wait for LDS
  bf16x8 op[A + 1];
  auto read = [&](int i) __attribute__((always_inline)) { return *(lds_bf16x8*)(kt + lc.koff[i >> 1] + (i & 1) * 8192); };
#pragma unroll
  for (int r = 0; r < 16; ++r) { s[0][r] = 0.f; s[1][r] = 0.f; }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < A; ++i) op[i] = read(i);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (i + A < 16) op[(i + A) % (A + 1)] = read(i + A);
    s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[i % (A + 1)], qf[i >> 1], s[i & 1], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Online softmax of one tile's scores: per lane = per query row; the other half-wave holds the other 32 rows of
// the tile.  Updates (m, l), rescales O when the running maximum moved, and leaves the probabilities rounded to
// bf16 in pb, laid out as the B operands of the second product.
// mask_rel: rows of the tile with index > mask_rel are masked for this lane (>= 63 means no masking).
__device__ __forceinline__ void pf_softmax(f32x16 (&s)[2], PfState& st, float c, bool masked, int mask_rel, int hl,
                                           bf16x8 (&pb)[2][2]) {
  if (masked) {
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * sb + 8 * (r >> 2) + 4 * hl + (r & 3);
        if (row > mask_rel) s[sb][r] = kNegBig;
      }
  }
  float mx = s[0][0];
#pragma unroll
  for (int sb = 0; sb < 2; ++sb)
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[sb][r]);
  mx = max_halves(mx);
  const float m_new = fmaxf(st.m, mx);
  if (__builtin_amdgcn_ballot_w64(m_new > st.m) != 0) {
    const float alpha = fast_exp2((st.m - m_new) * c);
    st.l *= alpha;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
    st.m = m_new;
  }
  const float mc = st.m * c;
  float lsum = 0.f;
#pragma unroll
  for (int sb = 0; sb < 2; ++sb)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float p = fast_exp2(__builtin_fmaf(s[sb][8 * u + j], c, -mc));
        lsum += p;
        pb[sb][u][j] = (__bf16)p;
      }
  st.l += lsum;
  // the conversions belong to this phase (the values are first used after the caller's barrier)
#pragma unroll
  for (int sb = 0; sb < 2; ++sb)
#pragma unroll
    for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(pb[sb][u]));
}

// Softmax phase of a steady-state tile whose scores left the matrix pipe as s - m (relative to the running
// reference m of the row: the score accumulators start from negm = -m instead of zero), so p = 2^(c (s - m)) is
// one multiplication and one exponential.  The reference only moves when it must: the lane's share of the row sum,
// which the phase needs anyway, bounds every p of the lane, and as long as it stays below kPfSumLimit the p are as
// harmless in fp32 and bf16 as p <= 1 - no maximum is taken at all.  On the rare tile where a lane's sum exceeds
// the limit (or overflowed), the row maxima are formed, O, l, this tile's scores and negm are rescaled in place,
// and the p are computed again.  Measured against taking the maximum of every tile first: 1270 -> 1320 TFLOP/s
// on the same device (32 of the phase's ~145 vector instructions gone).
constexpr float kPfSumLimit = 4096.0f;     // 2^12

__device__ __forceinline__ void pf_softmax_fast(f32x16 (&s)[2], PfState& st, float c, f32x16& negm,
                                                bf16x8 (&pb)[2][2]) {
  // p and the lane's share of the row sum first; the sum bounds every p of the lane, so the row maximum is only
  // needed on the rare tile whose sum says the reference has to move
  auto probs = [&]() __attribute__((always_inline)) {
    float lq[4];                            // four short accumulation chains, each started by its first term
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float p = fast_exp2(s[sb][8 * u + j] * c);
          lq[2 * sb + u] = j == 0 ? p : lq[2 * sb + u] + p;
          pb[sb][u][j] = (__bf16)p;
        }
    return (lq[0] + lq[1]) + (lq[2] + lq[3]);
  };
  float lsum = probs();
  if (__builtin_amdgcn_ballot_w64(!(lsum <= kPfSumLimit)) != 0) {     // also true for inf and NaN
    float mx = s[0][0];
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[sb][r]);
    mx = max_halves(mx);
    const float d = fmaxf(mx, 0.f);       // lanes whose maximum did not move keep their reference
    const float alpha = fast_exp2(-d * c);
    st.l *= alpha;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[sb][r] -= d;
    st.m += d;
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[r] = -st.m;
    lsum = probs();
  }
  st.l += lsum;
#pragma unroll
  for (int sb = 0; sb < 2; ++sb)
#pragma unroll
    for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(pb[sb][u]));
}

// One tile of a 4-wave kernel, the next tile's scores one step ahead: the wavefront's vector ALU works on the softmax of the tile
// whose scores are in s0 (rows 0..31) and s1 while its matrix pipe forms those of the tile behind it (K tile at kt; NEXT = false:
// there is none), and the second half of the exponentials goes between the first MFMAs of O^T += V^T P^T (V tile at vt).  The next
// tile's rows 32..63 come first, into next1; its rows 0..31 then take the place of those that have become weights, in s0.
// What bounds such a tile is the number of instructions of any kind: a wavefront issues one per 6 to 7 cycles, and two share a SIMD.
// So the operands of four MFMAs are read together and waited for once, the tile loads (load(i), eight of them, M0 set one MFMA
// before by load_at(i)) go between MFMAs instead of stalling in a row, and whatever the caller can keep out of the tile loop
// (addresses, the choice of masks) it keeps out.
// mask(s0, s1) hides scores, and is called where `masked` says so.  A lane that has seen nothing yet (m == kNegBig) adds
// weights of zero.
template <bool NEXT, class Mask, class At, class Load>
__device__ __forceinline__ void pf_tile4(lds_char* kt, lds_char* vt, const PfLaneConst& lc, const bf16x8 (&qf)[8],
                                         f32x16& s0, f32x16& s1, f32x16& next1, PfState& st, float c, bool masked, Mask mask,
                                         At load_at, Load load) {
  constexpr int F = NEXT ? 0 : 16, kMax = 2;
  bf16x8 op[2][4];
  u32x4 pw[2][2];                // the weights, two to a word: B operands of the second product
  // operand i: K fragment of (sub-block, contraction step) = (1 - i / 8, i % 8), from 16 on V^T of (keys, dim block) = ((i - 16) / 4, i % 4)
  auto read = [&](int i) __attribute__((always_inline)) {
    bf16x8& x = op[(i >> 2) & 1][i & 3];
    if (i < 16) { x = *(lds_bf16x8*)(kt + lc.koff[i & 7] + (i < 8 ? 8192 : 0)); return; }
    lds_char* p = vt + lc.voff[i & 3] + ((i - 16) >> 2) * 4096;
    const bf16x4 v0 = lds_read_tr8(p), v1 = lds_read_tr8(p + 2048);
    x = (bf16x8)__builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto mfma = [&](int i) __attribute__((always_inline)) {
    if (i < 16 && !NEXT) return;
    bf16x8 (&o4)[4] = op[(i >> 2) & 1];
    if ((i & 3) == 0) asm volatile("" : "+v"(o4[0]), "+v"(o4[1]), "+v"(o4[2]), "+v"(o4[3]));     // one wait for the four
    const bf16x8 x = o4[i & 3];
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    if (NEXT && i < 16 && (i & 1) == 0) {
      load_at(i >> 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (i < 8) next1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qf[i], i == 0 ? z : next1, 0, 0, 0);
    else if (i < 16) s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qf[i - 8], i == 8 ? z : s0, 0, 0, 0);
    else st.o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, __builtin_bit_cast(bf16x8, pw[(i - 16) >> 3][(i >> 2) & 1]), st.o[i & 3], 0, 0, 0);
    if (NEXT && i < 16 && (i & 1) == 0) {
      __builtin_amdgcn_sched_barrier(0);
      load(i >> 1);
    }
    if ((i & 3) < 2 && (i | 3) + 4 < 32) {                         // the next four operands
      read((i | 3) + 1 + 2 * (i & 3));
      read((i | 3) + 2 + 2 * (i & 3));
    }
  };
  if (masked) mask(s0, s1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) read(F + i);
  float mx = s0[0];
#pragma unroll
  for (int i = 0; i < kMax; ++i) {
    mfma(i);
#pragma unroll
    for (int r = 32 / kMax * i; r < 32 / kMax * (i + 1); ++r) mx = fmaxf(mx, r < 16 ? s0[r] : s1[r & 15]);
    __builtin_amdgcn_sched_barrier(0);
  }
  const float m_new = fmaxf(st.m, max_halves(mx));
  if (__builtin_amdgcn_ballot_w64(m_new > st.m) != 0) {
    const float alpha = fast_exp2((st.m - m_new) * c);
    st.l *= alpha;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
    st.m = m_new;
  }
  const float mc = st.m > kNegBig ? st.m * c : 0.f;
  float lq[4];
  // weights 2 p, 2 p + 1 of the tile: registers 8 (p / 4 % 2) + 2 (p % 4) .. of sub-block p / 8
  auto pair = [&](int p) __attribute__((always_inline)) {
    const int sb = p >> 3, u = (p >> 2) & 1, j = 2 * (p & 3);
    float w[2], &sum = lq[2 * sb + u];
#pragma unroll
    for (int e = 0; e < 2; ++e) w[e] = fast_exp2(__builtin_fmaf(sb == 0 ? s0[8 * u + j + e] : s1[8 * u + j + e], c, -mc));
    sum = (j == 0 ? w[0] : sum + w[0]) + w[1];
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    uint32_t word = __builtin_bit_cast(uint32_t, (bf16x2){(__bf16)w[0], (__bf16)w[1]});
    asm volatile("" : "+v"(sum), "+v"(word));          // here, and not where the sums and the operand are next used
    pw[sb][u][j >> 1] = word;
  };
#pragma unroll
  for (int i = kMax; i < 8; ++i) {
    mfma(i);
#pragma unroll
    for (int p = (i - kMax) * 8 / (8 - kMax); p < (i - kMax + 1) * 8 / (8 - kMax); ++p) pair(p);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 8; i < 16; ++i) {
    mfma(i);
    if (NEXT && (i & 1)) pair(8 + ((i - 8) >> 1));
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 16; i < 32; ++i) {
    mfma(i);
    if (!NEXT && i < 20) pair(8 + i - 16);
    if (i < 28 && i % 3 == 0) pair(12 + (i - 18) / 3);
    __builtin_amdgcn_sched_barrier(0);
  }
  st.l += (lq[0] + lq[1]) + (lq[2] + lq[3]);
}

// ---- helpers of the 8-wave kernel.  Its LDS holds a ring of K tiles at [0, 64 KiB) and a ring of V tiles at
// [64 KiB, 128 KiB); the lane constants koff / voff are absolute LDS byte addresses (voff includes the V ring's
// base), so that with a compile-time ring slot every operand read is "register + immediate" (the immediate of an
// LDS instruction reaches 64 KiB).
constexpr int kPdWaves = 8;
constexpr int kPdStages = 4;
constexpr uint32_t kPdVRing = 65536;
constexpr int kPdLdsBytes = 2 * kPdStages * kPfTileBytes;   // 128 KiB

// Matrix phase of the alternating schedule: O^T += V^T P^T of the previous tile (V tile at ring offset v_off,
// probabilities pb), then S^T = K Q^T of the next (K tile at ring offset k_off), as ONE software-pipelined
// sequence of 32 MFMAs whose LDS operand reads run kPfAhead steps ahead of their use: a wavefront that has the
// matrix pipe to itself must hide the LDS latency on its own.  Operand i < 16 is the V^T fragment of step
// (sb, u, db) = (i / 8, i / 4 % 2, i % 4); operand 16 + j is the K fragment of step (kk, sb) = (j / 2, j % 2).
constexpr int kPfAhead = 4;

// step i of a matrix phase: which sub-block, half, dim block (i < 16) or contraction step (i >= 16) it is
__device__ __forceinline__ constexpr int pd_sb(int i) { return i < 16 ? i >> 3 : (i - 16) & 1; }
__device__ __forceinline__ constexpr int pd_u(int i) { return (i >> 2) & 1; }
__device__ __forceinline__ constexpr int pd_db(int i) { return i & 3; }
__device__ __forceinline__ constexpr int pd_kk(int i) { return (i - 16) >> 1; }

__device__ __forceinline__ bf16x8 pd_operand(int i, uint32_t v_off, uint32_t k_off, const PfLaneConst& lc) {
  if (i < 16) {
    const int sb = pd_sb(i), u = pd_u(i), db = pd_db(i);
    const uint32_t ad = lc.voff[db] + v_off + sb * 8192 + u * 4096;
    const bf16x4 v0 = lds_read_tr8((lds_char*)(uintptr_t)ad);
    const bf16x4 v1 = lds_read_tr8((lds_char*)(uintptr_t)(ad + 2048));
    return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  const int kk = pd_kk(i), sb = pd_sb(i);
  return *(lds_bf16x8*)(uintptr_t)(lc.koff[kk] + k_off + sb * 8192);
}

// The tile loads a wavefront issues while it runs a matrix phase: its two K and two V instructions (full tiles
// only; k / v are null otherwise) ride in the gaps between the first MFMAs, where their scalar set-up and the
// issue itself cost next to nothing.
struct PfPhaseLoads {
  const char* k;      // K tile base (global), null: nothing to issue
  const char* v;      // V tile base
  uint32_t ldk, ldv;  // LDS byte address of this wave's first destination row group in the K / V tile
};

// the first kPfAhead operands of a matrix phase (they are V^T fragments), read ahead of the phase
__device__ __forceinline__ void pd_preread(uint32_t v_off, const PfLaneConst& lc, bf16x8 (&pre)[kPfAhead]) {
#pragma unroll
  for (int i = 0; i < kPfAhead; ++i) pre[i] = pd_operand(i, v_off, 0, lc);
}

// PREREAD: the caller has already read the first kPfAhead operands into pre (during its softmax phase).
// CINIT: the score accumulators start from cinit (minus the row's running reference) instead of zero.
// EARLY_BARRIER: the workgroup barrier that ends the phase is passed before the last MFMA is issued instead of after
// it (every LDS operand of the phase is in registers by then), so the barrier's latency and the other group's first
// issue hide under that MFMA; the caller then omits its own barrier.
template <bool LOADS_ALWAYS, bool PREREAD, bool CINIT, bool EARLY_BARRIER = false>
__device__ __forceinline__ void pd_matrix_phase(uint32_t v_off, uint32_t k_off, const PfLaneConst& lc,
                                                const bf16x8 (&qf)[8], const bf16x8 (&pb)[2][2], PfState& st,
                                                f32x16 (&s)[2], const PfPhaseLoads& ld,
                                                const bf16x8 (&pre)[kPfAhead], const f32x16& cinit) {
  static_assert(kPfAhead <= 16, "pre-read operands are V fragments");
  bf16x8 op[kPfAhead + 1];
#pragma unroll
  for (int i = 0; i < kPfAhead; ++i) op[i] = PREREAD ? pre[i] : pd_operand(i, v_off, k_off, lc);
  if (!CINIT) {
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[0][r] = 0.f; s[1][r] = 0.f; }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    if (i + kPfAhead < 32) op[(i + kPfAhead) % (kPfAhead + 1)] = pd_operand(i + kPfAhead, v_off, k_off, lc);
    bf16x8 x = op[i % (kPfAhead + 1)];
    if (EARLY_BARRIER && i == 31) {
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(x) : : "memory");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    if (i < 16) {
      const int sb = pd_sb(i), u = pd_u(i), db = pd_db(i);
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, pb[sb][u], st.o[db], 0, 0, 0);
    } else {
      const int kk = pd_kk(i), sb = pd_sb(i);
      if (CINIT && kk == 0) s[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qf[kk], cinit, 0, 0, 0);
      else s[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qf[kk], s[sb], 0, 0, 0);
    }
    if (i == 1 && (LOADS_ALWAYS || ld.k)) g2lds16_s<0>(ld.k, lc.gk[0], ld.ldk);
    if (i == 3 && (LOADS_ALWAYS || ld.k)) g2lds16_s<0>(ld.k, lc.gk[1], ld.ldk + 1024);
    if (i == 5 && (LOADS_ALWAYS || ld.v)) g2lds16_s<0>(ld.v, lc.gv, ld.ldv);
    if (i == 7 && (LOADS_ALWAYS || ld.v)) g2lds16_s<1024>(ld.v, lc.gv, ld.ldv);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Lane constants of a 4-wavefront workgroup whose LDS stage is a K tile followed by a V tile (offsets relative
// to the tile).
__device__ __forceinline__ PfLaneConst pf_lane_const_4w(int lane) {      // (gk and gv stay unused: its loads are streams)
  PfLaneConst lc;
  const int hl = lane >> 5, col = lane & 31;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) lc.koff[kk] = (uint32_t)(col * kRowBytes + (((2 * kk + hl) ^ swz_k(col)) << 4));
  const int s16 = lane & 15, q16 = col >> 4;
  const int row_lo = 4 * hl + (s16 >> 2);
#pragma unroll
  for (int db = 0; db < 4; ++db) {
    const int chunk = 4 * db + 2 * q16 + ((s16 & 3) >> 1);
    lc.voff[db] = (uint32_t)(row_lo * kRowBytes + ((chunk ^ swz_v(row_lo)) << 4) + ((s16 & 1) << 3));
  }
  return lc;
}

// A 4-wave kernel's load stream, with the lane's byte offsets of its four instructions.
struct PfStream4 : PfLoads { uint32_t off[4]; };
// V = false: K tiles, true: V tiles; row_of(r): where row r of the tile lies, in rows behind the stream's base
template <bool V, class RowOf>
__device__ __forceinline__ void pf_stream4_offsets(PfStream4& w, int wave, int lane, RowOf row_of) {
  const int r_in = lane >> 4, cpos = lane & 15;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (wave * 4 + i) * 4 + r_in;
    w.off[i] = (uint32_t)row_of(r) * kRowBytes + ((cpos ^ (V ? swz_v(r) : swz_k(r))) << 4);
  }
}
__device__ __forceinline__ void pf_stream4_issue(const PfStream4& w, uint32_t lds) {
#pragma unroll
  for (int i = 0; i < 4; ++i) g2lds16_s<0>(w.base, w.off[i], lds + i * 1024);
}

// All visits of a workgroup.  LDS: two places for K tiles, then two for V tiles; on entry the first two K tiles and the first V tile are
// on their way, sk stands at visit 2 and sv at visit 1 (STRAIGHT: the first K tile only, and both stand at visit 1).  masked(v): visit v hides rows of some query row of the wavefront; seen(): rows of
// that visit that the lane's query row sees.  Hidden scores become kNegBig as bit operations (comparisons and selects per
// element became branches, 83 -> 77 us a launch of prefill_window_kernel).
template <bool STRAIGHT, class GoOnK, class GoOnV, class Masked, class Seen>
__device__ __forceinline__ void pf_sweep4(lds_char* lds, uint32_t lds_wave, const PfLaneConst& lc, const bf16x8 (&qf)[8], PfState& st,
                                          float c, int T, int lane, PfStream4& sk, PfStream4& sv, GoOnK go_on_k, GoOnV go_on_v,
                                          Masked masked, Seen seen) {
  auto hide = [&](int v, f32x16& s0, f32x16& s1) __attribute__((always_inline)) {
    const uint64_t rows = seen(v) >> (4 * (formed_here(lane) >> 5));
    const uint32_t bits[2] = {(uint32_t)rows, (uint32_t)(rows >> 32)};
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        f32x16& s = sb == 0 ? s0 : s1;
        const uint32_t t = (uint32_t)__builtin_amdgcn_sbfe((int)bits[sb], 8 * (r >> 2) + (r & 3), 1);
        s[r] = __uint_as_float((__float_as_uint(s[r]) & t) | (__float_as_uint(kNegBig) & ~t));
      }
  };
  if constexpr (STRAIGHT) {
    auto step = [&](int v, auto parity) __attribute__((always_inline)) {
      constexpr int odd = decltype(parity)::value;
      wait_vmcnt<0>();
      __syncthreads();
      if (v + 1 < T) {
        pf_stream4_issue(sk, lds_wave + (1 - odd) * kPfTileBytes);
        pf_stream4_issue(sv, lds_wave + kPfStageBytes + (1 - odd) * kPfTileBytes);
        go_on_k();
        go_on_v();
      }
      f32x16 s[2], none;
      pf_scores(lds + odd * kPfTileBytes, lc, qf, s);
      const bool hides = masked(v);
      auto mask = [&](f32x16& s0, f32x16& s1) __attribute__((always_inline)) { hide(v, s0, s1); };
      auto nothing = [](int) __attribute__((always_inline)) {};
      pf_tile4<false>(lds, lds + kPfStageBytes + odd * kPfTileBytes, lc, qf, s[0], s[1], none, st, c, hides, mask, nothing, nothing);
    };
    int v = 0;
    for (; v + 1 < T; v += 2) {
      step(v, std::integral_constant<int, 0>());
      step(v + 1, std::integral_constant<int, 1>());
    }
    if (v < T) step(v, std::integral_constant<int, 0>());
    return;
  }
  f32x16 s0, s1a, s1b;         // scores of a visit's rows 0..31, and of its rows 32..63 (even and odd visits)
  wait_vmcnt<0>();
  __syncthreads();
  {
    f32x16 s[2];
    pf_scores(lds, lc, qf, s);
    s0 = s[0];
    s1a = s[1];
  }
  // Visit v: its weights and sums, and the scores of visit v + 1.  On entry both of v + 1's K rows and v's V rows are on their way;
  // behind the barrier everybody is done with the K tile of v and the V tile of v - 1, whose places take the next ones.
  // parity: v % 2, a constant where every LDS address shall be an immediate.
  auto step = [&](int v, auto parity, auto more, f32x16& cur, f32x16& nxt) __attribute__((always_inline)) {
    const int odd = parity;
    constexpr bool NEXT = decltype(more)::value;
    wait_vmcnt<0>();
    __syncthreads();
    const bool hides = masked(v);
    auto mask = [&](f32x16& s0, f32x16& s1) __attribute__((always_inline)) { hide(v, s0, s1); };
    // K of visit v + 2 into the place of v's, V of v + 1 into that of v - 1's
    auto at = [&](int i) __attribute__((always_inline)) {
      set_m0(lds_wave + (i < 4 ? odd * kPfTileBytes : kPfStageBytes + (1 - odd) * kPfTileBytes) + (i & 3) * 1024);
    };
    auto load = [&](int i) __attribute__((always_inline)) { g2lds16_m0(i < 4 ? sk.base : sv.base, i < 4 ? sk.off[i] : sv.off[i & 3]); };
    pf_tile4<NEXT>(lds + (1 - odd) * kPfTileBytes, lds + kPfStageBytes + odd * kPfTileBytes, lc, qf, s0, cur, nxt, st, c, hides, mask,
                   at, load);
    if (NEXT) {
      go_on_k();
      go_on_v();
    }
  };
  int v = 0;
  for (;;) {
    if (v + 1 >= T) break;
    step(v++, std::integral_constant<int, 0>(), std::true_type(), s1a, s1b);
    if (v + 1 >= T) { s1a = s1b; break; }
    step(v++, std::integral_constant<int, 1>(), std::true_type(), s1b, s1a);
  }
  step(v, v & 1, std::false_type(), s1a, s1b);
}

// The 4-wave kernel: short chunks, and units of few workgroups.  One wavefront or two on a SIMD, so what bounds it is a wavefront's own
// chain: matrix phase, softmax, matrix phase of one tile after the other.  The scores are formed one visit ahead (pf_tile4; K and V
// tiles have two places each in LDS, the loads are streams), straight through before: 1239 rows of 6 heads of 4 queries 31 -> 27 us,
// 1500 of one head of 2 behind 395 42.1 -> 35.3, 1000 of 8 heads of 4 27.2 -> 24.2, 204 of one 9.0 -> 8.5; ranges of 5 to 7 tiles
// (276 rows of 2 heads behind 3111) the same 13.5.
// STRAIGHT: scores, softmax and product of a tile one after the other, its loads a tile ahead in a row behind the barrier; the same bits.  For
// launches of more workgroups than compute units: two wavefronts share each SIMD and hide each other's softmax, so that a visit ahead gains
// nothing there, and what it costs is the clock of the kernels around it.  A prompt of 12288 rows of 8 heads, two a call, in chunks of
// 5955, whose last chunk is cut into 504 workgroups: 1885 us a pass with this kernel a visit ahead (at 2.11 GHz; every other kernel
// of the pass 3 % slower too), 1815 straight (2.18 GHz); 16 two-query heads one by one in chunks of 5266 2675 and 2650; 2 rows of 8 heads
// behind 88778 86.2 and 85.0, 20 behind 67854 91.2 and 87.3.  With 256 workgroups and fewer it is the other way round: calls of 209 rows of a
// one-query head behind 32701 (116 workgroups) 1530 us for 32 of them against 1640, 459 behind 459 (30) 18.6 against 20.2.
// SPLIT: a.split workgroups per block of positions, each on its range of the unit's tiles (pf_narrow_range) with a state
// image of its own, merged after the last launch (prefill_merge4_kernel).
template <bool SPLIT, bool STRAIGHT>
__global__ __launch_bounds__(256, 2) void prefill_kernel(PrefillArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds_raw[kPfLdsBytes];
  lds_char* lds = (lds_char*)lds_raw;
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
  const int lane = lane_id();
  const int wave = wave_id();
  const int hl = lane >> 5;            // which half of the wavefront
  const int col = lane & 31;           // query row within the wave's 32

  const int gl = a.G < 4 ? a.G : 4;
  const int strip = 32 * (4 / gl);
  int bx = gridDim.x - 1 - blockIdx.x;              // deepest causal rows are dispatched first
  int64_t image = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  bool fresh = a.first != 0;
  int a0 = 0, b0 = 0, ta_range = 0, t_range = 0;    // SPLIT: first past and own tile of this workgroup, its tiles
  if constexpr (SPLIT) {
    const int blocks = a.img_row / a.split;         // neighbours in the numbering sweep the same range
    const int w = pf_wg_index(blockIdx.x, gridDim.x, a.xcd), k = w / blocks;
    bx = blocks - 1 - w % blocks;
    const int own = (int)(((a.C < bx * strip + strip ? a.C : bx * strip + strip) + kPfTileRows - 1) / kPfTileRows);
    const int ta_launch = (int)((a.na + kPfTileRows - 1) / kPfTileRows);
    const PfRange r = pf_narrow_range(a.past_tiles, own, k, a.split, a.tile0, ta_launch, a.last);
    if (r.lo >= r.hi) return;
    fresh = r.fresh != 0;
    image = (int64_t)blockIdx.y * a.img_row + k * blocks + bx;
    const int lo = __builtin_amdgcn_readfirstlane(r.lo), hi = __builtin_amdgcn_readfirstlane(r.hi);
    a0 = lo - a.tile0;
    b0 = lo > a.past_tiles ? lo - a.past_tiles : 0;
    ta_range = (hi < a.past_tiles ? hi : a.past_tiles) - lo;
    if (ta_range < 0) ta_range = 0;
    t_range = hi - lo;
  }
  const int g = pf_select_head(a) * 4 + (wave % gl);
  const int i0 = bx * strip + 32 * (wave / gl);     // first query position of this wave
  const int i_hi = bx * strip + strip - 1;          // last query position of the workgroup
  int qi = i0 + col;
  const int my_i = qi;
  if (qi > a.C - 1) qi = a.C - 1;

  const PfLaneConst lc = pf_lane_const_4w(lane);

  // Q^T operand: lane holds q[g][qi][16*kk + 8*hl .. +7]
  bf16x8 qf[8];
  {
    const uint16_t* qrow = a.q + ((int64_t)g * a.C + qi) * kHeadDim + 8 * hl;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, *(const uint4*)(qrow + 16 * kk));
  }

  // tiles: segment A (all of it), then the part of segment B at or below the workgroup's causal boundary
  PfNarrow n;
  n.na = (int)a.na; n.nb = (int)a.nb;               // (a 64-bit comparison would put all that follows from it into vector registers)
  n.a0 = a0; n.b0 = b0;
  n.jump_tile = SPLIT ? a.a_jump_tile : 0;
  n.jump_bytes = a.a_jump_bytes;
  const int nb_vis = n.nb < i_hi + 1 ? n.nb : i_hi + 1;
  n.ta = SPLIT ? ta_range : n.na / kPfTileRows + (n.na % kPfTileRows != 0);
  n.T = SPLIT ? t_range : n.ta + (nb_vis + kPfTileRows - 1) / kPfTileRows;           // >= 1

  PfStream4 sk, sv;
  sk.v = sv.v = sk.usual = sv.usual = 0;
  auto meet = [&](PfStream4& w, auto v_tag) __attribute__((always_inline)) {
    constexpr bool V = decltype(v_tag)::value;
    int rows;
    if (pf_narrow_meet(w, n, V ? a.va : a.ka, V ? a.vb : a.kb, rows))
      pf_stream4_offsets<V>(w, wave, formed_here(lane), [&](int r) { return r < rows ? r : rows - 1; });
  };
  using KPlane = std::false_type;
  using VPlane = std::true_type;
  auto go_on_k = [&]() __attribute__((always_inline)) { if (pf_loads_next(sk, n.T)) meet(sk, KPlane()); };
  auto go_on_v = [&]() __attribute__((always_inline)) { if (pf_loads_next(sv, n.T)) meet(sv, VPlane()); };
  const uint32_t lds_wave = lds_base + wave * 4096;
  meet(sk, KPlane());
  meet(sv, VPlane());
  pf_stream4_issue(sk, lds_wave);
  pf_stream4_issue(sv, lds_wave + kPfStageBytes);
  go_on_k();
  go_on_v();
  if (!STRAIGHT) {
    pf_stream4_issue(sk, lds_wave + kPfTileBytes);
    go_on_k();
  }

  PfState st;
  float* carry = a.carry + image * (kCarryFloatsPerLane * kWgThreads) + threadIdx.x;
  if (fresh) {
    st.m = kNegBig;
    st.l = 0.f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] = 0.f;
  } else {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] = carry[(db * 16 + r) * kWgThreads];
    st.m = carry[64 * kWgThreads];
    st.l = carry[65 * kWgThreads];
  }
  // the compiler's own waits for the loads above belong here, not inside the tile loop
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) asm volatile("" : "+v"(qf[kk]));
  asm volatile("" : "+v"(st.m), "+v"(st.l));
#pragma unroll
  for (int db = 0; db < 4; ++db) asm volatile("" : "+v"(st.o[db]));

  const PfOpen open = pf_narrow_open(n, i0);
  pf_sweep4<STRAIGHT>(lds, lds_wave, lc, qf, st, a.c, n.T, lane, sk, sv, go_on_k, go_on_v,
            [&](int v) __attribute__((always_inline)) { return !(v < open.a || (v >= n.ta && v < open.b)); },
            [&](int v) __attribute__((always_inline)) { return pf_narrow_seen(n, v, i0 + (formed_here(lane) & 31)); });

  if (SPLIT || !a.last) {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) carry[(db * 16 + r) * kWgThreads] = st.o[db][r];
    carry[64 * kWgThreads] = st.m;
    carry[65 * kWgThreads] = st.l;
    return;
  }

  pf_write_row(a.out, a.out_fp32, a.C, g, my_i, hl, st.o, st.l);
}

// ---------------------------------------------------------------------------------------------------------
// The 8-wave kernel: 8 wavefronts per workgroup (two per SIMD, 32 positions each: the G query heads at 64
// positions for G = 4), one workgroup per compute unit, four K and four V tiles in LDS, every K/V byte pulled
// from L2 serves 256 query rows.  The two wavefronts of a SIMD alternate between a matrix phase and a softmax
// phase (see the schedule below); used for chunks long enough to give every compute unit a workgroup.
__global__ __launch_bounds__(512, 2) void prefill_kernel_deep(PrefillArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char lds_dyn[];
  lds_char* lds = (lds_char*)lds_dyn;
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
  const int lane = lane_id();
  const int wave = wave_id();
  const int hl = lane >> 5;
  const int col = lane & 31;

  const int gl = a.G < 4 ? a.G : 4;
  const int strip = 32 * (kPdWaves / gl);
  const int g = pf_select_head(a) * 4 + (wave % gl);

  PfLaneConst lc;
  {
    const int r_in = lane >> 4, cpos = lane & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (wave * 2 + i) * 4 + r_in;
      lc.gk[i] = (uint32_t)(r * kRowBytes + ((cpos ^ swz_k(r)) << 4));
    }
    const int r0 = wave * 8 + r_in;
    lc.gv = (uint32_t)(r0 * kRowBytes + ((cpos ^ swz_v(r0)) << 4));
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      lc.koff[kk] = lds_base + (uint32_t)(col * kRowBytes + (((2 * kk + hl) ^ swz_k(col)) << 4));
    const int s16 = lane & 15, q16 = col >> 4;
    const int row_lo = 4 * hl + (s16 >> 2);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      const int chunk = 4 * db + 2 * q16 + ((s16 & 3) >> 1);
      lc.voff[db] = lds_base + kPdVRing +
                    (uint32_t)(row_lo * kRowBytes + ((chunk ^ swz_v(row_lo)) << 4) + ((s16 & 1) << 3));
    }
  }


  // How the launch divides its tiles among workgroups is pure arithmetic on the launch's shape: at most two passes
  // per workgroup, each over a range of one block's tile sequence (its past tiles, then the chunk's own tiles up to
  // the block's causal boundary), each with a softmax state of its own.
  const PfShape sh = pf_shape_of(a, strip);
  constexpr int kLanes = kPdWaves * 64;
  constexpr int kImageFloats = kCarryFloatsPerLane * kLanes;
  float* const images = a.carry + (int64_t)blockIdx.y * a.img_row * kImageFloats + threadIdx.x;
  // the pass that holds past tiles goes first, so that the workgroups of a range walk the past rows in step
  const int wg = pf_wg_index(blockIdx.x, gridDim.x, a.xcd);
  int first_which = 0;
  {
    const PfPass d = pf_pass(sh, wg, 0, a.last), sw = pf_pass(sh, wg, 1, a.last);
    if (sw.run && sw.a1 > sw.a0 && !(d.run && d.a1 > d.a0)) first_which = 1;
  }
#pragma nounroll
  for (int pi = 0; pi < 2; ++pi) {
    const PfPass ps = pf_pass(sh, wg, first_which ^ pi, a.last);
    if (ps.init) {                 // a range without tiles in the first launch of a unit: an empty state
      float* im = images + (int64_t)ps.store * kImageFloats;
#pragma unroll
      for (int i = 0; i < 64; ++i) im[i * kLanes] = 0.f;
      im[64 * kLanes] = kNegBig;
      im[65 * kLanes] = 0.f;
    }
    if (!ps.run) continue;
    __syncthreads();               // the LDS rings are free again (a previous pass may still be reading V tiles)
    const int bx = ps.bx;
    const int i0 = bx * strip + 32 * (wave / gl);
    int qi = i0 + col;
    const int my_i = qi;
    if (qi > a.C - 1) qi = a.C - 1;

    // Q^T operand: lane holds q[g][qi][16*kk + 8*hl .. +7]
    bf16x8 qf[8];
    {
      const uint16_t* qrow = a.q + ((int64_t)g * a.C + qi) * kHeadDim + 8 * hl;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, *(const uint4*)(qrow + 16 * kk));
    }

    // this pass's tiles: past rows [64 a0, min(64 a1, na)) of the launch, own tiles [b0, b1) of the chunk
    const char* const ka_p = a.ka + (int64_t)ps.a0 * kPfTileBytes;
    const char* const va_p = a.va + (int64_t)ps.a0 * kPfTileBytes;
    int64_t na_p = (int64_t)ps.a1 * kPfTileRows;
    if (na_p > a.na) na_p = a.na;
    na_p -= (int64_t)ps.a0 * kPfTileRows;
    const int b_t0 = ps.b0;
    const int tb = ps.b1 - ps.b0;

    PfState st;
    if (ps.load < 0) {
      st.m = kNegBig;
      st.l = 0.f;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.o[db][r] = 0.f;
    } else {
      const float* im = images + (int64_t)ps.load * kImageFloats;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.o[db][r] = im[(db * 16 + r) * kLanes];
      st.m = im[64 * kLanes];
      st.l = im[65 * kLanes];
    }
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) asm volatile("" : "+v"(qf[kk]));
    asm volatile("" : "+v"(st.m), "+v"(st.l));
#pragma unroll
    for (int db = 0; db < 4; ++db) asm volatile("" : "+v"(st.o[db]));

    const int ta = (int)((na_p + kPfTileRows - 1) / kPfTileRows);
    const int T = ta + tb;
    const int tb_base = b_t0 - ta;      // tile t >= ta of the sweep is tile t + tb_base of the chunk's own rows

    // K tile t (which = 0) or V tile t (which = 1) of the sweep: this wave's share of its loads
    auto issue = [&](int t, int which) __attribute__((always_inline)) {
      if (t >= T) return;
      const bool in_b = t >= ta;
      const int64_t row0 = (int64_t)(in_b ? t + tb_base : t) * kPfTileRows;
      const int64_t left = (in_b ? a.nb : na_p) - row0;
      const int rows = left < kPfTileRows ? (int)left : kPfTileRows;
      const uint32_t slot = lds_base + (uint32_t)(t & (kPdStages - 1)) * kPfTileBytes;
      if (which == 0) pf_issue_k((in_b ? a.kb : ka_p) + row0 * kRowBytes, rows, slot, wave, lane, lc);
      else pf_issue_v((in_b ? a.vb : va_p) + row0 * kRowBytes, rows, slot + kPdVRing, wave, lane, lc);
    };
    // Every wave issues, in this order: K0 | K1 V0 | K2 V1 | then, in the matrix phase of tile t, K(t+3) V(t+2)
    // (2 instructions each).  The one wait per tile is at the end of the softmax phase of tile t: everything up to
    // V(t+1) has landed when at most K(t+3) V(t+2) are still in flight.
    auto wait_landed = [&](int t) {
      if (t + 3 < T) wait_vmcnt<4>();
      else wait_vmcnt<0>();
    };
    auto phase_barrier = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
      __builtin_amdgcn_sched_barrier(0);
    };

    // The two wavefronts of a SIMD alternate: while one runs its matrix phase (O += V P of the previous tile, then
    // the scores of the next), the other runs its softmax phase on the vector ALU.  Both groups execute the same
    // program with two barriers per tile; group 1 passes one extra barrier first, so it is always one phase behind
    // (and group 0 passes one extra at the end: every wave executes the same number of barriers).
    //   phase index (barriers passed so far):  group 0: matrix(t) = 2t, softmax(t) = 2t + 1;  group 1: one later.
    //   Reads: K(t) in phases 2t, 2t+1; V(t) in phases 2t+1 (operands read ahead during softmax(t)) .. 2t+3.
    //   Writes: K(t+3) replaces K(t-1) (last read in phase 2t-1) and V(t+2) replaces V(t-2) (last read in phase
    //   2t-1): both are issued in matrix(t), phase >= 2t.
    //   Landing: each wave waits at the end of softmax(t-1) for its share of everything up to V(t): that is phase
    //   2t at the latest, and K(t+1) is first read in phase 2t+2, V(t) in phase 2t+1.
    const int group = wave >> 2;       // waves w and w + 4 share a SIMD
    const float c = a.c;
    wait_vmcnt<0>();                   // the waits below count this pass's tile loads only (a previous pass's stores are done)
    issue(0, 0);
    issue(1, 0); issue(0, 1);
    issue(2, 0); issue(1, 1);
    wait_landed(-1);                           // K(0), K(1), V(0)
    phase_barrier();
    if (group == 1) phase_barrier();

    f32x16 sc[2];
    bf16x8 pb[2][2];
    auto softmax_phase = [&](int t) __attribute__((always_inline)) {
      const bool in_b = t >= ta;
      const int64_t j0 = (int64_t)(in_b ? t + tb_base : t) * kPfTileRows;
      const int64_t n_seg = in_b ? a.nb : na_p;
      const bool masked = (j0 + kPfTileRows > n_seg) || (in_b && (j0 + kPfTileRows - 1 > i0));
      int rel = kPfTileRows;
      if (masked) {
        int64_t lim = n_seg - 1;
        if (in_b && (int64_t)my_i < lim) lim = my_i;
        const int64_t d = lim - j0;
        rel = d < -1 ? -1 : (d > kPfTileRows ? kPfTileRows : (int)d);
      }
      pf_softmax(sc, st, c, masked, rel, hl, pb);
    };
    // tile 0: nothing to accumulate yet
    issue(3, 0);
    issue(2, 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) { sc[0][r] = 0.f; sc[1][r] = 0.f; }
#pragma unroll
    for (int i = 16; i < 32; ++i)
      sc[pd_sb(i)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pd_operand(i, 0, 0, lc), qf[pd_kk(i)], sc[pd_sb(i)], 0, 0, 0);
    phase_barrier();
    softmax_phase(0);
    wait_landed(0);
    phase_barrier();
    bf16x8 pre[kPfAhead];
    f32x16 negm;       // minus the row's running reference, the start value of the steady-state score accumulators
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[r] = 0.f;
    // any tile t >= 1
    auto generic_tile = [&](int t) __attribute__((always_inline)) {
      // K(t+3) and V(t+2): full tiles are issued from inside the matrix phase, partial ones (row clamping) here
      PfPhaseLoads ld;
      ld.k = ld.v = nullptr;
      const int tk = t + 3, tv = t + 2;
      const bool kb = tk >= ta, vb = tv >= ta;
      const int64_t krow0 = (int64_t)(kb ? tk + tb_base : tk) * kPfTileRows;
      const int64_t vrow0 = (int64_t)(vb ? tv + tb_base : tv) * kPfTileRows;
      const bool kfull = tk < T && (kb ? a.nb : na_p) - krow0 >= kPfTileRows;
      const bool vfull = tv < T && (vb ? a.nb : na_p) - vrow0 >= kPfTileRows;
      if (kfull) ld.k = (kb ? a.kb : ka_p) + krow0 * kRowBytes; else issue(tk, 0);
      if (vfull) ld.v = (vb ? a.vb : va_p) + vrow0 * kRowBytes; else issue(tv, 1);
      ld.ldk = lds_base + (uint32_t)(tk & (kPdStages - 1)) * kPfTileBytes + wave * 2048;
      ld.ldv = lds_base + kPdVRing + (uint32_t)(tv & (kPdStages - 1)) * kPfTileBytes + wave * 2048;
      pd_matrix_phase<false, false, false>((uint32_t)((t - 1) & (kPdStages - 1)) * kPfTileBytes,
                                           (uint32_t)(t & (kPdStages - 1)) * kPfTileBytes, lc, qf, pb, st, sc, ld, pre,
                                           negm);
      phase_barrier();
      softmax_phase(t);
      wait_landed(t);
      phase_barrier();
    };
    // Steady state: tile t of the past segment with K(t+3), V(t+2) full tiles of the same segment and nothing
    // masked.  The stage t % 4 is a compile-time constant (every LDS address is an immediate) and the scalar work
    // per tile is two pointer increments.
    const char* kp = ka_p;     // K(t+3), V(t+2) of the next fast tile
    const char* vp = va_p;
    const uint32_t ld_wave = lds_base + wave * 2048;
    auto fast_tile = [&](auto stage_tag) __attribute__((always_inline)) {
      constexpr int S = decltype(stage_tag)::value;
      PfPhaseLoads ld;
      ld.k = kp;
      ld.v = vp;
      ld.ldk = ld_wave + ((S + 3) & 3) * kPfTileBytes;
      ld.ldv = ld_wave + kPdVRing + ((S + 2) & 3) * kPfTileBytes;
      __builtin_amdgcn_s_setprio(2);
      pd_matrix_phase<true, true, true, true>(((S + 3) & 3) * kPfTileBytes, S * kPfTileBytes, lc, qf, pb, st, sc, ld,
                                              pre, negm);       // passes the phase's barrier itself
      __builtin_amdgcn_s_setprio(0);
      pd_preread(S * kPfTileBytes, lc, pre);     // V(t), for the next matrix phase
      __builtin_amdgcn_sched_barrier(0);
      pf_softmax_fast(sc, st, c, negm, pb);
      wait_vmcnt<4>();
      phase_barrier();
      kp += kPfTileBytes;
      vp += kPfTileBytes;
    };
    // A run of steady-state tiles [t, t_end) of one segment whose tile 0 is tile `tile0` of the sweep and whose rows
    // start at kbase / vbase: general tiles up to a multiple of four, then the unrolled loop.
    int t = 1;
    auto fast_run = [&](int t_end, const char* kbase, const char* vbase, int tile0) __attribute__((always_inline)) {
      if (t_end - t < 8) return;
      while (t & 3) { generic_tile(t); ++t; }
      kp = kbase + (int64_t)(t + 3 - tile0) * kPfTileBytes;
      vp = vbase + (int64_t)(t + 2 - tile0) * kPfTileBytes;
      pd_preread((uint32_t)((t - 1) & (kPdStages - 1)) * kPfTileBytes, lc, pre);
#pragma unroll
      for (int r = 0; r < 16; ++r) negm[r] = -st.m;
      for (; t + 4 <= t_end; t += 4) {
        fast_tile(std::integral_constant<int, 0>());
        fast_tile(std::integral_constant<int, 1>());
        fast_tile(std::integral_constant<int, 2>());
        fast_tile(std::integral_constant<int, 3>());
      }
    };
    // past segment: tile t qualifies if K(t+3) and V(t+2) are full tiles of the segment too
    fast_run((int)(na_p / kPfTileRows) - 3, ka_p, va_p, 0);
    // the chunk's own rows: tiles that end at or before the first position of the workgroup are not masked for any
    // of its lanes (own tile j = t + tb_base; its rows are 64 j .. 64 j + 63)
    while (t < ta && t < T) { generic_tile(t); ++t; }
    {
      const int64_t unmasked = ((int64_t)bx * strip + 1) / kPfTileRows;          // own tiles 0 .. unmasked - 1
      const int64_t loadable = a.nb / kPfTileRows - 3;                           // K(t+3), V(t+2) full
      const int64_t j_end = unmasked < loadable ? unmasked : loadable;
      const int64_t t_end = j_end - tb_base < T - 3 ? j_end - tb_base : T - 3;
      fast_run((int)t_end, a.kb, a.vb, -tb_base);
    }
    for (; t < T; ++t) generic_tile(t);
    {
      const uint32_t v_off = (uint32_t)((T - 1) & (kPdStages - 1)) * kPfTileBytes;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        st.o[pd_db(i)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pd_operand(i, v_off, 0, lc), pb[pd_sb(i)][pd_u(i)],
                                                                 st.o[pd_db(i)], 0, 0, 0);
    }
    if (group == 0) phase_barrier();

    if (ps.store >= 0) {
      float* im = images + (int64_t)ps.store * kImageFloats;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) im[(db * 16 + r) * kLanes] = st.o[db][r];
      im[64 * kLanes] = st.m;
      im[65 * kLanes] = st.l;
    } else {
      pf_write_row(a.out, a.out_fp32, a.C, g, my_i, hl, st.o, st.l);
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// The 8-wave kernel on the 16x16x32 bf16 MFMA.  Same tiles, LDS rings, alternating schedule, barrier protocol, pass
// loop and work partition as prefill_kernel_deep; what differs is the matrix instruction and with it the register
// layouts (and so the layout of a state image, which has a merge kernel of its own).  Measured on this part, a
// register-only loop of v_mfma_f32_16x16x32_bf16 on random operands sustains 2.10 PFLOP/s under the board's power limit
// where v_mfma_f32_32x32x16_bf16 sustains 1.84: less energy per flop, and the kernel runs against that limit.
// PRESCALED: the queries carry the softmax scale (a.c is 1), and the steady-state softmax has no multiplication.
//   * A wavefront still owns 32 query rows of one query head, now as two blocks of 16 (qb = 0, 1): lane = (query
//     l % 16 of each block, g = l / 16).  S^T = K Q^T per 16-key block kb: register r of s[kb][qb] is key row
//     16 kb + 4 g + r.  A K operand read (16 keys x 32 dims) feeds the MFMAs of both query blocks.
//   * O^T += V^T P^T over 32 keys per MFMA: the lane's 4 + 4 scores of key blocks 2 kp and 2 kp + 1 are, rounded to
//     bf16, its B operand (contraction index 8 g + j is key 32 kp + 16 (j / 4) + 4 g + j % 4), and the V^T operand
//     takes the same permutation: two transpose reads of 4 consecutive rows each.  Register r of o[db][qb] is dim
//     16 db + 4 g + r of the lane's query in block qb.
//   * A lane serves two query rows, so it carries two running references and two shares of the row sums.
//   * V tiles take one more swizzle bit than in the other kernels (rows 4 apart are read by neighbouring 16-lane
//     groups of one transpose read and must not share banks).
static_assert(kCarryFloatsPerLane >= 68, "a state image holds 64 O^T accumulators, two running maxima and two row-sum shares per lane");

__device__ __forceinline__ int swz_v16(int row) { return swz_v(row) ^ (((row >> 2) & 1) << 1); }

struct PfLane16 {
  uint32_t gk[2];     // global byte offset inside a 64-row K tile of this lane's 2 load instructions
  uint32_t gv[2];     // same for V
  uint32_t koff[4];   // absolute LDS address of the K operand read of contraction step kk (key block kb adds 4096)
  uint32_t voff[8];   // absolute LDS address of the V^T transpose read of dim block db (+4096: the second 16 rows
                      // of the key pair, +8192: key pair 1)
};

// The 4-register accumulator tiles of the 16x16x32 MFMA are kept as quarters of 16-register vectors: a result that has to
// land in a quarter of the vector its accumulator came from is computed in place, where free-standing 4-register tiles
// were moved from tuple to tuple by most MFMAs (and the register file overflowed).
__device__ __forceinline__ f32x4 q4_get(const f32x16& v, int k) { return (f32x4){v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]}; }
__device__ __forceinline__ void q4_set(f32x16& v, int k, const f32x4& x) {
  v[4 * k] = x[0]; v[4 * k + 1] = x[1]; v[4 * k + 2] = x[2]; v[4 * k + 3] = x[3];
}

// NQ: blocks of 16 query rows the wavefront works on (2; 1 where the chunk's end leaves the second one empty)
template <int NQ>
struct PfState16 {
  f32x16 o[2 * NQ];   // tile (db, qb) is quarter (NQ db + qb) % 4 of o[(NQ db + qb) / 4]
  float m[NQ], l[NQ];
};
// element r of accumulator tile (db, qb) of O^T, and of score tile (kb, qb) in f32x16 s[NQ]
#define PF16_O(st, db, qb, r) (st).o[(NQ * (db) + (qb)) >> 2][4 * ((NQ * (db) + (qb)) & 3) + (r)]
#define PF16_S(s, kb, qb, r) (s)[(NQ * (kb) + (qb)) >> 2][4 * ((NQ * (kb) + (qb)) & 3) + (r)]

__device__ __forceinline__ void pf16_issue_k(const char* kt, int rows, uint32_t lds_tile, int wave, int lane,
                                             const PfLane16& lc) {
  const uint32_t ldk = lds_tile + wave * 2048;
  if (rows >= kPfTileRows) {
    g2lds16_s<0>(kt, lc.gk[0], ldk);
    g2lds16_s<0>(kt, lc.gk[1], ldk + 1024);
  } else {
    const int r_in = lane >> 4, cpos = lane & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (wave * 2 + i) * 4 + r_in;
      const int rc = r < rows ? r : rows - 1;
      g2lds16_s<0>(kt, (uint32_t)(rc * kRowBytes + ((cpos ^ swz_k(r)) << 4)), ldk + i * 1024);
    }
  }
}

__device__ __forceinline__ void pf16_issue_v(const char* vt, int rows, uint32_t lds_tile, int wave, int lane,
                                             const PfLane16& lc) {
  const uint32_t ldv = lds_tile + wave * 2048;
  if (rows >= kPfTileRows) {
    g2lds16_s<0>(vt, lc.gv[0], ldv);
    g2lds16_s<0>(vt, lc.gv[1], ldv + 1024);
  } else {
    const int r_in = lane >> 4, cpos = lane & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (wave * 2 + i) * 4 + r_in;
      const int rc = r < rows ? r : rows - 1;
      g2lds16_s<0>(vt, (uint32_t)(rc * kRowBytes + ((cpos ^ swz_v16(r)) << 4)), ldv + i * 1024);
    }
  }
}

// operand i of a matrix phase: i < 16 the V^T fragment of (key pair, dim block) = (i / 8, i % 8), i >= 16 the K
// fragment of (contraction step, key block) = ((i - 16) / 4, (i - 16) % 4); each feeds the MFMAs of both query blocks
__device__ __forceinline__ constexpr int pd16_kp(int i) { return i >> 3; }
__device__ __forceinline__ constexpr int pd16_db(int i) { return i & 7; }
__device__ __forceinline__ constexpr int pd16_kk(int i) { return (i - 16) >> 2; }
__device__ __forceinline__ constexpr int pd16_kb(int i) { return (i - 16) & 3; }

__device__ __forceinline__ bf16x8 pd16_operand(int i, uint32_t v_off, uint32_t k_off, const PfLane16& lc) {
  if (i < 16) {
    const uint32_t ad = lc.voff[pd16_db(i)] + v_off + pd16_kp(i) * 8192;
    const bf16x4 v0 = lds_read_tr8((lds_char*)(uintptr_t)ad);
    const bf16x4 v1 = lds_read_tr8((lds_char*)(uintptr_t)(ad + 4096));
    return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  return *(lds_bf16x8*)(uintptr_t)(lc.koff[pd16_kk(i)] + k_off + pd16_kb(i) * 4096);
}

__device__ __forceinline__ void pd16_preread(uint32_t v_off, const PfLane16& lc, bf16x8 (&pre)[kPfAhead]) {
#pragma unroll
  for (int i = 0; i < kPfAhead; ++i) pre[i] = pd16_operand(i, v_off, 0, lc);
}

// The matrix phase: O^T += V^T P^T of the previous tile, then S^T = K Q^T of the next - 64 MFMAs, their 32 LDS operands
// read kPfAhead operands ahead; the caller has read the first of them into pre (during its softmax phase).  The phase issues the
// global loads that ld names, and passes the workgroup barrier that ends it before its last MFMAs (as EARLY_BARRIER in
// pd_matrix_phase).  CINIT: the score accumulators start from cinit instead of zero.
template <bool CINIT, int NQ>
__device__ __forceinline__ void pd16_matrix_phase(uint32_t v_off, uint32_t k_off, const PfLane16& lc,
                                                  const bf16x8 (&qf)[4][NQ], const bf16x8 (&pb)[2][NQ], PfState16<NQ>& st,
                                                  f32x16 (&s)[NQ], const PfPhaseLoads& ld,
                                                  const bf16x8 (&pre)[kPfAhead], const f32x4 (&cinit)[NQ]) {
  bf16x8 op[kPfAhead + 1];
#pragma unroll
  for (int i = 0; i < kPfAhead; ++i) op[i] = pre[i];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    if (i + kPfAhead < 32) op[(i + kPfAhead) % (kPfAhead + 1)] = pd16_operand(i + kPfAhead, v_off, k_off, lc);
    bf16x8 x = op[i % (kPfAhead + 1)];
    if (i == 31) {
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(x) : : "memory");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    if (i < 16) {
      const int kp = pd16_kp(i), db = pd16_db(i);
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) {
        const int t4 = NQ * db + qb;
        q4_set(st.o[t4 >> 2], t4 & 3,
               __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, pb[kp][qb], q4_get(st.o[t4 >> 2], t4 & 3), 0, 0, 0));
      }
    } else {
      const int kk = pd16_kk(i), kb = pd16_kb(i);
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) {
        const int t4 = NQ * kb + qb;
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        const f32x4 c0 = kk == 0 ? (CINIT ? cinit[qb] : z) : q4_get(s[t4 >> 2], t4 & 3);
        q4_set(s[t4 >> 2], t4 & 3, __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, qf[kk][qb], c0, 0, 0, 0));
      }
    }
    if (i == 1) g2lds16_s<0>(ld.k, lc.gk[0], ld.ldk);
    if (i == 3) g2lds16_s<0>(ld.k, lc.gk[1], ld.ldk + 1024);
    if (i == 5) g2lds16_s<0>(ld.v, lc.gv[0], ld.ldv);
    if (i == 7) g2lds16_s<0>(ld.v, lc.gv[1], ld.ldv + 1024);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// combine the values of the four 16-lane groups that hold the key rows of one query: rows of 16 lanes, then halves, change
// places inside the register file (no LDS round trip)
__device__ __forceinline__ float max_groups16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max_halves(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float sum_groups16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return sum_halves(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Online softmax of one tile (general form: raw scores, running maximum moved when it must, masks).  rel[qb]: key
// rows of the tile with index > rel[qb] are hidden from the lane's query of block qb.
template <int NQ>
__device__ __forceinline__ void pf16_softmax(f32x16 (&s)[NQ], PfState16<NQ>& st, float c, bool masked, const int (&rel)[NQ],
                                             int g16, bf16x8 (&pb)[2][NQ]) {
  if (masked) {
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * kb + 4 * g16 + r > rel[qb]) PF16_S(s, kb, qb, r) = kNegBig;
  }
  float m_new[NQ];
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    float mx = PF16_S(s, 0, qb, 0);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, PF16_S(s, kb, qb, r));
    m_new[qb] = fmaxf(st.m[qb], max_groups16(mx));
  }
  if (__builtin_amdgcn_ballot_w64(m_new[0] > st.m[0] || m_new[NQ - 1] > st.m[NQ - 1]) != 0) {
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      const float alpha = fast_exp2((st.m[qb] - m_new[qb]) * c);
      st.l[qb] *= alpha;
#pragma unroll
      for (int db = 0; db < 8; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) PF16_O(st, db, qb, r) *= alpha;
      st.m[qb] = m_new[qb];
    }
  }
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    const float mc = st.m[qb] * c;
    float lsum = 0.f;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = fast_exp2(__builtin_fmaf(PF16_S(s, kb, qb, r), c, -mc));
        lsum += p;
        pb[kb >> 1][qb][4 * (kb & 1) + r] = (__bf16)p;
      }
    st.l[qb] += lsum;
  }
#pragma unroll
  for (int kp = 0; kp < 2; ++kp)
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) asm volatile("" : "+v"(pb[kp][qb]));
}

// Softmax phase of a steady-state tile: the scores left the matrix pipe relative to the running reference (the
// accumulators started from cinit = -m), p = 2^(c s); the reference only moves when a lane's share of a row sum says
// it must (see pf_softmax_fast).  The scores are scaled in place first, so that the 32 multiplications and the 32
// exponentials are independent instructions (with a shared temporary they formed one dependent chain).
// PRESCALED: the queries carry the softmax scale already (c is 1): the scores are exponents as they leave the matrix pipe.
template <bool PRESCALED, int NQ>
__device__ __forceinline__ void pf16_softmax_fast(f32x16 (&s)[NQ], PfState16<NQ>& st, float c, f32x4 (&cinit)[NQ],
                                                  bf16x8 (&pb)[2][NQ]) {
  if (!PRESCALED) {
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[j][r] *= c;
  }
  float ls[NQ];
  auto probs = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      float lq[2];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = fast_exp2(PF16_S(s, kb, qb, r));
          lq[kb & 1] = (kb < 2 && r == 0) ? p : lq[kb & 1] + p;
          pb[kb >> 1][qb][4 * (kb & 1) + r] = (__bf16)p;
        }
      ls[qb] = lq[0] + lq[1];
    }
  };
  probs();
  if (__builtin_amdgcn_ballot_w64(!(ls[0] <= kPfSumLimit) || !(ls[NQ - 1] <= kPfSumLimit)) != 0) {    // also inf and NaN
    const float inv_c = 1.0f / c;
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      float mx = PF16_S(s, 0, qb, 0);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, PF16_S(s, kb, qb, r));
      // queries whose maximum did not move keep their reference; the step is taken in score units (the reference
      // is kept in them) and applied here as the exponent it becomes
      const float d = fmaxf(max_groups16(mx), 0.f) * inv_c;
      const float dc = d * c;
      const float alpha = fast_exp2(-dc);
      st.l[qb] *= alpha;
#pragma unroll
      for (int db = 0; db < 8; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) PF16_O(st, db, qb, r) *= alpha;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) PF16_S(s, kb, qb, r) -= dc;
      st.m[qb] += d;
#pragma unroll
      for (int r = 0; r < 4; ++r) cinit[qb][r] = -st.m[qb];
    }
    probs();
  }
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) st.l[qb] += ls[qb];
#pragma unroll
  for (int kp = 0; kp < 2; ++kp)
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) asm volatile("" : "+v"(pb[kp][qb]));
}

// Normalise and write the lane's parts of the query row of block QB: dims 16 (db0 + d) + 4 g16 + 0..3 for d < NDB
// (o[d] holds dim block db0 + d); l is the lane's share of the row sum.
template <int NDB>
__device__ __forceinline__ void pf16_write_row(void* out, int out_fp32, int C, int g, int i, int g16, int db0,
                                               const f32x4 (&o)[NDB], float l) {
  const float inv = 1.0f / sum_groups16(l);
  if (i >= C) return;
  const int64_t base = ((int64_t)g * C + i) * kHeadDim;
#pragma unroll
  for (int d = 0; d < NDB; ++d) {
    const f32x4 v = o[d];
    const int dim = 16 * (db0 + d) + 4 * g16;
    const float x0 = v[0] * inv, x1 = v[1] * inv, x2 = v[2] * inv, x3 = v[3] * inv;
    if (out_fp32) {
      *(float4*)((float*)out + base + dim) = make_float4(x0, x1, x2, x3);
    } else {
      uint2 pk;
      pk.x = (uint32_t)float_to_bf16_bits(x0) | ((uint32_t)float_to_bf16_bits(x1) << 16);
      pk.y = (uint32_t)float_to_bf16_bits(x2) | ((uint32_t)float_to_bf16_bits(x3) << 16);
      *(uint2*)((uint16_t*)out + base + dim) = pk;
    }
  }
}

// The wavefront's two blocks of 16 query rows in block bx of positions: the first position, and how many of the two hold rows
// before the chunk's end.
struct Pf16Rows { int i0, nq; };
__device__ __forceinline__ Pf16Rows pf16_rows(const PrefillArgs& a, int bx, int gl, int wave) {
  Pf16Rows r;
  r.i0 = 32 * (bx * (kPdWaves / gl) + wave / gl);
  r.nq = a.C - r.i0 > 16 ? 2 : a.C > r.i0 ? 1 : 0;
  return r;
}

// One pass of a workgroup of prefill_kernel_deep16: the tiles of `ps` on a softmax state of their own, by a wavefront that
// has NQ blocks of 16 query rows before the chunk's end (NQ = 0: it has none, and only takes its share of the tile loads and
// the barriers).  Rows that are not there cost matrix instructions, and with them clock: the kernel runs at the power limit.
// pos: the first position of the workgroup's block.
// Which tiles take their maxima first is pf_next_run's rule: the steady ones do not, and the largest weight of a row is then no
// longer exactly 1.  With the maxima of the first eight tiles only, short launches were 6 us faster and 1 to 3 % further off
// (600 rows behind 3001 1.53e-3 -> 1.55e-3, 300 behind 4000 1.46e-3 -> 1.50e-3, 200 behind 50 thousand 1.64e-3 -> 1.66e-3).
// What a pass costs, by time stamps of 600 rows of 8 heads behind 3000 (240 workgroups of 17 or 18 tiles): 6.5 us until the first
// tile is done (the fill of 144 KB per workgroup), 2.3 us for a tile that takes its maximum (two in three), 1.5 for a steady
// one, 2 to store the state.  Before, a tile of the first kind took 2.6 us, in which it chose its ring slot and its loads tile by
// tile and added every operand's address between the MFMAs, and integer divisions took 3 us at the start: 57 us a
// launch, now 53 (shortest of 33; medians 59 and 55).
template <bool PRESCALED, int NQ>
__device__ __forceinline__ void pd16_pass(const PrefillArgs& a, const PfPass& ps, uint32_t lds_base, int lane,
                                          int wave, int g, int pos, int i0, float* images) {
  constexpr int kLanes = kPdWaves * 64;
  constexpr int kImageFloats = kCarryFloatsPerLane * kLanes;
  constexpr int NS = NQ > 0 ? NQ : 1;                 // array sizes
  asm volatile("" : "+v"(lane));                      // lane constants are formed in the pass, not kept across passes
  const int g16 = lane >> 4;
  const int c16 = lane & 15;

  PfLane16 lc;
  {
    const int r_in = lane >> 4, cpos = lane & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (wave * 2 + i) * 4 + r_in;
      lc.gk[i] = (uint32_t)(r * kRowBytes + ((cpos ^ swz_k(r)) << 4));
      lc.gv[i] = (uint32_t)(r * kRowBytes + ((cpos ^ swz_v16(r)) << 4));
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      lc.koff[kk] = lds_base + (uint32_t)(c16 * kRowBytes + (((4 * kk + g16) ^ swz_k(c16)) << 4));
    const int row = 4 * g16 + (c16 >> 2);             // the row of the 4-row block this lane addresses
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const int chunk = 2 * db + ((c16 & 3) >> 1);
      lc.voff[db] = lds_base + kPdVRing +
                    (uint32_t)(row * kRowBytes + ((chunk ^ swz_v16(row)) << 4) + ((c16 & 1) << 3));
    }
  }

  PfSweep sw;
  const char *ka_p = a.ka, *va_p = a.va;
  {
    const int64_t start = pf_sweep_of(sw, ps, a.na, a.nb, a.a_jump_tile, a.a_jump_bytes);
    ka_p += start;
    va_p += start;
  }
  const int T = sw.T;

  auto issue = [&](int t, int which) __attribute__((always_inline)) {
    if (t >= T) return;
    const uint32_t slot = lds_base + (uint32_t)(t & (kPdStages - 1)) * kPfTileBytes;
    if (which == 0) pf16_issue_k((t >= sw.ta ? a.kb : ka_p) + pf_tile_offset(sw, t), pf_tile_rows(sw, t), slot, wave, lane, lc);
    else pf16_issue_v((t >= sw.ta ? a.vb : va_p) + pf_tile_offset(sw, t), pf_tile_rows(sw, t), slot + kPdVRing, wave, lane, lc);
  };
  auto wait_landed = [&](int t) __attribute__((always_inline)) {
    if (t + 3 < T) wait_vmcnt<4>();
    else wait_vmcnt<0>();
  };
  auto phase_barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  };

  // the alternating schedule, barrier protocol and ring discipline of prefill_kernel_deep
  const int group = wave >> 2;
  const float c = a.c;
  wait_vmcnt<0>();                   // the waits below count this pass's tile loads only (a previous pass's stores are done)
  issue(0, 0);                       // asked for before the queries: one latency for both
  issue(1, 0); issue(0, 1);
  issue(2, 0); issue(1, 1);

  if constexpr (NQ == 0) {
    wait_landed(-1);
    phase_barrier();
    if (group == 1) phase_barrier();
    for (int t = 0; t < T; ++t) {
      issue(t + 3, 0);
      issue(t + 2, 1);
      phase_barrier();
      wait_landed(t);
      phase_barrier();
    }
    if (group == 0) phase_barrier();
    if (ps.store >= 0 && !a.last) {          // a later launch may read the image in a kernel that works on all rows
      float* im = images + (int64_t)ps.store * kImageFloats;
#pragma unroll
      for (int i = 0; i < 64; ++i) im[i * kLanes] = 0.f;
      im[64 * kLanes] = im[65 * kLanes] = kNegBig;
      im[66 * kLanes] = im[67 * kLanes] = 0.f;
    }
    return;
  }

  // Q^T operands: lane holds q[g][qi[qb]][32*kk + 8*g16 .. +7]
  int my_i[NS];
  bf16x8 qf[4][NS];
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    my_i[qb] = i0 + 16 * qb + c16;
    const int qi = my_i[qb] > a.C - 1 ? a.C - 1 : my_i[qb];
    const uint16_t* qrow = a.q + ((int64_t)g * a.C + qi) * kHeadDim + 8 * g16;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qf[kk][qb] = __builtin_bit_cast(bf16x8, *(const uint4*)(qrow + 32 * kk));
  }

  PfState16<NS> st;
  if (ps.load < 0) {
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      st.m[qb] = kNegBig;
      st.l[qb] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < 2 * NQ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[j][r] = 0.f;
  } else {
    const float* im = images + (int64_t)ps.load * kImageFloats;
#pragma unroll
    for (int db = 0; db < 8; ++db)
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
        for (int r = 0; r < 4; ++r) PF16_O(st, db, qb, r) = im[((2 * db + qb) * 4 + r) * kLanes];
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      st.m[qb] = im[(64 + qb) * kLanes];
      st.l[qb] = im[(66 + qb) * kLanes];
    }
  }
  // the compiler's own waits for the loads above belong here
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(qf[kk][qb]));
    asm volatile("" : "+v"(st.m[qb]), "+v"(st.l[qb]));
  }
#pragma unroll
  for (int j = 0; j < 2 * NQ; ++j) asm volatile("" : "+v"(st.o[j]));

  wait_landed(-1);                   // K(0), K(1), V(0)
  phase_barrier();
  if (group == 1) phase_barrier();

  f32x16 sc[NS];
  bf16x8 pb[2][NS];
  // is tile t partly hidden from a row of this wavefront, and which of its rows each query sees (up to rel)
  auto hidden = [&](int t) __attribute__((always_inline)) {
    return pf_tile_rows(sw, t) < kPfTileRows || (t >= sw.ta && (t + sw.own0) * kPfTileRows + kPfTileRows - 1 > i0);
  };
  auto last_seen = [&](int t, int (&rel)[NS]) __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      int lim = pf_tile_rows(sw, t) - 1;
      if (t >= sw.ta) {
        const int d = my_i[qb] - (t + sw.own0) * kPfTileRows;
        lim = d < lim ? d : lim;
      }
      rel[qb] = lim;
    }
  };
  // a tile's softmax that takes its maximum first
  auto softmax_phase = [&](int t) __attribute__((always_inline)) {
    int rel[NS];
    const bool h = hidden(t);
    if (h) last_seen(t, rel);
    pf16_softmax<NS>(sc, st, c, h, rel, g16, pb);
  };
  // tile 0: nothing to accumulate yet
  issue(3, 0);
  issue(2, 1);
#pragma unroll
  for (int i = 16; i < 32; ++i) {
    const bf16x8 x = pd16_operand(i, 0, 0, lc);
    const int kk = pd16_kk(i), kb = pd16_kb(i);
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      const int t4 = NQ * kb + qb;
      q4_set(sc[t4 >> 2], t4 & 3,
             __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, qf[kk][qb], kk == 0 ? z : q4_get(sc[t4 >> 2], t4 & 3), 0, 0, 0));
    }
  }
  phase_barrier();
  softmax_phase(0);
  wait_landed(0);
  phase_barrier();
  bf16x8 pre[kPfAhead];
  f32x4 cinit[NS];     // minus the running references, the start values of the score accumulators behind the first tiles
  pd16_preread(0, lc, pre);
  // The tiles a tile's matrix phase asks for, K(t+3) and V(t+2), as two streams (see PfStream): every tile issues the same four
  // loads and waits for the same number, and all but a few per pass cost a pointer increment, in the softmax phase.
  PfStream sk, sv;
  auto clamp_rows = [&](uint32_t (&g)[2], int rows, bool is_v) __attribute__((always_inline)) {
    const int r_in = lane >> 4, cpos = lane & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (wave * 2 + i) * 4 + r_in;
      g[i] = (uint32_t)((r < rows ? r : rows - 1) * kRowBytes + ((cpos ^ (is_v ? swz_v16(r) : swz_k(r))) << 4));
    }
  };
  pf_stream_start(sk, sw, 4, ka_p, a.kb);
  pf_stream_start(sv, sw, 3, va_p, a.vb);
  clamp_rows(lc.gk, sk.rows, false);
  clamp_rows(lc.gv, sv.rows, true);
  const uint32_t ld_wave = lds_base + wave * 2048;
  // Tile t's matrix phase, which passes the barrier in its middle itself, with the two tiles at the streams' heads asked for
  // on the way.  CINIT: the scores start from minus the running references.
  auto matrix_phase = [&](uint32_t v_off, uint32_t k_off, uint32_t ldk, uint32_t ldv, auto cinit_tag) __attribute__((always_inline)) {
    PfPhaseLoads ld;
    ld.k = sk.p;
    ld.v = sv.p;
    ld.ldk = ld_wave + ldk;
    ld.ldv = ld_wave + kPdVRing + ldv;
    __builtin_amdgcn_s_setprio(2);
    pd16_matrix_phase<decltype(cinit_tag)::value, NS>(v_off, k_off, lc, qf, pb, st, sc, ld, pre, cinit);
    __builtin_amdgcn_s_setprio(0);
  };
  // the streams' heads have reached tiles t + 3 and t + 2: do they meet something there?
  auto meet = [&](int t) __attribute__((always_inline)) {
    if (sk.left == 0) {
      pf_stream_meet(sk, sw, t + 3, ka_p, a.kb);
      clamp_rows(lc.gk, sk.rows, false);
    }
    if (sv.left == 0) {
      pf_stream_meet(sv, sw, t + 2, va_p, a.vb);
      clamp_rows(lc.gv, sv.rows, true);
    }
  };
  int t = 1, piece = 0;
  uint32_t slot = 0;                             // ring offset of tile t - 1; the operand addresses move with it
#pragma nounroll
  for (;;) {
    const PfRun run = pf_next_run(sw, piece, t, pos);
#pragma nounroll
    for (; t < run.begin; ++t) {
      const uint32_t next = (slot + kPfTileBytes) & (kPdStages * kPfTileBytes - 1);
      const uint32_t d = next - slot, prev = (slot - kPfTileBytes) & (kPdStages * kPfTileBytes - 1);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) lc.koff[kk] += d;
      matrix_phase(0, 0, slot, prev, std::false_type());
#pragma unroll
      for (int db = 0; db < 8; ++db) lc.voff[db] += d;
      pd16_preread(0, lc, pre);                  // V(t)'s first operands, for the next matrix phase
      __builtin_amdgcn_sched_barrier(0);
      softmax_phase(t);
      __builtin_amdgcn_sched_barrier(0);
      sk.p += sk.step;
      sv.p += sv.step;
      --sk.left;
      --sv.left;
      meet(t + 1);
      wait_vmcnt<4>();                           // everything up to V(t+1) has landed
      phase_barrier();
      slot = next;
    }
    if (t >= T) break;
    // tile t in ring slot S = t % 4, a compile-time constant: every LDS address is an immediate
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      lc.koff[kk] -= 3 * kPfTileBytes;
      asm volatile("" : "+v"(lc.koff[kk]));      // (the compiler would carry the difference into every operand's address)
    }
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      lc.voff[db] -= 3 * kPfTileBytes;
      asm volatile("" : "+v"(lc.voff[db]));
    }
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
      for (int r = 0; r < 4; ++r) cinit[qb][r] = -st.m[qb];
    auto steady = [&](auto stage_tag) __attribute__((always_inline)) {
      constexpr uint32_t S = decltype(stage_tag)::value, kT = kPfTileBytes;
      matrix_phase(((S + 3) & 3) * kT, S * kT, ((S + 3) & 3) * kT, ((S + 2) & 3) * kT, std::true_type());
      pd16_preread(S * kT, lc, pre);
      __builtin_amdgcn_sched_barrier(0);
      pf16_softmax_fast<PRESCALED, NS>(sc, st, c, cinit, pb);
      wait_vmcnt<4>();
      phase_barrier();
      sk.p += kPfTileBytes;
      sv.p += kPfTileBytes;
    };
    sk.left -= run.end - run.begin;
    sv.left -= run.end - run.begin;
#pragma nounroll
    for (; t < run.end; t += 4) {
      steady(std::integral_constant<uint32_t, 0>());
      steady(std::integral_constant<uint32_t, 1>());
      steady(std::integral_constant<uint32_t, 2>());
      steady(std::integral_constant<uint32_t, 3>());
    }
    meet(t);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) lc.koff[kk] += 3 * kPfTileBytes;
#pragma unroll
    for (int db = 0; db < 8; ++db) lc.voff[db] += 3 * kPfTileBytes;
  }
  {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const bf16x8 x = pd16_operand(i, 0, 0, lc);
      const int kp2 = pd16_kp(i), db = pd16_db(i);
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) {
        const int t4 = NQ * db + qb;
        q4_set(st.o[t4 >> 2], t4 & 3,
               __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, pb[kp2][qb], q4_get(st.o[t4 >> 2], t4 & 3), 0, 0, 0));
      }
    }
  }
  wait_vmcnt<0>();                   // no load may reach the LDS of a workgroup that has ended
  if (group == 0) phase_barrier();

  if (ps.store >= 0) {
    float* im = images + (int64_t)ps.store * kImageFloats;
#pragma unroll
    for (int db = 0; db < 8; ++db)
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
        for (int r = 0; r < 4; ++r) im[((2 * db + qb) * 4 + r) * kLanes] = PF16_O(st, db, qb, r);
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      im[(64 + qb) * kLanes] = st.m[qb];
      im[(66 + qb) * kLanes] = st.l[qb];
    }
    if (NQ == 1 && !a.last) {                // the empty block's state, as above
#pragma unroll
      for (int db = 0; db < 8; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) im[((2 * db + 1) * 4 + r) * kLanes] = 0.f;
      im[65 * kLanes] = kNegBig;
      im[67 * kLanes] = 0.f;
    }
  } else {
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      f32x4 rows[8];
#pragma unroll
      for (int db = 0; db < 8; ++db) rows[db] = q4_get(st.o[(NQ * db + qb) >> 2], (NQ * db + qb) & 3);
      pf16_write_row<8>(a.out, a.out_fp32, a.C, g, my_i[qb], g16, 0, rows, st.l[qb]);
    }
  }
}

template <bool PRESCALED>
__global__ __launch_bounds__(512, 2) void prefill_kernel_deep16(PrefillArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char lds_dyn[];
  lds_char* lds = (lds_char*)lds_dyn;
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
  const int lane = lane_id();
  const int wave = wave_id();
  const int gl = a.G < 4 ? a.G : 4;
  const int g = pf_select_head(a) * 4 + (wave % gl);

  const int strip = 32 * (kPdWaves / gl);
  const PfShape sh = pf_shape_of(a, strip);
  constexpr int kLanes = kPdWaves * 64;
  constexpr int kImageFloats = kCarryFloatsPerLane * kLanes;
  float* const images = a.carry + (int64_t)blockIdx.y * a.img_row * kImageFloats + threadIdx.x;
  const int wg = pf_wg_index(blockIdx.x, gridDim.x, a.xcd);
  // the pass that holds past tiles goes first, so that the workgroups of a range walk the past rows in step
  PfPass ps = pf_pass(sh, wg, 0, a.last), other;
  other.run = other.init = 0;
  if (a.paired) {
    other = pf_pass(sh, wg, 1, a.last);
    if (other.run && other.a1 > other.a0 && !(ps.run && ps.a1 > ps.a0)) {
      const PfPass x = ps;
      ps = other;
      other = x;
    }
  }
#pragma nounroll
  for (int pi = 0; pi < 2; ++pi) {
    if (ps.init) {
      float* im = images + (int64_t)ps.store * kImageFloats;
#pragma unroll
      for (int i = 0; i < 64; ++i) im[i * kLanes] = 0.f;
      im[64 * kLanes] = kNegBig;
      im[65 * kLanes] = kNegBig;
      im[66 * kLanes] = 0.f;
      im[67 * kLanes] = 0.f;
    }
    if (ps.run) {
      __syncthreads();               // the LDS rings are free again (a previous pass may still be reading V tiles)
      const Pf16Rows rows = pf16_rows(a, ps.bx, gl, wave);
      if (rows.nq == 2) pd16_pass<PRESCALED, 2>(a, ps, lds_base, lane, wave, g, ps.bx * strip, rows.i0, images);
      else if (rows.nq == 1) pd16_pass<PRESCALED, 1>(a, ps, lds_base, lane, wave, g, ps.bx * strip, rows.i0, images);
      else pd16_pass<PRESCALED, 0>(a, ps, lds_base, lane, wave, g, ps.bx * strip, rows.i0, images);
    }
    ps = other;
    other.run = other.init = 0;
  }
}

// The chunk's rows on their way into an HBM-resident cache, 16 bytes per thread: in the blocks of a merge launch from z = first_z
// on, or in a launch of their own (kv_append_kernel).
struct PrefillAppendArgs {
  const char* k; const char* v;     // [heads][head_bytes]
  char* dk; char* dv;               // row 0 of the first head's new rows; the heads head_stride bytes apart
  int64_t head_bytes, head_stride;
  int heads, first_z;
};
__device__ __forceinline__ void pf_append(const PrefillAppendArgs& p, int64_t unit) {
  const int64_t per_head = p.head_bytes / 16, per_plane = per_head * p.heads;
  const bool is_v = unit >= per_plane;
  if (is_v) unit -= per_plane;
  if (unit >= per_plane) return;
  const int64_t head = per_plane >> 32 ? unit / per_head : (int64_t)((uint32_t)unit / (uint32_t)per_head);
  const int64_t at = (unit - head * per_head) * 16;
  *(uint4*)((is_v ? p.dv : p.dk) + head * p.head_stride + at) = *(const uint4*)((is_v ? p.v : p.k) + unit * 16);
}
// this block's share of the append, if it is one of the blocks that do nothing else
__device__ __forceinline__ bool pf_append_block(const PrefillAppendArgs& p) {
  if ((int)blockIdx.z < p.first_z) return false;
  const int64_t block = ((int64_t)(blockIdx.z - p.first_z) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
  pf_append(p, block * blockDim.x + threadIdx.x);
  return true;
}

// Merge of the states of prefill_kernel_deep16 (its own image layout): grid (blocks, grid rows, 8): z is one dim block
// of both query rows of the lane; where that is no workgroup for every compute unit, z = 16: one dim block of one query row (APART;
// a kernel of its own: with all four bodies in one, chosen at run time, it had 3604 instructions instead of 2498).
// Bound by the read of the images (139 KB each, up to 64 per block), and where a block has
// few of them by its latency: CH images are in flight per lane, and behind the first CH the references of all others.  The largest
// reference comes first, then the sums in the images' order, each image with one weight.  Shortest and median time with the
// append: 8 heads of 2 blocks of 16 images 7.4 and 8.4 us (128 workgroups, both rows in each: 9.7 and 10.7), of 10 blocks of 3 images 9.5 and
// 10.0 (1280 workgroups of one row each: 10.4 and 10.8); without the append, four images
// in flight in two loops, 10.0 and 11.6, 9.2 and 10.0.  (A single pass that rescales what it has summed takes 1 us less for the
// first, and gives other bits.)  Behind the merge's blocks others append the chunk's rows to the cache: as a launch of its own
// behind this one that took 4.3 us and the gap before it.
template <int NQ, int CH>
__device__ __forceinline__ void pf16_merge(const PrefillArgs& a, const PfShape& sh, const Pf16Rows& rows16, int bx, int db, int qb0,
                                           int n_e, int n, int g, int g16, int c16) {
  constexpr int kLanes = kPdWaves * 64;
  constexpr int kImageFloats = kCarryFloatsPerLane * kLanes;
  const float* images = a.carry + (int64_t)blockIdx.y * a.img_row * kImageFloats + threadIdx.x;
  auto image_of = [&](int i) __attribute__((always_inline)) {
    if (i >= n) i = n - 1;                            // (behind the last image: the last one again, which then takes no part)
    return images + (int64_t)(i < n_e ? pf_image_e(sh, bx, i) : pf_image_x(sh, bx, i - n_e)) * kImageFloats;
  };
  float m[NQ], l[NQ];
  f32x4 o[NQ];
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    m[qb] = kNegBig;
    l[qb] = 0.f;
    o[qb] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
#pragma nounroll
  for (int i0 = 0; i0 < n; i0 += CH) {
    float mi[CH][NQ], li[CH][NQ], oi[CH][NQ][4];
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const float* im = image_of(i0 + j);
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) {
        mi[j][qb] = im[(64 + qb0 + qb) * kLanes];
        li[j][qb] = im[(66 + qb0 + qb) * kLanes];
#pragma unroll
        for (int r = 0; r < 4; ++r) oi[j][qb][r] = im[((db * 2 + qb0 + qb) * 4 + r) * kLanes];
      }
    }
    if (i0 == 0) {
#pragma nounroll
      for (int k0 = CH; k0 < n; k0 += 6) {
        float x[6][NQ];
#pragma unroll
        for (int j = 0; j < 6; ++j) {
          const float* im = image_of(k0 + j);
#pragma unroll
          for (int qb = 0; qb < NQ; ++qb) x[j][qb] = im[(64 + qb0 + qb) * kLanes];
        }
#pragma unroll
        for (int j = 0; j < 6; ++j)
#pragma unroll
          for (int qb = 0; qb < NQ; ++qb) m[qb] = fmaxf(m[qb], x[j][qb]);
      }
#pragma unroll
      for (int j = 0; j < CH; ++j)
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) m[qb] = fmaxf(m[qb], mi[j][qb]);
    }
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const bool there = i0 + j < n;                  // (a weight of 0 would make NaN of an infinite value)
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) {
        const float w = fast_exp2((mi[j][qb] - m[qb]) * a.c);
        const float ls = l[qb] + w * li[j][qb];
        l[qb] = there ? ls : l[qb];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float os = o[qb][r] + w * oi[j][qb][r];
          o[qb][r] = there ? os : o[qb][r];
        }
      }
    }
  }
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    const f32x4 rows[1] = {o[qb]};
    pf16_write_row<1>(a.out, a.out_fp32, a.C, g, rows16.i0 + 16 * (qb0 + qb) + c16, g16, db, rows, l[qb]);
  }
}

template <bool APART>
__global__ __launch_bounds__(512, 4) void prefill_merge16_kernel(PrefillArgs a, PrefillAppendArgs append) {
  if (pf_append_block(append)) return;
  const int lane = lane_id();
  const int wave = wave_id();
  const int gl = a.G < 4 ? a.G : 4;
  const int bx = blockIdx.x;
  const int db = APART ? blockIdx.z & 7 : blockIdx.z, qb = APART ? blockIdx.z >> 3 : 0;
  const int g = pf_select_head(a) * 4 + (wave % gl);
  const Pf16Rows rows16 = pf16_rows(a, bx, gl, wave);
  if (qb >= rows16.nq) return;              // rows past the end
  const PfShape sh = pf_shape_of(a, 32 * (kPdWaves / gl));
  int n_e, n_x;
  pf_block_images(sh, bx, n_e, n_x);
  const int n = n_e + n_x;
  if (n == 1 && a.split == 1) return;
  if constexpr (APART) {
    if (n > 8) pf16_merge<1, 16>(a, sh, rows16, bx, db, qb, n_e, n, g, lane >> 4, lane & 15);
    else pf16_merge<1, 8>(a, sh, rows16, bx, db, qb, n_e, n, g, lane >> 4, lane & 15);
  } else {
    if (rows16.nq == 1) pf16_merge<1, 8>(a, sh, rows16, bx, db, 0, n_e, n, g, lane >> 4, lane & 15);
    else if (n <= 4) pf16_merge<2, 4>(a, sh, rows16, bx, db, 0, n_e, n, g, lane >> 4, lane & 15);
    else pf16_merge<2, 8>(a, sh, rows16, bx, db, 0, n_e, n, g, lane >> 4, lane & 15);
  }
}

#include "hi_prefill_wide.inc"

// One dim block (32 of the 128 output dims) of pf_write_row: register r of o is dim 32*db + 8*(r/4) + 4*hl + r%4.
__device__ __forceinline__ void pf_write_row_db(void* out, int out_fp32, int C, int g, int i, int hl, int db,
                                                const f32x16& o, float l) {
  const float inv = 1.0f / sum_halves(l);
  if (i >= C) return;
  const int64_t base = ((int64_t)g * C + i) * kHeadDim;
#pragma unroll
  for (int rq = 0; rq < 4; ++rq) {
    const int dim = 32 * db + 8 * rq + 4 * hl;
    const float x0 = o[4 * rq] * inv, x1 = o[4 * rq + 1] * inv, x2 = o[4 * rq + 2] * inv, x3 = o[4 * rq + 3] * inv;
    if (out_fp32) {
      *(float4*)((float*)out + base + dim) = make_float4(x0, x1, x2, x3);
    } else {
      uint2 pk;
      pk.x = (uint32_t)float_to_bf16_bits(x0) | ((uint32_t)float_to_bf16_bits(x1) << 16);
      pk.y = (uint32_t)float_to_bf16_bits(x2) | ((uint32_t)float_to_bf16_bits(x3) << 16);
      *(uint2*)((uint16_t*)out + base + dim) = pk;
    }
  }
}

// Merge of the states of the 8-wave kernel, run once after a unit's last launch when a block of positions can have
// more than one state (split > 1, or the paired partition): grid (blocks, grid rows, 4 dim blocks), the kernel's
// own lane layout, so every lane combines its own register images - m = max m_i, O = sum O_i 2^(c (m_i - m)),
// l likewise - then normalises and writes its part of out[g][i][:].  A block with a single state was written by
// the pass that computed it.
__global__ __launch_bounds__(512) void prefill_merge_kernel(PrefillArgs a, PrefillAppendArgs append) {
  if (pf_append_block(append)) return;
  const int lane = lane_id();
  const int wave = wave_id();
  const int hl = lane >> 5;
  const int col = lane & 31;
  const int gl = a.G < 4 ? a.G : 4;
  const int strip = 32 * (kPdWaves / gl);
  const int bx = blockIdx.x;
  const int db = blockIdx.z;
  const int g = pf_select_head(a) * 4 + (wave % gl);
  const int my_i = bx * strip + 32 * (wave / gl) + col;
  constexpr int kLanes = kPdWaves * 64;
  constexpr int kImageFloats = kCarryFloatsPerLane * kLanes;
  const PfShape sh = pf_shape_of(a, strip);
  int n_e, n_x;
  pf_block_images(sh, bx, n_e, n_x);
  if (n_e + n_x == 1 && a.split == 1) return;
  const float* images = a.carry + (int64_t)blockIdx.y * a.img_row * kImageFloats + threadIdx.x;
  auto image_of = [&](int i) { return images + (int64_t)(i < n_e ? pf_image_e(sh, bx, i) : pf_image_x(sh, bx, i - n_e)) * kImageFloats; };
  float m = kNegBig;
  for (int i = 0; i < n_e + n_x; ++i) m = fmaxf(m, image_of(i)[64 * kLanes]);
  f32x16 o;
#pragma unroll
  for (int r = 0; r < 16; ++r) o[r] = 0.f;
  float l = 0.f;
  for (int i = 0; i < n_e + n_x; ++i) {
    const float* im = image_of(i);
    const float w = fast_exp2((im[64 * kLanes] - m) * a.c);
    l += w * im[65 * kLanes];
#pragma unroll
    for (int r = 0; r < 16; ++r) o[r] += w * im[(db * 16 + r) * kLanes];
  }
  pf_write_row_db(a.out, a.out_fp32, a.C, g, my_i, hl, db, o, l);
}

// Merge of the ranges of the 4-wave kernel: grid (blocks, grid rows, 16), z = 4 (dim block) + quarter: four of its
// registers, dims 32 db + 8 rq + 4 hl ..; that kernel's own lane layout.  A lane whose query sees none of a range's keys (own
// rows only, all behind it) left its image's reference at kNegBig and its sums at zero; it takes no part.
// Bound by the latency of its reads (70 KB per image, up to 64 images of a block, and few blocks where there are many), so
// the grid splits an image finely and many images are in flight per lane: 63 images of 8 blocks take 18 us, 16 images
// of 16 blocks 6.4 (30 and 9.3 with whole dim blocks and four images in flight).
__global__ __launch_bounds__(256) void prefill_merge4_kernel(PrefillArgs a, PrefillAppendArgs append) {
  if (pf_append_block(append)) return;
  const int lane = lane_id();
  const int wave = wave_id();
  const int hl = lane >> 5;
  const int gl = a.G < 4 ? a.G : 4;
  const int strip = 32 * (4 / gl);
  const int blocks = gridDim.x, bx = blockIdx.x, db = blockIdx.z >> 2, rq = blockIdx.z & 3;
  const int g = pf_select_head(a) * 4 + (wave % gl);
  const int my_i = bx * strip + 32 * (wave / gl) + (lane & 31);
  constexpr int kImageFloats = kCarryFloatsPerLane * kWgThreads;
  const float* images = a.carry + ((int64_t)blockIdx.y * a.img_row + bx) * kImageFloats + threadIdx.x;
  const int64_t pitch = (int64_t)blocks * kImageFloats;
  float m = kNegBig;
#pragma unroll 16
  for (int k = 0; k < a.split; ++k) m = fmaxf(m, images[k * pitch + 64 * kWgThreads]);
  float o[4] = {0.f, 0.f, 0.f, 0.f}, l = 0.f;
#pragma unroll 8
  for (int k = 0; k < a.split; ++k) {
    const float* im = images + k * pitch;
    const float mk = im[64 * kWgThreads], lk = im[65 * kWgThreads];
    const float w = fast_exp2((mk - m) * a.c);
    const bool seen = mk > kNegBig;
    l += seen ? w * lk : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float x = im[(db * 16 + 4 * rq + r) * kWgThreads];
      o[r] += seen ? w * x : 0.f;
    }
  }
  const float inv = 1.0f / sum_halves(l);
  if (my_i >= a.C) return;
  const int64_t at = ((int64_t)g * a.C + my_i) * kHeadDim + 32 * db + 8 * rq + 4 * hl;
  const float x0 = o[0] * inv, x1 = o[1] * inv, x2 = o[2] * inv, x3 = o[3] * inv;
  if (a.out_fp32) {
    *(float4*)((float*)a.out + at) = make_float4(x0, x1, x2, x3);
  } else {
    uint2 pk;
    pk.x = (uint32_t)float_to_bf16_bits(x0) | ((uint32_t)float_to_bf16_bits(x1) << 16);
    pk.y = (uint32_t)float_to_bf16_bits(x2) | ((uint32_t)float_to_bf16_bits(x3) << 16);
    *(uint2*)((uint16_t*)a.out + at) = pk;
  }
}

// ---------------------------------------------------------------------------------------------------------
// Streaming heads (Appendix E, head-wise sparsity: a streaming head keeps only recent tokens - here n_sink initial
// tokens and the n_recent most recent ones - and lives in HBM).  Query row at absolute position p sees key j iff
// j <= p and (j < n_sink or p - j < n_recent).  The head's K/V is a bounded store of n_sink + n_recent rows: sink
// row j at row j, token j >= n_sink in ring slot n_sink + (j - n_sink) mod n_recent.
//
// One launch computes a chunk.  The keys form two sequences: A, what the store holds of the past (its ns sink
// rows, then the m most recent past rows in token order, read through the ring mapping), and B, the chunk's own
// rows.  A workgroup visits only the 64-row tiles some of its rows can see: the sink tiles and the tiles from its
// first row's window start on, in each sequence.
struct PrefillWindowArgs : PfWindow {
  const uint16_t* q;      // [G][C][128]
  const char* ks; const char* vs;   // the store's K and V planes
  const char* kb; const char* vb;   // the chunk's own rows
  void* out;
  int G, out_fp32, gy;
  float c;
  int64_t s_head_stride;  // bytes between the heads' stores
  // The chunk's rows on their way into the store (update = 0: in a launch of their own, 4.2 us behind this one of 61).  The last of the
  // workgroups that read what they replace writes all the head's rows; without such readers every workgroup writes its own.
  int update;
  PfStoreRows rows;
  int* counters;          // one per head, zero between launches (rows.readers > 0)
};

// A launch over 4 heads x 8192 rows (1024 workgroups, two rounds of two per compute unit, 11 tiles each) keeps one of a SIMD's two
// pipes at work nearly all the time: 56 % of the cycles the vector ALU, 41 % the matrix pipe.  The scores of a visit are formed
// under the softmax of the one before it (pf_tile4), two K and two V tiles have places in LDS, and the loads are streams that
// cost a pointer's increment: 53 thousand cycles a workgroup, of which 14 thousand to fetch queries and first tiles and to write the
// rows, instead of 59 - at a clock that falls for it (2.1 GHz over many launches); 155.6 -> 152.6 us for two chunks in a row, a
// pass with its hand-over to the caller's stream 165.4 -> 162.9.  Before: asking for the first tile before the queries and keeping
// neighbouring blocks on one XCD took a launch from 72 to 66 us; a ring of four stages with one workgroup of 8 wavefronts, or of
// three K and two V tiles with two of 4, was no faster (87, 84 against 83 us), and starting the scores from minus the
// running reference spilled registers (89).
__global__ __launch_bounds__(256, 2) void prefill_window_kernel(PrefillWindowArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds_raw[kPfLdsBytes];
  lds_char* lds = (lds_char*)lds_raw;
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
  const int lane = lane_id();
  const int wave = wave_id();
  const int hl = lane >> 5;
  const int col = lane & 31;

  const int gl = a.G < 4 ? a.G : 4;
  const int strip = 32 * (4 / gl);
  // neighbouring blocks of positions read the same rows: let them share an XCD's L2 (pf_wg_index for any number of workgroups; over
  // all heads, so that the strips that read the store, a head's first ones, come early everywhere)
  const int n_wgs = gridDim.x * gridDim.y, id = blockIdx.y * gridDim.x + blockIdx.x, more = n_wgs & 7;
  const int wg = (id & 7) * (n_wgs >> 3) + ((id & 7) < more ? id & 7 : more) + (id >> 3);
  const int by = wg / (int)gridDim.x, bx = wg - by * (int)gridDim.x;
  const int head = by / a.gy;
  {  // group launches: this workgroup's head
    const int64_t rows = (int64_t)head * a.C;
    a.q += rows * a.G * kHeadDim;
    a.out = (char*)a.out + rows * a.G * kHeadDim * (a.out_fp32 ? 4 : 2);
    a.ks += head * a.s_head_stride;
    a.vs += head * a.s_head_stride;
    a.kb += rows * kRowBytes;
    a.vb += rows * kRowBytes;
  }
  const int g = (by - head * a.gy) * 4 + (wave % gl);
  const int i_lo = bx * strip;                      // first and last query position of the workgroup
  const int i_hi = i_lo + strip - 1;
  const int i0 = i_lo + 32 * (wave / gl);           // first query position of this wave
  const int my_i = i0 + col;
  const int qi = my_i > a.C - 1 ? a.C - 1 : my_i;

  const PfLaneConst lc = pf_lane_const_4w(lane);

  PfState st;
  st.m = kNegBig;
  st.l = 0.f;
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) st.o[db][r] = 0.f;

  const PfWindowTiles t = pf_window_tiles(a, i_lo, i_hi);

  PfStream4 sk, sv;
  sk.v = sv.v = sk.usual = sv.usual = 0;
  auto meet = [&](PfStream4& w, auto v_tag) __attribute__((always_inline)) {
    constexpr bool V = decltype(v_tag)::value;
    int rows, row0;
    if (!pf_window_meet(w, a, t, V ? a.vs : a.ks, V ? a.vb : a.kb, rows, row0)) return;
    const int nA = a.ns + a.m;
    pf_stream4_offsets<V>(w, wave, formed_here(lane), [&](int r) __attribute__((always_inline)) {
      return rows ? (r < rows ? r : rows - 1) : pf_window_row(a, row0 + r < nA ? row0 + r : nA - 1);
    });
  };
  using KPlane = std::false_type;
  using VPlane = std::true_type;
  auto go_on_k = [&]() __attribute__((always_inline)) { if (pf_loads_next(sk, t.T)) meet(sk, KPlane()); };
  auto go_on_v = [&]() __attribute__((always_inline)) { if (pf_loads_next(sv, t.T)) meet(sv, VPlane()); };
  const uint32_t lds_wave = lds_base + wave * 4096;
  meet(sk, KPlane());
  meet(sv, VPlane());
  pf_stream4_issue(sk, lds_wave);                // before the queries: one wait for all
  pf_stream4_issue(sv, lds_wave + kPfStageBytes);
  go_on_k();
  go_on_v();
  pf_stream4_issue(sk, lds_wave + kPfTileBytes);
  bf16x8 qf[8];
  {
    const uint16_t* qrow = a.q + ((int64_t)g * a.C + qi) * kHeadDim + 8 * hl;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, *(const uint4*)(qrow + 16 * kk));
  }
  go_on_k();
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) asm volatile("" : "+v"(qf[kk]));
  const PfSeenVisits open = pf_window_open(a, t, i0);
  bool in_b = false;
  int j0 = 0;
  pf_sweep4<false>(lds, lds_wave, lc, qf, st, a.c, t.T, lane, sk, sv, go_on_k, go_on_v,
            [&](int v) __attribute__((always_inline)) {
              if ((uint32_t)(v - open.first) < (uint32_t)open.n) return false;
              j0 = pf_window_locate(t, v, in_b) * kPfTileRows;
              return !pf_window_full(a, in_b, j0, i0);
            },
            [&](int) __attribute__((always_inline)) { return pf_window_seen(a, in_b, j0, i0 + (formed_here(lane) & 31)); });

  pf_write_row(a.out, a.out_fp32, a.C, g, my_i, hl, st.o, st.l);
  if (!a.update) return;
  if (a.rows.readers == 0) {                             // nobody reads what the rows replace
    if (by != head * a.gy) return;
    for (int j = threadIdx.x; j < strip * 16; j += 256) {
      const int u = i_lo + (j >> 4);
      if (!(u < a.rows.cs || (u >= a.rows.u0 && u < a.rows.u0 + a.rows.cr))) continue;
      const int64_t src = (int64_t)u * kRowBytes + (j & 15) * 16, at = (int64_t)pf_store_row(a.rows, a.n_sink, a.n_recent, u) * kRowBytes + (j & 15) * 16;
      const uint4 k = *(const uint4*)(a.kb + src), v = *(const uint4*)(a.vb + src);
      *(uint4*)((char*)a.ks + at) = k;
      *(uint4*)((char*)a.vs + at) = v;
    }
    return;
  }
  if (bx >= a.rows.readers) return;
  // every wavefront's last loads have landed (it waited for them in its last step); the counter orders nothing else
  int* const flag = (int*)lds_raw;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int before = __hip_atomic_fetch_add(a.counters + head, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = before == a.rows.readers * a.gy - 1;
    if (last) __hip_atomic_store(a.counters + head, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = last;
  }
  __syncthreads();
  if (*flag == 0) return;
  const int parts = (a.rows.cs + a.rows.cr) * 16;
#pragma unroll 4
  for (int j = threadIdx.x; j < parts; j += 256) {
    const int u = (j >> 4) < a.rows.cs ? j >> 4 : a.rows.u0 + (j >> 4) - a.rows.cs;
    const int64_t src = (int64_t)u * kRowBytes + (j & 15) * 16, at = (int64_t)pf_store_row(a.rows, a.n_sink, a.n_recent, u) * kRowBytes + (j & 15) * 16;
    const uint4 k = *(const uint4*)(a.kb + src), v = *(const uint4*)(a.vb + src);
    *(uint4*)((char*)a.ks + at) = k;
    *(uint4*)((char*)a.vs + at) = v;
  }
}

// The chunk's rows enter a streaming head's store (after the chunk's attention has read it): chunk rows that are
// sink tokens go to their sink rows, the last n_recent rows (that are not sinks) to their ring slots.
// grid (row blocks, heads, 2: K and V); 16 bytes per thread.
__global__ __launch_bounds__(256) void stream_store_update_kernel(const char* __restrict__ k_new,
                                                                  const char* __restrict__ v_new,
                                                                  char* __restrict__ ks, char* __restrict__ vs, int C,
                                                                  int64_t P, int n_sink, int n_recent, int cs, int u0r,
                                                                  int cr, int64_t s_head_stride) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int r = (int)(idx >> 4), part = (int)(idx & 15);
  if (r >= cs + cr) return;
  const int u = r < cs ? r : u0r + (r - cs);                       // chunk row
  const int64_t j = P + u;                                         // its token
  const int64_t dst = r < cs ? j : n_sink + (j - n_sink) % n_recent;
  const char* src = (blockIdx.z ? v_new : k_new) + ((int64_t)blockIdx.y * C + u) * kRowBytes + part * 16;
  char* d = (blockIdx.z ? vs : ks) + blockIdx.y * s_head_stride + dst * kRowBytes + part * 16;
  *(uint4*)d = *(const uint4*)src;
}


// A chunk's K and V rows of a group of HBM-resident heads enter the cache, where no merge launch takes them along.
// Bound by one load and one store latency: 16 bytes per thread (four guarded loads per thread ran one after the other, 12 us
// for 600 rows of 8 heads against 4).
__global__ __launch_bounds__(256) void kv_append_kernel(PrefillAppendArgs p) {
  pf_append(p, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

static hi_status append_args(const PrefillAppend& ap, PrefillAppendArgs& p, int64_t& units) {
  p = {(const char*)ap.k_new, (const char*)ap.v_new, (char*)ap.k_dst, (char*)ap.v_dst, ap.rows * kRowBytes, ap.head_stride, ap.heads, 0};
  units = 2 * ap.heads * (p.head_bytes / 16);
  if (ap.rows < 1 || ap.heads < 1 || ceil_div(units, 256) > 0x7FFFFFFF) { set_last_error("append launch: bad shape"); return HI_ERR_ARG; }
  return HI_OK;
}

hi_status launch_kv_append(void* stream, const PrefillAppend& ap, void* done) {
  PrefillAppendArgs p;
  int64_t units;
  const hi_status st = append_args(ap, p, units);
  if (st != HI_OK) return st;
  launch_kernel(kv_append_kernel, dim3((unsigned)ceil_div(units, 256)), dim3(256), 0, stream, done, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error("append launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

hi_status launch_prefill(void* stream, const void* q, int G, int chunk_len, const PrefillSegment& sa,
                         const PrefillSegment& sb, int first, int last, void* carry, void* out, int out_fp32,
                         int variant, const PrefillLaunch& unit, int n_heads, int64_t carry_bytes, const PrefillAppend* append, void* done) {
  if (n_heads < 1 || (variant & 3) == 2) { set_last_error("prefill launch: head group or variant"); return HI_ERR_UNSUPPORTED; }
  if (chunk_len < 1 || !(G == 1 || G == 2 || G == 4 || G == 8)) { set_last_error("prefill launch: bad shape"); return HI_ERR_ARG; }
  if (sa.causal || (sb.n > 0 && !sb.causal)) { set_last_error("prefill launch: segment order"); return HI_ERR_ARG; }
  if (sa.n + sb.n <= 0) { set_last_error("prefill launch: no rows"); return HI_ERR_ARG; }
  PrefillArgs a;
  a.q = (const uint16_t*)q;
  a.ka = (const char*)sa.k; a.va = (const char*)sa.v; a.na = sa.n;
  a.kb = (const char*)sb.k; a.vb = (const char*)sb.v; a.nb = sb.n;
  a.carry = (float*)carry;
  a.out = out;
  a.G = G; a.C = chunk_len; a.first = first; a.last = last; a.out_fp32 = out_fp32;
  const bool q_prescaled = (variant & 32) != 0;
  a.c = softmax_scale_log2(q_prescaled);
  const int strip = prefill_strip(G);
  const int gy = prefill_grid_y(G);
  a.gy = gy;
  a.a_jump_tile = (int)(sa.jump_rows / kPfTileRows);
  a.a_jump_bytes = sa.jump_bytes;
  if (sa.jump_rows != 0 && (sa.jump_rows % kPfTileRows != 0 || sa.jump_rows < 0 || sa.jump_rows >= sa.n)) {
    set_last_error("prefill launch: a past segment in two pieces breaks at a multiple of 64 rows inside it");
    return HI_ERR_ARG;
  }
  a.a_head_stride = sa.head_stride;
  const PrefillLaunch pl = prefill_launch_of(unit, last, sb.n > 0);
  if (sa.n >= (1LL << 31) || sb.n >= (1LL << 31)) { set_last_error("prefill launch: more than 2^31 rows"); return HI_ERR_RANGE; }
  if (pl.carry_bytes > carry_bytes) {     // the carry must hold every state image of the launch
    set_last_error("prefill launch: carry of %lld bytes needed, %lld provided", (long long)pl.carry_bytes, (long long)carry_bytes);
    return HI_ERR_ARG;
  }
  // the rows to append ride on the merge launch, as blocks behind its z_merge x (threads) ones
  if (append && !pl.merge) { set_last_error("prefill launch: rows to append, but no merge to take them along"); return HI_ERR_ARG; }
  PrefillAppendArgs app = {};
  int64_t app_units = 0;
  if (append) {
    const hi_status st = append_args(*append, app, app_units);
    if (st != HI_OK) return st;
  }
  auto merge_grid = [&](unsigned x, unsigned y, unsigned z_merge, int threads) {
    app.first_z = (int)z_merge;
    return dim3(x, y, z_merge + (unsigned)ceil_div(app_units, (int64_t)x * y * threads));
  };
  void* const kernel_done = pl.merge ? nullptr : done;      // the attention kernel's, if no merge follows it
  a.split = pl.split;
  a.paired = pl.paired;
  a.nbk = pl.nbk;
  a.img_row = pl.img_row;
  a.xcd = pl.xcd;
  a.by_split = a.by_nbk = 0;
  if (pl.deep) {
    const PfShape sh = pf_shape_of(a, 2 * strip);
    a.by_split = pf_magic((uint32_t)pl.split, pf_largest_cut(sh));
    a.by_nbk = pf_magic((uint32_t)pl.nbk, (uint64_t)pl.nbk * (uint64_t)pl.split);
  }
  a.tile0 = (int)sa.tile0;
  a.past_tiles = pl.past_tiles;
  if (!pl.deep && pl.split > 1 && (sa.tile0 < 0 || sa.tile0 + ceil_div(sa.n, kPfTileRows) > pl.past_tiles ||
                                   (last && (sa.tile0 + ceil_div(sa.n, kPfTileRows) != pl.past_tiles || sb.n < 1)) ||
                                   (int64_t)pl.img_row != (int64_t)pl.split * ceil_div(chunk_len, strip))) {
    set_last_error("prefill launch: the segment does not fit the unit's tiles");
    return HI_ERR_ARG;
  }
  if (sa.jump_rows != 0 && !(pl.deep ? (variant & 16) == 0 : pl.split > 1)) {
    set_last_error("prefill launch: this kernel takes its past segment in one piece");
    return HI_ERR_UNSUPPORTED;
  }
  if (pl.deep) {
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [] {
      attr_err = hipFuncSetAttribute((const void*)prefill_kernel_deep, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     kPdLdsBytes);
      if (attr_err == hipSuccess)
        attr_err = hipFuncSetAttribute((const void*)prefill_kernel_deep16<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       kPdLdsBytes);
      if (attr_err == hipSuccess)
        attr_err = hipFuncSetAttribute((const void*)prefill_kernel_deep16<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       kPdLdsBytes);
      if (attr_err == hipSuccess)
        attr_err = hipFuncSetAttribute((const void*)prefill_kernel_wide<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       kPdLdsBytes);
      if (attr_err == hipSuccess)
        attr_err = hipFuncSetAttribute((const void*)prefill_kernel_wide<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       kPdLdsBytes);
    });
    if (attr_err != hipSuccess) { set_last_error("hipFuncSetAttribute: %s", hipGetErrorString(attr_err)); return HI_ERR_HIP; }
    dim3 grid((unsigned)(pl.nbk * pl.split), (unsigned)(gy * n_heads));
    const bool mfma32 = (variant & 16) != 0;        // the 32x32x16 form of the kernel (its state images differ)
    // the 4-wave, 64-rows-per-wavefront form of the 16x16x32 kernel: for workgroups that sweep enough tiles to pay for its
    // slow straight-line ones (it gains about 3 % per steady-state tile and loses about 20 tiles' worth at the ends)
    const bool wide = prefill_is_wide(variant, pl.split, sa.n + sb.n);
    auto attend = [&](auto kernel, int waves) { launch_kernel(kernel, grid, dim3(waves * 64), kPdLdsBytes, stream, kernel_done, a); };
    if (mfma32) attend(prefill_kernel_deep, kPdWaves);
    else if (wide && q_prescaled) attend(prefill_kernel_wide<true>, kPwWaves);
    else if (wide) attend(prefill_kernel_wide<false>, kPwWaves);
    else if (q_prescaled) attend(prefill_kernel_deep16<true>, kPdWaves);
    else attend(prefill_kernel_deep16<false>, kPdWaves);
    if (pl.merge) {
      hipError_t e1 = hipGetLastError();
      if (e1 != hipSuccess) { set_last_error("prefill launch: %s", hipGetErrorString(e1)); return HI_ERR_HIP; }
      if (mfma32) launch_kernel(prefill_merge_kernel, merge_grid((unsigned)pl.nbk, grid.y, 4, kPdWaves * 64), dim3(kPdWaves * 64), 0, stream, done, a, app);
      else if (8u * pl.nbk * grid.y < kPrefillCus) launch_kernel(prefill_merge16_kernel<true>, merge_grid((unsigned)pl.nbk, grid.y, 16, kPdWaves * 64), dim3(kPdWaves * 64), 0, stream, done, a, app);
      else launch_kernel(prefill_merge16_kernel<false>, merge_grid((unsigned)pl.nbk, grid.y, 8, kPdWaves * 64), dim3(kPdWaves * 64), 0, stream, done, a, app);
    }
  } else {
    const dim3 blocks((unsigned)ceil_div(chunk_len, strip), (unsigned)(gy * n_heads));
    if (pl.split > 1) {
      const dim3 cut(blocks.x * (unsigned)pl.split, blocks.y);
      // more than one wavefront on a SIMD: straight (see prefill_kernel, with both sides' times)
      if ((int64_t)cut.x * cut.y > kPrefillCus) launch_kernel(prefill_kernel<true, true>, cut, dim3(kWgThreads), 0, stream, kernel_done, a);
      else launch_kernel(prefill_kernel<true, false>, cut, dim3(kWgThreads), 0, stream, kernel_done, a);
      if (pl.merge) {
        hipError_t e1 = hipGetLastError();
        if (e1 != hipSuccess) { set_last_error("prefill launch: %s", hipGetErrorString(e1)); return HI_ERR_HIP; }
        launch_kernel(prefill_merge4_kernel, merge_grid(blocks.x, blocks.y, 16, kWgThreads), dim3(kWgThreads), 0, stream, done, a, app);
      }
    } else {
      launch_kernel(prefill_kernel<false, false>, blocks, dim3(kWgThreads), 0, stream, kernel_done, a);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error("prefill launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

hi_status launch_prefill_window(void* stream, const void* q, int G, int chunk_len, const void* store_k,
                                const void* store_v, int64_t store_head_stride, const void* k_new, const void* v_new,
                                int64_t past_len, int n_sink, int n_recent, void* out, int out_fp32, int n_heads,
                                bool q_prescaled, const PrefillWindowUpdate* update, void* done) {
  if (n_heads < 1 || chunk_len < 1 || !(G == 1 || G == 2 || G == 4 || G == 8) || past_len < 0 || n_sink < 0 ||
      n_recent < 1 || (int64_t)n_sink + n_recent > kStreamMaxRows) {
    set_last_error("windowed prefill launch: bad shape");
    return HI_ERR_ARG;
  }
  PrefillWindowArgs a;
  (PfWindow&)a = pf_window_of(past_len, chunk_len, n_sink, n_recent);
  a.q = (const uint16_t*)q;
  a.ks = (const char*)store_k; a.vs = (const char*)store_v;
  a.kb = (const char*)k_new; a.vb = (const char*)v_new;
  a.out = out;
  a.G = G; a.out_fp32 = out_fp32;
  a.gy = prefill_grid_y(G);
  a.c = softmax_scale_log2(q_prescaled);
  a.s_head_stride = store_head_stride;
  a.update = update != nullptr;
  if (update) {
    a.rows = update->rows;
    a.counters = update->counters;
    if (a.rows.readers > 0 && !a.counters) { set_last_error("windowed prefill launch: no counters"); return HI_ERR_ARG; }
  }
  dim3 grid((unsigned)ceil_div(chunk_len, prefill_strip(G)), (unsigned)(a.gy * n_heads));
  launch_kernel(prefill_window_kernel, grid, dim3(kWgThreads), 0, stream, done, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error("windowed prefill launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

hi_status launch_stream_store_update(void* stream, const void* k_new, const void* v_new, int chunk_len,
                                     int64_t past_len, int n_sink, int n_recent, void* store_k, void* store_v,
                                     int64_t store_head_stride, int n_heads, void* done) {
  if (n_heads < 1 || chunk_len < 1 || past_len < 0 || n_sink < 0 || n_recent < 1) {
    set_last_error("store update launch: bad shape");
    return HI_ERR_ARG;
  }
  const int cs = (int)(n_sink > past_len ? (n_sink - past_len < chunk_len ? n_sink - past_len : chunk_len) : 0);
  int u0r = chunk_len - n_recent;
  if (u0r < cs) u0r = cs;
  const int cr = chunk_len - u0r;
  if (cs + cr == 0) return HI_OK;
  dim3 grid((unsigned)ceil_div((int64_t)(cs + cr) * 16, 256), (unsigned)n_heads, 2);
  launch_kernel(stream_store_update_kernel, grid, dim3(256), 0, stream, done, (const char*)k_new, (const char*)v_new,
                (char*)store_k, (char*)store_v, chunk_len, past_len, n_sink, n_recent, cs, u0r, cr, store_head_stride);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error("store update launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

}  // namespace hi
