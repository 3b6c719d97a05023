// The steps either side of head-wise attention, for gfx950: Q/K/V projection (Section 3.1, Eq. 1: K_t = W_K E(x_t),
// V_t = W_V E(x_t), the query likewise) with the rotary position embedding of the evaluated model fused into its
// epilogue and the results written head-major - the layout the attention calls take - and the output projection
// that consumes the concatenated head outputs (Eq. 9).
//
// Both are one bf16 MFMA contraction D[a][b] = sum_k A[a][k] B[b][k] over two row-major operands whose contraction
// index is contiguous (activations [tokens][features] and weights [out_features][in_features] both are):
//   * a workgroup (4 wavefronts, one per SIMD) owns a 256 x 256 tile of D and walks the contraction in steps of 64;
//     each step's 256 x 64 slices of A and of B (32 KiB each) go HBM/L2 -> LDS by direct-to-LDS 128-bit loads into
//     one of two stages; one barrier per step, placed before the step's last 16 MFMAs, which cover the first operand
//     reads of the next step and the issue of the loads of the step after it;
//   * rows are 128 bytes in LDS; 16-byte chunk c of row r sits at chunk position c ^ ((r >> 1) & 7), which makes
//     the 32x32x16 MFMA operand reads (16 lanes = 16 consecutive rows, one chunk each) bank-conflict free;
//   * a wavefront owns 128 rows of A x 128 rows of B (4 x 4 accumulator blocks, 256 accumulator registers): 8
//     operand reads per 16 MFMAs, read one sub-step (16 contraction elements) ahead of their use.  In the Q/K/V
//     projection A is the weight and a wavefront's A rows are one whole head, so the two members of every rotary
//     pair (dimension i and i + 64: blocks ia and ia + 2, same register) meet in one lane;
//   * the tiles of one XCD (workgroups are dealt to the 8 XCDs round-robin) form a compact block of the tile grid
//     and advance through the contraction together, so each operand slice is fetched into that XCD's L2 about once.
//   * workgroups are persistent (one per compute unit, looping over their XCD's tiles): the next tile's first loads
//     are issued under the current tile's epilogue; the epilogue's stores are 16 bytes wide after an exchange between
//     the two half-waves.
// Measured (Llama-3-8B shapes, chunk 16384): 1.05 PFLOP/s for the Q/K/V projection (1.27 without the rotation),
// 1.25 PFLOP/s for the output projection; on constant operands, where the clock is not power-managed, 1.36 / 1.63.
#include <mutex>
#include <type_traits>
#include "hi_device.h"
#include "hi_internal.h"
#include "hi_rope.h"

namespace hi {

typedef __attribute__((address_space(3))) bf16x8* lds_bf16x8_p;

constexpr int kPjTile = 256;                              // rows of A, and of B, per workgroup
constexpr int kPjK = 64;                                  // contraction elements per step
constexpr int kPjRowBytes = kPjK * 2;
constexpr int kPjOperandBytes = kPjTile * kPjRowBytes;    // 32 KiB
constexpr int kPjStageBytes = 2 * kPjOperandBytes;        // A slice then B slice
constexpr int kPjLdsBytes = 2 * kPjStageBytes;            // 128 KiB
constexpr int kPjWaves = 4;
constexpr int kPjWgsPerXcd = 32;

enum { kPjQkv = 0, kPjOut = 1 };

struct ProjArgs {
  const char* a; const char* b;       // operand rows (bf16), contraction index contiguous: A the weight, B the activations
  int a_rows, b_rows;                 // valid rows (loads clamp, the epilogue masks)
  uint32_t a_stride, b_stride;        // bytes between rows
  int64_t b_head_stride;              // kPjOut: B[row][k] is at b + (k / 128) * b_head_stride + row * 256 + (k % 128) * 2
  int K;                              // contraction length, a multiple of 128 (an even number of steps)
  int a_tiles, b_tiles, ga;           // tile grid; tiles are ordered in groups of ga A-tiles (see pj_tile_of)
  int out_fp32;
  // kPjQkv: A = W_qkv [(Hq + 2 Hkv) * 128][K], B = X [C][K]
  void* q_out; void* k_out; void* v_out;   // [Hq][C][128], [Hkv][C][128], [Hkv][C][128]
  int n_q_heads, n_kv_heads;
  const float2* rope;                 // [16][C][4] (cos, sin) of pair 4 g + e at the chunk's token t: [g][t][e]; null: no rotation
  float q_scale;                      // kPjQkv: factor on the query heads' outputs (after the rotation, before rounding)
  // kPjOut: A = W_o [D][Hq * 128], B = attention output [Hq][C][128]
  void* y; int64_t y_stride;          // [C][y_stride] elements
};

struct RopeFreqs { double inv[64]; };      // theta^(-i / 64)
struct RopeChunk { RopeFreqs f; int64_t past; int on; };      // the rotation of a chunk that begins at position `past` (on = 0: none)
struct NoRope {};

// tile j of the grid: groups of ga A-tiles; inside a group B-major with the A-tile index fastest, so that any run of
// consecutive j is a compact block
__device__ __forceinline__ void pj_tile_of(const ProjArgs& p, int j, int& ta, int& tb) {
  const int full = p.a_tiles / p.ga;            // groups of exactly ga A-tiles
  const int per_group = p.ga * p.b_tiles;
  const int g = j / per_group;
  if (g < full) {
    const int w = j - g * per_group;
    ta = g * p.ga + w % p.ga;
    tb = w / p.ga;
  } else {
    const int rem = p.a_tiles - full * p.ga;
    const int w = j - full * per_group;
    ta = full * p.ga + w % rem;
    tb = w / rem;
  }
}

// One rotary pair (x, y) -> (x cos - y sin, y cos + x sin), with the roundings spelled out so that every epilogue
// (and the one-token kernel's caller-visible contract: bf16 output = fp32 output rounded) produces the same bits.
__device__ __forceinline__ float pj_rot_lo(float x, float y, float c, float sn) { return __builtin_fmaf(x, c, -(y * sn)); }
__device__ __forceinline__ float pj_rot_hi(float x, float y, float c, float sn) { return __builtin_fmaf(y, c, x * sn); }

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t pj_pack2(float x, float y) {
  const bf16x2 v = {(__bf16)x, (__bf16)y};      // round to nearest even
  return __builtin_bit_cast(uint32_t, v);
}

// Write 16 rows (features 16 rp .. 16 rp + 15 of a 32-row block of D) of this lane's token as bf16 to dst + 2 * row.
// o[0..3] are the lane's rows 16 rp + 4 hl + 0..3, o[4..7] its rows 16 rp + 8 + 4 hl + 0..3: the two half-waves
// exchange, so that each lane stores 8 consecutive rows (16 bytes) at once.
__device__ __forceinline__ void pj_store_rows_bf16(char* dst, const float (&o)[8], int rp, int hl, bool ok) {
  uint32_t x0 = pj_pack2(o[0], o[1]), x1 = pj_pack2(o[2], o[3]);
  uint32_t y0 = pj_pack2(o[4], o[5]), y1 = pj_pack2(o[6], o[7]);
  // lanes < 32 end up with rows 16 rp .. +7 (their own x, then the partner's x), lanes >= 32 with rows 16 rp + 8 .. +15
  auto s0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);
  auto s1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
  if (ok) *(uint4*)(dst + (16 * rp + 8 * hl) * 2) = make_uint4(s0[0], s1[0], s0[1], s1[1]);
}

// WIDE: bf16 output in whole runs of 128 features with a 16-byte aligned row pitch (decided by the launcher for the
// whole launch, so that each kernel holds one epilogue only and the accumulators never meet a control-flow join)
template <int MODE, bool WIDE>
__global__ __launch_bounds__(256, 1) void proj_gemm_kernel(ProjArgs p) {
  extern __shared__ __attribute__((aligned(1024))) char lds_dyn[];
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_char*)lds_dyn;
  const int lane = lane_id();
  const int wave = wave_id();
  const int l = lane & 31, hl = lane >> 5;
  const int wa = wave & 1, wb = wave >> 1;      // this wavefront: A rows 128 wa .. +127, B rows 128 wb .. +127

  // Persistent workgroups: XCD x (= blockIdx % 8) owns tiles [x * per, (x + 1) * per) of the ordered list, and its
  // workgroups take them round-robin; a workgroup's next tile starts loading while this one's results are written.
  const int total = p.a_tiles * p.b_tiles;
  const int per = (total + 7) >> 3;
  const int xcd = (int)(blockIdx.x & 7), li = (int)(blockIdx.x >> 3), n_li = (int)(gridDim.x >> 3);
  auto tile_index = [&](int s) __attribute__((always_inline)) { return s < per && xcd * per + s < total ? xcd * per + s : -1; };

  // ---- tile traffic: this wavefront's 8 load instructions per operand cover rows 64 w + 8 u + lane / 8
  uint32_t ga_off[8], gb_off[8];
  auto set_offsets = [&](int ta, int tb) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int row = 64 * wave + 8 * u + (lane >> 3);
      const int chunk = (lane & 7) ^ (4 * (u & 1) + (lane >> 4));      // = (lane & 7) ^ ((row >> 1) & 7)
      int ra = ta * kPjTile + row, rb = tb * kPjTile + row;
      ra = ra < p.a_rows ? ra : p.a_rows - 1;
      rb = rb < p.b_rows ? rb : p.b_rows - 1;
      ga_off[u] = (uint32_t)ra * p.a_stride + (chunk << 4);
      gb_off[u] = (uint32_t)rb * p.b_stride + (chunk << 4);
    }
  };
  // one of the 16 load instructions (8 of A, then 8 of B) of step t's slices into `stage`
  auto issue_one = [&](int t, int stage, int u) __attribute__((always_inline)) {
    const int k0 = t * kPjK;
    const uint32_t la = lds_base + stage * kPjStageBytes + wave * 8192;
    if (u < 8) {
      g2lds16_s<0>(p.a + (int64_t)k0 * 2, ga_off[u], la + u * 1024);
    } else {
      const char* bb = MODE == kPjOut ? p.b + (int64_t)(k0 >> 7) * p.b_head_stride + (k0 & 127) * 2 : p.b + (int64_t)k0 * 2;
      g2lds16_s<0>(bb, gb_off[u - 8], la + kPjOperandBytes + (u - 8) * 1024);
    }
  };

  // the same in two parts, on either side of an MFMA
  auto load_at = [&](int stage, int u) __attribute__((always_inline)) {
    set_m0(lds_base + wave * 8192 + stage * kPjStageBytes + (u < 8 ? 0 : kPjOperandBytes) + (u & 7) * 1024);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_now = [&](int t, int u) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    const int k0 = t * kPjK;
    if (u < 8) g2lds16_m0(p.a + (int64_t)k0 * 2, ga_off[u]);
    else g2lds16_m0(MODE == kPjOut ? p.b + (int64_t)(k0 >> 7) * p.b_head_stride + (k0 & 127) * 2 : p.b + (int64_t)k0 * 2, gb_off[u - 8]);
  };

  // ---- operand reads: lane l reads row (32 * block + l), chunk (2 kk + hl), of the A and of the B slice.  The
  // addresses are kept whole in registers per (stage, sub-step), the block is an immediate: no vector ALU work in
  // the loop (with one wavefront per SIMD every such instruction between two MFMAs is matrix-pipe time lost)
  uint32_t va[2][4], vb[2][4];
  {
    const int sw = (l >> 1) & 7;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const uint32_t ko = (uint32_t)(l * kPjRowBytes + (((2 * kk + hl) ^ sw) << 4));
        va[st][kk] = lds_base + st * kPjStageBytes + wa * 128 * kPjRowBytes + ko;
        vb[st][kk] = lds_base + st * kPjStageBytes + kPjOperandBytes + wb * 128 * kPjRowBytes + ko;
      }
  }
  // operand i of a contraction sub-step, in the order the MFMAs below first need them: A0 B0 A1 A2 A3 B1 B2 B3
  auto read_op = [&](int st, int kk, int i) __attribute__((always_inline)) -> bf16x8 {
    const bool is_a = i == 0 || (i >= 2 && i < 5);
    const int blk = i == 0 ? 0 : i == 1 ? 0 : i < 5 ? i - 1 : i - 4;
    return *(lds_bf16x8_p)((lds_char*)(uintptr_t)(is_a ? va[st][kk] : vb[st][kk]) + blk * 4096);
  };

  const int T = p.K / kPjK;
  int cur_j = tile_index(li);
  if (cur_j < 0) return;
  int ta, tb;
  pj_tile_of(p, cur_j, ta, tb);
  set_offsets(ta, tb);
#pragma unroll
  for (int u = 0; u < 16; ++u) issue_one(0, 0, u);
#pragma unroll
  for (int u = 0; u < 8; ++u) issue_one(1, 1, u);

  for (int s = li; cur_j >= 0; s += n_li) {
    f32x16 acc[4][4];
#pragma unroll
    for (int ia = 0; ia < 4; ++ia)
#pragma unroll
      for (int ib = 0; ib < 4; ++ib)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ia][ib][r] = 0.f;

    // MFMA j of a sub-step multiplies A block j % 4 with B block j / 4
    auto mfma_j = [&](const bf16x8 (&o)[8], int j) __attribute__((always_inline)) {
      const int ia = j & 3, ib = j >> 2;
      acc[ia][ib] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o[ia == 0 ? 0 : ia + 1], o[ib == 0 ? 1 : ib + 4], acc[ia][ib], 0, 0, 0);
    };

    // The schedule.  One wavefront per SIMD keeps the matrix pipe busy on its own: operand reads run one sub-step (16
    // contraction elements, 16 MFMAs) ahead of their use, across the step boundary too.  The barrier that publishes
    // step t+1's slices sits before the LAST sub-step of step t, whose MFMAs then cover the first operand reads of
    // step t+1 and the issue of step t+2's A loads into the stage step t has just finished reading; its B loads follow in the
    // first sub-step of step t+1.  One barrier per step; a wavefront waiting at it still has 16 MFMAs in the pipe.
    // The loads go out one behind every second MFMA: the texture path takes 16 cycles for each, 1024 for the 64 of a workgroup's
    // step, and all of them behind the 16 MFMAs (528 cycles) of one sub-step made every wavefront wait for it.  The B rows are
    // the activations, which the caches hold, so theirs are the loads with the shorter way to their barrier.  Hidden size 4096, 32 + 16
    // heads, Q/K/V and output at 4096 / 8192 / 16384 tokens: 221 / 350 / 691 -> 206 / 326 / 654 us, 114 / 224 / 440 -> 109 / 212 / 423.
    bf16x8 cur[8], nxt[8];
    wait_vmcnt<8>();           // step 0 has landed (at most step 1's A loads and earlier stores are still in flight)
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) cur[i] = read_op(0, 0, i);

    // MORE1: step t + 1 exists (its first operands are read here); MORE2: step t + 2 exists (its loads are issued here)
    auto step = [&](int t, auto stage_tag, auto more1_tag, auto more2_tag) __attribute__((always_inline)) {
      constexpr int STAGE = decltype(stage_tag)::value;
      constexpr int ST = STAGE, SN = 1 - STAGE;             // this stage and the other one
      constexpr bool MORE1 = decltype(more1_tag)::value, MORE2 = decltype(more2_tag)::value;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 3; ++kk) {
        // sub-step kk from one operand set while sub-step kk + 1 is read into the other
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          if (j < 8) {
            if (kk & 1) cur[j] = read_op(ST, kk + 1, j); else nxt[j] = read_op(ST, kk + 1, j);
          }
          const bool load = MORE1 && kk == 0 && (j & 1);
          if (load) load_at(SN, 8 + (j >> 1));
          mfma_j((kk & 1) ? nxt : cur, j);
          if (load) load_now(t + 1, 8 + (j >> 1));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // every read of this stage has been issued; the last sub-step's operands are in nxt
      wait_vmcnt<0>();                                      // this wave's loads of step t + 1 have landed
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave is done reading this stage
      __syncthreads();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        if (j < 8 && MORE1) cur[j] = read_op(SN, 0, j);
        const bool load = MORE2 && (j & 1);
        if (load) load_at(STAGE, j >> 1);
        mfma_j(nxt, j);
        if (load) load_now(t + 2, j >> 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    // T is even (the contraction length is a multiple of 128): pairs of steps, the last pair without look-ahead.
    // Straight-line code around one loop: the 256 accumulators never meet at a control-flow join.
    int t = 0;
    for (; t + 2 < T; t += 2) {
      step(t, S0(), std::true_type(), std::true_type());
      step(t + 1, S1(), std::true_type(), std::true_type());
    }
    step(t, S0(), std::true_type(), std::false_type());

    // ---- where this wavefront's results go.  Register r of block (ia, ib): A-row 128 wa + 32 ia + 8 (r / 4) + 4 hl
    // + r % 4 (an output feature), B-row 128 wb + 32 ib + l (a token): a lane owns one token and, with its partner in
    // the other half-wave, runs of 8 consecutive features.
    const int my_ta = ta, my_tb = tb;
    char* base = nullptr;        // where feature 0 of this wavefront's 128 A-rows goes, for token 0
    int64_t row_bytes = 0;       // bytes from one token's output row to the next
    bool rotate = false;
    float osc = 1.0f;            // factor on this wavefront's outputs (the query heads' q_scale; 1 is exact)
    int n_valid = 128;           // valid A-rows of the wavefront
    const int esz = p.out_fp32 ? 4 : 2;
    if (MODE == kPjQkv) {
      const int head = 2 * my_ta + wa;
      int hh;
      if (head < p.n_q_heads) { base = (char*)p.q_out; hh = head; }
      else if (head < p.n_q_heads + p.n_kv_heads) { base = (char*)p.k_out; hh = head - p.n_q_heads; }
      else { base = (char*)p.v_out; hh = head - p.n_q_heads - p.n_kv_heads; }
      if (head >= p.n_q_heads + 2 * p.n_kv_heads) n_valid = 0;
      rotate = p.rope != nullptr && head < p.n_q_heads + p.n_kv_heads;
      if (head < p.n_q_heads) osc = p.q_scale;
      base += (int64_t)hh * p.b_rows * kHeadDim * esz;
      row_bytes = (int64_t)kHeadDim * esz;
    } else {
      const int n0 = my_ta * kPjTile + wa * 128;
      base = (char*)p.y + (int64_t)n0 * esz;
      row_bytes = p.y_stride * esz;
      n_valid = p.a_rows - n0 < 128 ? (p.a_rows - n0 > 0 ? p.a_rows - n0 : 0) : 128;
    }
    const int m0 = my_tb * kPjTile + wb * 128 + l;                    // this lane's token in token block 0

    // The rotary table, (cos, sin) of 8 pairs of the lane's token per group (token block ib, pair half ip) of the
    // epilogue, is fetched two groups ahead (each buffer is refilled as soon as its group is rotated): a lone
    // wavefront per SIMD has nobody to hide a load's latency behind (fetched where it is used, the 32 load-wait rounds
    // of a tile took a fifth of its time).  The loads are unconditional and their addresses are a wave-uniform base, one lane
    // offset and immediates: the table of C tokens is [16 groups of 4 pairs][C][4] (cos, sin), 32 bytes per (group,
    // token), and holds a token block's worth of slack behind its last row, so that lanes past the end of a ragged
    // chunk still read inside it.  A wavefront that has no table reads the first bytes of the weights instead and,
    // like a V head, keeps its unrotated values.
    const bool have_table = MODE == kPjQkv && p.rope != nullptr;
    const char* tab_base = have_table ? (const char*)p.rope : p.a;
    const uint32_t group_bytes = have_table ? (uint32_t)p.b_rows * 32u : 0u;
    const uint32_t tab_lane = have_table ? (uint32_t)m0 * 32u + (uint32_t)hl * group_bytes : 0u;
    float4 tab0[8], tab1[8];     // the buffers of pair half 0 and 1 (two arrays: every index is a compile-time constant)
    auto tab_load = [&](int ib, int ip, float4 (&dst)[8]) __attribute__((always_inline)) {
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        // pairs i0 .. i0 + 3 with i0 = 32 ip + 8 rq + 4 hl: group i0 / 4 = 8 ip + 2 rq + hl
        const char* src = tab_base + (size_t)(8 * ip + 2 * rq) * group_bytes;       // wave-uniform
        const float4* cs = (const float4*)(src + tab_lane + ib * 1024);
        dst[2 * rq] = cs[0];
        dst[2 * rq + 1] = cs[1];
      }
    };
    step(t + 1, S1(), std::false_type(), std::false_type());

    // nobody reads LDS after the last barrier: the next tile's first two steps start loading under the epilogue
    cur_j = tile_index(s + n_li);
    if (cur_j >= 0) {
      pj_tile_of(p, cur_j, ta, tb);
      set_offsets(ta, tb);
#pragma unroll
      for (int u = 0; u < 16; ++u) issue_one(0, 0, u);
#pragma unroll
      for (int u = 0; u < 8; ++u) issue_one(1, 1, u);
    }

    if (MODE == kPjQkv) { tab_load(0, 0, tab0); tab_load(0, 1, tab1); }
    if (WIDE) {
      // bf16 output of whole heads / whole 128-feature runs: straight-line code, 16-byte stores
      auto group = [&](int ib, int ip, float4 (&tb8)[8], char* row, bool tok_ok) __attribute__((always_inline)) {
        if (MODE == kPjQkv) __builtin_amdgcn_sched_barrier(0);    // one group at a time: nothing of the next is computed early
        float lo[16], hi[16];                     // blocks ip and ip + 2 hold the rotary pairs
#pragma unroll
        for (int r = 0; r < 16; ++r) { lo[r] = acc[ip][ib][r]; hi[r] = acc[ip + 2][ib][r]; }
        if (MODE == kPjQkv) {
#pragma unroll
          for (int rq = 0; rq < 4; ++rq) {
            const float4 c01 = tb8[2 * rq], c23 = tb8[2 * rq + 1];                   // (cos, sin) of two pairs each
            const float cv[4] = {c01.x, c01.z, c23.x, c23.z}, sv[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float x = lo[4 * rq + e], y = hi[4 * rq + e];
              const float xr = pj_rot_lo(x, y, cv[e], sv[e]), yr = pj_rot_hi(x, y, cv[e], sv[e]);
              lo[4 * rq + e] = (rotate ? xr : x) * osc;   // selects, not a branch: V heads keep their values bit for bit
              hi[4 * rq + e] = (rotate ? yr : y) * osc;
            }
          }
          if (ib + 1 < 4) tab_load(ib + 1, ip, tb8);      // the buffer this group has just used: two groups ahead
        }
#pragma unroll
        for (int rp = 0; rp < 2; ++rp) {
          const float l8[8] = {lo[8 * rp], lo[8 * rp + 1], lo[8 * rp + 2], lo[8 * rp + 3],
                               lo[8 * rp + 4], lo[8 * rp + 5], lo[8 * rp + 6], lo[8 * rp + 7]};
          const float h8[8] = {hi[8 * rp], hi[8 * rp + 1], hi[8 * rp + 2], hi[8 * rp + 3],
                               hi[8 * rp + 4], hi[8 * rp + 5], hi[8 * rp + 6], hi[8 * rp + 7]};
          pj_store_rows_bf16(row + 32 * ip * 2, l8, rp, hl, tok_ok);
          pj_store_rows_bf16(row + 32 * (ip + 2) * 2, h8, rp, hl, tok_ok);
        }
      };
#pragma unroll
      for (int ib = 0; ib < 4; ++ib) {
        const int m = m0 + ib * 32;
        const bool tok_ok = m < p.b_rows && n_valid > 0;              // n_valid is 128 or, for a head past the last, 0
        char* row = base + (int64_t)m * row_bytes;                    // only stored to when tok_ok
        group(ib, 0, tab0, row, tok_ok);
        group(ib, 1, tab1, row, tok_ok);
      }
    } else {
      // fp32 output, a ragged last run of features or an odd row pitch: element by element
      int hl_slow = hl;            // opaque per tile: keeps this path's offsets from being hoisted out of the tile loop,
      asm volatile("" : "+v"(hl_slow));   // where they would sit in registers (or scratch) for nothing
      auto group = [&](int ib, int ip, float4 (&tb8)[8], char* row, bool tok_ok) __attribute__((always_inline)) {
        if (MODE == kPjQkv && ib > 0) tab_load(ib, ip, tb8);          // token block 0 was fetched above
        if (!tok_ok) return;
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int f = 32 * (ip + 2 * half) + 8 * (r >> 2) + 4 * hl_slow + (r & 3);
            float x = half ? acc[ip + 2][ib][r] : acc[ip][ib][r];
            if (MODE == kPjQkv && rotate) {
              const float4 cq = tb8[2 * (r >> 2) + ((r & 3) >> 1)];
              const float c = (r & 1) ? cq.z : cq.x, sn = (r & 1) ? cq.w : cq.y;
              const float other = half ? acc[ip][ib][r] : acc[ip + 2][ib][r];
              x = half ? pj_rot_hi(other, x, c, sn) : pj_rot_lo(x, other, c, sn);
            }
            if (MODE == kPjQkv) x *= osc;
            if (f >= n_valid) continue;
            if (p.out_fp32) *(float*)(row + f * 4) = x;
            else *(uint16_t*)(row + f * 2) = float_to_bf16_bits(x);
          }
      };
#pragma unroll
      for (int ib = 0; ib < 4; ++ib) {
        const int m = m0 + ib * 32;
        char* row = base + (int64_t)m * row_bytes;
        group(ib, 0, tab0, row, m < p.b_rows);
        group(ib, 1, tab1, row, m < p.b_rows);
      }
    }
    // The next tile's load offsets are formed again here rather than kept across the epilogue: kept, they are spilled
    // and reloaded, and the waits the compiler then puts before their first uses inside the contraction loop count
    // memory operations it cannot see - they would drain the operand loads that are meant to stay in flight.
    if (cur_j >= 0) {
      int ta2 = ta, tb2 = tb;
      asm volatile("" : "+v"(ta2), "+v"(tb2));
      set_offsets(ta2, tb2);
    }
  }
}

// ---- chunks too short to fill the chip with 256 x 256 tiles: the same contraction in 128 x 128 tiles, one per workgroup.
// 600 tokens of Llama-3-8B are 72 (Q/K/V) and 48 (output) of the large tiles on 256 compute units, 240 and 160 of these.
// A wavefront owns 64 x 64 (2 x 2 blocks of the 32x32x16 MFMA; its A rows are 32 wa .. +31 and 64 + 32 wa .. +31, so that
// rotary pairs still meet in one lane).  A step of 64 contraction elements moves 32 KB into LDS and 64 KB out of it.  Measured over contractions of 1024 to
// 8192 at 600 tokens, kernel time is 5 to 6 us to launch, fill the ring and write, and per step 0.53 us with weights from
// HBM and 0.43 with weights from the caches for the 240 workgroups of Q/K/V, 0.45 and 0.35 for the 160 of the output.  A step's
// MFMAs, its loads through the texture path (64 bytes a cycle) and its operand reads (128 bytes a cycle) take 512 cycles each; it takes 720, at a clock
// that falls with them (2.3 GHz with 48 workgroups at work, 1.8 with 240).  One workgroup per compute unit has to cover the
// latency of its loads itself: five stages of 32 KB, loads three steps (of 64 elements) ahead and spread evenly over the step,
// operand reads two sub-steps ahead with one wait for the four of a sub-step.  The order of every sum is the large
// tile's, so the results are the same bits.  Measured (hidden size 4096, 32 + 16 heads, weights of 6 layers in turn;
// large tile -> small): Q/K/V with its table at 64 / 600 / 1000 / 2000 tokens 90 -> 33, 97 -> 40, 102 -> 69, 110 -> 108 us,
// output 74 -> 24, 77 -> 28, 78 -> 35, 80 -> 66 us.  With four stages, all loads in the half step behind the barrier and a wait for the
// stage's last reads in front of it: 100 tokens 35.1 and 24.0 us, now 33.5 and 22.0; 600 40.0 and 32.3, now 39.1 and 31; 2000 110 and
// 67, now 107 and 65.
constexpr int kPsTile = 128;
constexpr int kPsOperandBytes = kPsTile * kPjRowBytes;    // 16 KiB
constexpr int kPsStageBytes = 2 * kPsOperandBytes;
constexpr int kPsStages = 5;
constexpr int kPsLdsBytes = kPsStages * kPsStageBytes;    // 160 KiB

// The rotation needs (cos, sin) of 64 pairs at the tile's 128 tokens.  Every workgroup forms them itself, under the latency of its first
// loads: a wavefront takes 32 tokens, a lane one pair (RopeRun, as the table of the 256-row tile does: the same bits), keeps them in
// 64 registers (there is one wavefront per SIMD) and puts them into the ring's place in LDS for the epilogue.  As a table of its own launch
// they were 5 us in front of this one: Q/K/V of 65 / 300 / 600 tokens at a hidden size of 4096 32.5 / 33.0 / 38.9 -> 30.2 / 30.9 / 37.1 us,
// of 600 tokens at 1024 12.3 -> 10.6.  The lane's frequency is in its register before the first load goes out: with a wait for it (and
// so for all loads) behind them, and 190 instructions less for the angles, 65 / 100 / 300 / 600 tokens take 33.7 / 37.1 / 32.7 / 38.9 us where
// this takes 33.4 / 36.7 / 32.4 / 38.6 (other weights and clocks than above; at a hidden size of 1024 10.28 and 10.33).
constexpr int kPsTrigPitch = kPsTile * 32 + 32;      // a group of 4 pairs: [token][4] (cos, sin), and 32 bytes against bank conflicts
static_assert(16 * kPsTrigPitch <= kPsLdsBytes, "the table takes the ring's place");

template <int MODE, class Rope>
__global__ __launch_bounds__(256, 1) void proj_gemm_small_kernel(ProjArgs p, Rope rope) {
  extern __shared__ __attribute__((aligned(1024))) char lds_dyn[];
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_char*)lds_dyn;
  const int lane = lane_id();
  const int wave = wave_id();
  const int l = lane & 31, hl = lane >> 5;
  const int wa = wave & 1, wb = wave >> 1;

  // XCD x (= blockIdx % 8) owns tiles [x * per, (x + 1) * per) of the ordered list: a compact block of the tile grid
  const int total = p.a_tiles * p.b_tiles;
  const int per = (total + 7) >> 3;
  const int slot = (int)(blockIdx.x >> 3), tile = (int)(blockIdx.x & 7) * per + slot;
  if (slot >= per || tile >= total) return;
  // this lane's frequency, asked for and waited for in front of the ring's first loads: the compiler does not count those, and a wait
  // behind them would be for all of them
  double freq = 0.0;
  if constexpr (MODE == kPjQkv) freq = rope.f.inv[lane];
  int ta, tb;
  pj_tile_of(p, tile, ta, tb);

  // tile traffic: this wavefront's 4 load instructions per operand and step cover rows 32 w + 8 u + lane / 8
  uint32_t ga_off[4], gb_off[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = 32 * wave + 8 * u + (lane >> 3);
    const int chunk = (lane & 7) ^ (4 * (u & 1) + (lane >> 4));      // = (lane & 7) ^ ((row >> 1) & 7)
    int ra = ta * kPsTile + row, rb = tb * kPsTile + row;
    ra = ra < p.a_rows ? ra : p.a_rows - 1;
    rb = rb < p.b_rows ? rb : p.b_rows - 1;
    ga_off[u] = (uint32_t)ra * p.a_stride + (chunk << 4);
    gb_off[u] = (uint32_t)rb * p.b_stride + (chunk << 4);
  }
  const uint32_t lds_wave = lds_base + wave * 4096;
  // load u of the step whose slices begin at ap and bp
  auto issue_one = [&](const char* ap, const char* bp, uint32_t stage, int u) __attribute__((always_inline)) {
    const uint32_t dst = lds_wave + stage + (u & 3) * 1024;
    if (u < 4) g2lds16_s<0>(ap, ga_off[u], dst);
    else g2lds16_s<0>(bp, gb_off[u - 4], dst + kPsOperandBytes);
  };
  auto b_slice = [&](int t) __attribute__((always_inline)) {
    const int k0 = t * kPjK;
    return MODE == kPjOut ? p.b + (int64_t)(k0 >> 7) * p.b_head_stride + (k0 & 127) * 2 : p.b + (int64_t)k0 * 2;
  };

  // operand reads: lane l reads row (block + l), chunk (2 kk + hl); operands 0, 1: A blocks, 2, 3: B blocks
  uint32_t va[4], vb[4];
  {
    const int sw = (l >> 1) & 7;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint32_t ko = (uint32_t)(l * kPjRowBytes + (((2 * kk + hl) ^ sw) << 4));
      va[kk] = lds_base + wa * 32 * kPjRowBytes + ko;
      vb[kk] = lds_base + kPsOperandBytes + wb * 64 * kPjRowBytes + ko;
    }
  }
  auto read_op = [&](uint32_t stage, int kk, int i) __attribute__((always_inline)) -> bf16x8 {
    return i < 2 ? *(lds_bf16x8_p)((lds_char*)(uintptr_t)(va[kk] + stage) + i * 64 * kPjRowBytes)
                 : *(lds_bf16x8_p)((lds_char*)(uintptr_t)(vb[kk] + stage) + (i - 2) * 32 * kPjRowBytes);
  };

  const int T = p.K / kPjK;        // at least 4 (the launcher's rule)
  if constexpr (MODE == kPjQkv) asm volatile("" : "+v"(freq) : : "memory");
#pragma unroll
  for (int t = 0; t < kPsStages - 1; ++t)
#pragma unroll
    for (int u = 0; u < (t < kPsStages - 2 ? 8 : 4); ++u) issue_one(p.a + t * kPjRowBytes, b_slice(t), t * kPsStageBytes, u);

  bool rotate = false;
  float trig_c[kRopeRun], trig_s[kRopeRun];  // this lane's pair at tokens 32 wave .. +31 of the tile
  if constexpr (MODE == kPjQkv) {
    rotate = rope.on && ta < p.n_q_heads + p.n_kv_heads;
    if (rotate) {
      RopeRun run(rope.past + tb * kPsTile + kRopeRun * wave, freq);
#pragma unroll
      for (int i = 0; i < kRopeRun; ++i) {
        run.next(trig_c[i], trig_s[i]);
        asm volatile("" : "+v"(trig_c[i]), "+v"(trig_s[i]));     // here, and not in front of the epilogue
      }
    }
  }

  f32x16 acc[2][2];
#pragma unroll
  for (int ia = 0; ia < 2; ++ia)
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ia][ib][r] = 0.f;
  bf16x8 op[4][4];
  auto mfma4 = [&](int kk, int j) __attribute__((always_inline)) {
    acc[j & 1][j >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[kk][j & 1], op[kk][2 + (j >> 1)], acc[j & 1][j >> 1], 0, 0, 0);
  };

  // one wait for the four operands of a sub-step
  auto here = [](bf16x8 (&x)[4]) __attribute__((always_inline)) { asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3])); };

  wait_vmcnt<20>();          // step 0 has landed
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int i = 0; i < 4; ++i) op[kk][i] = read_op(0, kk, i);

  // Step t, in stage st: sub-steps 0 and 1 read the operands of 2 and 3; the barrier publishes step t + 1 (stage sn); sub-steps 2
  // and 3 cover its first reads.  The loads go out evenly, one behind every second MFMA: the texture path takes 16 cycles for
  // each, 512 for the 32 of a workgroup's step, and four wavefronts that issue all of theirs in one half of a step wait for it.
  // In the first half these are the B rows of step t + 3 (stage sb), in the second the A rows of step t + 4, into stage sa, that of
  // step t - 1: every wavefront has used the last of that stage's operands before it came to this barrier, so nobody has to
  // wait for its reads there.  LEFT: steps after this one whose loads may still be in flight behind step t + 1's (8 per step).
  auto step = [&](uint32_t st, uint32_t sn, uint32_t sb, uint32_t sa, const char* bp, const char* ap, auto left_tag, auto a_tag, auto b_tag)
                  __attribute__((always_inline)) {
    constexpr int LEFT = decltype(left_tag)::value;          // -1: this is the last step
    constexpr bool A = decltype(a_tag)::value, B = decltype(b_tag)::value;
    const uint32_t fill_a = lds_wave + sa, fill_b = lds_wave + sb + kPsOperandBytes;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      here(op[kk]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = kk * 2 + (j >> 1);
        if (B && (j & 1)) set_m0(fill_b + u * 1024);
        op[kk + 2][j] = read_op(st, kk + 2, j);
        __builtin_amdgcn_sched_barrier(0);
        mfma4(kk, j);
        __builtin_amdgcn_sched_barrier(0);
        if (B && (j & 1)) g2lds16_m0(bp, gb_off[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (LEFT >= 0) {
      wait_vmcnt<LEFT < 0 ? 0 : 8 * LEFT>();                // this wave's loads of step t + 1 have landed
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      here(op[kk + 2]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = kk * 2 + (j >> 1);
        if (A && (j & 1)) set_m0(fill_a + u * 1024);
        if (LEFT >= 0) op[kk][j] = read_op(sn, kk, j);
        __builtin_amdgcn_sched_barrier(0);
        mfma4(kk + 2, j);
        __builtin_amdgcn_sched_barrier(0);
        if (A && (j & 1)) g2lds16_m0(ap, ga_off[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto after = [](uint32_t stage) __attribute__((always_inline)) { return stage + kPsStageBytes < (uint32_t)kPsLdsBytes ? stage + kPsStageBytes : 0u; };
  using Yes = std::true_type;
  using No = std::false_type;
  uint32_t st = 0, sb = (kPsStages - 2) * kPsStageBytes, sa = (kPsStages - 1) * kPsStageBytes;
  const char* ap = p.a + (kPsStages - 1) * kPjRowBytes;
  int t = 0;
  for (; t + kPsStages - 1 < T; ++t) {
    const uint32_t sn = after(st);
    step(st, sn, sb, sa, b_slice(t + kPsStages - 2), ap, std::integral_constant<int, 2>(), Yes(), Yes());
    ap += kPjRowBytes;
    sb = sa;
    sa = st;
    st = sn;
  }
  step(st, after(st), sb, 0, b_slice(T - 1), nullptr, std::integral_constant<int, 2>(), No(), Yes());
  st = after(st);
  step(st, after(st), 0, 0, nullptr, nullptr, std::integral_constant<int, 1>(), No(), No());
  st = after(st);
  step(st, after(st), 0, 0, nullptr, nullptr, std::integral_constant<int, 0>(), No(), No());
  step(after(st), 0, 0, 0, nullptr, nullptr, std::integral_constant<int, -1>(), No(), No());

  if (MODE == kPjQkv && rotate) {
    __syncthreads();             // nobody reads the ring any more
    char* const at = lds_dyn + (lane >> 2) * kPsTrigPitch + wave * 1024 + (lane & 3) * 8;
#pragma unroll
    for (int i = 0; i < 32; ++i) *(float2*)(at + i * 32) = make_float2(trig_c[i], trig_s[i]);
    __syncthreads();
  }

  // Register r of block (ia, ib): feature 64 ia + 32 wa + 8 (r / 4) + 4 hl + r % 4 of the tile, token 64 wb + 32 ib + l.
  char* base;
  int64_t row_bytes;
  float osc = 1.0f;
  if (MODE == kPjQkv) {
    const int head = ta;
    int hh;
    if (head < p.n_q_heads) { base = (char*)p.q_out; hh = head; osc = p.q_scale; }
    else if (head < p.n_q_heads + p.n_kv_heads) { base = (char*)p.k_out; hh = head - p.n_q_heads; }
    else { base = (char*)p.v_out; hh = head - p.n_q_heads - p.n_kv_heads; }
    base += (int64_t)hh * p.b_rows * kRowBytes;
    row_bytes = kRowBytes;
  } else {
    base = (char*)p.y + (int64_t)ta * kPsTile * 2;
    row_bytes = p.y_stride * 2;
  }
#pragma unroll
  for (int ib = 0; ib < 2; ++ib) {
    const int m = tb * kPsTile + 64 * wb + 32 * ib + l;
    const bool ok = m < p.b_rows;
    float lo[16], hi[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) { lo[r] = acc[0][ib][r]; hi[r] = acc[1][ib][r]; }
    if (MODE == kPjQkv) {
      if (rotate) {
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          const float4* cs = (const float4*)(lds_dyn + (8 * wa + 2 * rq + hl) * kPsTrigPitch + (64 * wb + 32 * ib + l) * 32);
          const float4 c01 = cs[0], c23 = cs[1];
          const float cv[4] = {c01.x, c01.z, c23.x, c23.z}, sv[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = lo[4 * rq + e], y = hi[4 * rq + e];
            lo[4 * rq + e] = pj_rot_lo(x, y, cv[e], sv[e]);
            hi[4 * rq + e] = pj_rot_hi(x, y, cv[e], sv[e]);
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) { lo[r] *= osc; hi[r] *= osc; }
    }
    char* row = base + (int64_t)m * row_bytes + 32 * wa * 2;
#pragma unroll
    for (int rp = 0; rp < 2; ++rp) {
      const float l8[8] = {lo[8 * rp], lo[8 * rp + 1], lo[8 * rp + 2], lo[8 * rp + 3],
                           lo[8 * rp + 4], lo[8 * rp + 5], lo[8 * rp + 6], lo[8 * rp + 7]};
      const float h8[8] = {hi[8 * rp], hi[8 * rp + 1], hi[8 * rp + 2], hi[8 * rp + 3],
                           hi[8 * rp + 4], hi[8 * rp + 5], hi[8 * rp + 6], hi[8 * rp + 7]};
      pj_store_rows_bf16(row, l8, rp, hl, ok);
      pj_store_rows_bf16(row + 128, h8, rp, hl, ok);
    }
  }
}

// (cos, sin) of position (past + t) times theta^(-i / 64) for i < 64: a thread takes a pair at 32 tokens, the runs of the 128-row tile
__global__ __launch_bounds__(64) void rope_table_kernel(float2* __restrict__ out, int64_t past, int n, RopeFreqs f) {
  const int i = threadIdx.x, t0 = blockIdx.x * kRopeRun;
  RopeRun run(past + t0, f.inv[i]);
  float2* const at = out + ((int64_t)(i >> 2) * n + t0) * 4 + (i & 3);   // [i / 4][token][i % 4]
  const int left = n - t0 < kRopeRun ? n - t0 : kRopeRun;
  for (int k = 0; k < left; ++k) {
    float c, s;
    run.next(c, s);
    at[4 * k] = make_float2(c, s);
  }
}

// ---- 2 to 64 tokens: the read of the weights is the bound (50 MB of Q/K/V at a hidden size of 4096), and the 128-row tiles
// would leave it to 48 compute units.  A workgroup takes 16 RB weight rows (of Q/K/V: 8 RB rotary pairs of a head) and all
// tokens, NT blocks of 16; its 4 wavefronts share the contraction in turns of 64 elements and add their sums through LDS at
// the end.  Each wavefront streams its rows through an LDS ring of its own (direct-to-LDS loads, partial vmcnt waits, no
// barrier in the loop).  The rotation's angles are formed in double precision while the first loads are in flight; no table
// is needed.  One row block and two workgroups per compute unit (17 KB per wavefront) up to 16 tokens, and for the output
// projection up to 32; with more tokens the activations are most of what a workgroup reads, so Q/K/V takes two row blocks,
// and one workgroup has all of LDS (36 KB per wavefront).
// Measured at 2 / 16 / 32 / 64 tokens (weights of 6 layers in turn, hidden size 4096, 32 + 16 heads; the 256-row tiles took
// 87 to 91 and 74 us, the 128-row tiles 30 to 33 and 23): Q/K/V 12.2 / 13.6 / 16.0 / 18.5 us (4.1 TB/s of weights at 2),
// output 7.9 / 8.0 / 8.5 / 10.3 us.  Q/K/V of 16 tokens with two row blocks: 15.4 us; of 64 with one: 24.0.
template <int MODE, int NT> constexpr int kPfwRowBlocks = MODE == kPjQkv && NT > 1 ? 2 : 1;
template <int MODE, int NT> constexpr int kPfwStageBytes = (kPfwRowBlocks<MODE, NT> + NT) * 16 * kPjRowBytes;
template <int MODE, int NT> constexpr int kPfwWaveBytes = (kPfwRowBlocks<MODE, NT> == 1 && NT <= 2 ? 17 : 36) * 1024;
template <int MODE, int NT> constexpr int kPfwStages =
    kPfwWaveBytes<MODE, NT> / kPfwStageBytes<MODE, NT> < 8 ? kPfwWaveBytes<MODE, NT> / kPfwStageBytes<MODE, NT> : 8;
template <int MODE, int NT> constexpr int kPfwRings = 4 * kPfwStages<MODE, NT> * kPfwStageBytes<MODE, NT>;
template <int MODE, int NT> constexpr int kPfwLdsBytes = kPfwRings<MODE, NT> + 16 * 16 * NT * 8;     // then (cos, sin) of the pairs
constexpr int kPfwMaxTokens = 64;

template <int MODE, int NT>
__global__ __launch_bounds__(256, 1) void proj_few_kernel(ProjArgs p, int64_t past, RopeFreqs f, int rotate_heads) {
  constexpr int RB = kPfwRowBlocks<MODE, NT>, kPairs = 8 * RB;
  constexpr int kStage = kPfwStageBytes<MODE, NT>, kStages = kPfwStages<MODE, NT>, kLoads = 2 * (RB + NT);
  static_assert(kStages >= 2 && (kStages - 1) * kLoads < 64 && kPfwLdsBytes<MODE, NT> <= 160 * 1024, "ring");
  static_assert(4 * 16 * RB * 16 * NT * 4 <= kPfwRings<MODE, NT>, "the sums take the rings' place");
  extern __shared__ __attribute__((aligned(1024))) char lds_dyn[];
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_char*)lds_dyn;
  const int lane = lane_id();
  const int wave = wave_id();
  const int c16 = lane & 15, g4 = lane >> 4;
  const uint32_t ring = lds_base + wave * (kStages * kStage);

  // weight row of tile row r: the first half of the Q/K/V rows are dims i0 .. of the head, the second their partners i0 + 64 ..
  const int head = blockIdx.x / (64 / kPairs), i0 = blockIdx.x % (64 / kPairs) * kPairs;
  auto weight_row = [&](int r) { return MODE == kPjQkv ? head * kHeadDim + i0 + r % kPairs + 64 * (r / kPairs) : (int)blockIdx.x * 16 + r; };
  uint32_t off[kLoads];          // this lane's byte offset of each load instruction (8 rows of 128 bytes)
#pragma unroll
  for (int u = 0; u < kLoads; ++u) {
    const int r = 8 * u + (lane >> 3);
    const int chunk = (lane & 7) ^ ((r >> 1) & 7);
    if (u < 2 * RB) {
      int row = weight_row(r);
      row = row < p.a_rows ? row : p.a_rows - 1;
      off[u] = (uint32_t)row * p.a_stride + (chunk << 4);
    } else {
      int row = r - 16 * RB;
      row = row < p.b_rows ? row : p.b_rows - 1;
      off[u] = (uint32_t)row * p.b_stride + (chunk << 4);
    }
  }
  const int T = p.K / kPjK;
  const int cnt = wave < T ? (T - wave + 3) / 4 : 0;           // steps of this wavefront: wave, wave + 4, ...
  auto issue = [&](int i, int stage) __attribute__((always_inline)) {
    const int k0 = (wave + 4 * i) * kPjK;
    const char* ab = p.a + (int64_t)k0 * 2;
    const char* bb = MODE == kPjOut ? p.b + (int64_t)(k0 >> 7) * p.b_head_stride + (k0 & 127) * 2 : p.b + (int64_t)k0 * 2;
    const uint32_t dst = ring + stage * kStage;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) g2lds16_s<0>(u < 2 * RB ? ab : bb, off[u], dst + u * 1024);
  };
#pragma unroll
  for (int i = 0; i < kStages - 1; ++i)
    if (i < cnt) issue(i, i);

  // (cos, sin) of pair i0 + tid % 16 at tokens tid / 16 + 16 n: the first angle, then steps of 16 positions, all in double
  float2* trig = (float2*)(lds_dyn + kPfwRings<MODE, NT>);
  const bool rotate = MODE == kPjQkv && head < rotate_heads;
  const int my_pair = threadIdx.x & 15, t0 = threadIdx.x >> 4;
  if (rotate && my_pair < kPairs) {
    const double w = f.inv[i0 + my_pair];
    double s, c, s16 = 0.0, c16d = 1.0;
    sincos((double)(past + t0) * w, &s, &c);
    if (NT > 1) sincos(16.0 * w, &s16, &c16d);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      trig[my_pair * (16 * NT) + t0 + 16 * n] = make_float2((float)c, (float)s);
      const double cn = c * c16d - s * s16;
      s = s * c16d + c * s16;
      c = cn;
    }
  }

  f32x4 acc[RB][NT];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[rb][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  uint32_t rd[2];                // operand reads: row c16 of a 16-row block, chunk 4 kk + g4
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) rd[kk] = ring + c16 * kPjRowBytes + (((4 * kk + g4) ^ ((c16 >> 1) & 7)) << 4);
  int stage = 0, fill = kStages - 1;
  for (int i = 0; i < cnt; ++i) {
    if (i + kStages - 1 < cnt) {
      issue(i + kStages - 1, fill);
      wait_vmcnt<(kStages - 1) * kLoads>();          // the oldest stage has landed
    } else {
      wait_vmcnt<0>();
    }
    const uint32_t at = stage * kStage;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      bf16x8 a[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) a[rb] = *(lds_bf16x8_p)((lds_char*)(uintptr_t)(rd[kk] + at) + rb * 2048);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const bf16x8 b = *(lds_bf16x8_p)((lds_char*)(uintptr_t)(rd[kk] + at) + (RB + nt) * 2048);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[rb][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb], b, acc[rb][nt], 0, 0, 0);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // done reading before the stage is filled again
    stage = stage + 1 < kStages ? stage + 1 : 0;
    fill = fill + 1 < kStages ? fill + 1 : 0;
  }

  // sums of the four wavefronts, [wavefront][row][token]
  __syncthreads();
  float* red = (float*)lds_dyn;
  constexpr int kTok = 16 * NT, kPlane = 16 * RB * kTok;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave * kPlane + (16 * rb + 4 * g4 + r) * kTok + 16 * nt + c16] = acc[rb][nt][r];
  __syncthreads();
  const int j4 = threadIdx.x & 3, tok = threadIdx.x >> 2;      // this thread writes features (or pairs) 4 j4 .. + 3 of token tok
  if (tok >= p.b_rows || tok >= kTok || (MODE == kPjQkv && 4 * j4 >= kPairs)) return;
  float v[2][4];                 // Q/K/V: the pairs' first and second members
#pragma unroll
  for (int half = 0; half < (MODE == kPjQkv ? 2 : 1); ++half)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* src = red + (kPairs * half + 4 * j4 + e) * kTok + tok;
      v[half][e] = (src[0] + src[kPlane]) + (src[2 * kPlane] + src[3 * kPlane]);
    }
  const int esz = p.out_fp32 ? 4 : 2;
  if (MODE == kPjQkv) {
    char* base;
    int hh;
    float osc = 1.0f;
    if (head < p.n_q_heads) { base = (char*)p.q_out; hh = head; osc = p.q_scale; }
    else if (head < p.n_q_heads + p.n_kv_heads) { base = (char*)p.k_out; hh = head - p.n_q_heads; }
    else { base = (char*)p.v_out; hh = head - p.n_q_heads - p.n_kv_heads; }
    base += (((int64_t)hh * p.b_rows + tok) * kHeadDim + i0 + 4 * j4) * esz;
    float lo[4], hi[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = v[0][e], y = v[1][e];
      const float2 t = rotate ? trig[(4 * j4 + e) * kTok + tok] : make_float2(1.f, 0.f);
      lo[e] = (rotate ? pj_rot_lo(x, y, t.x, t.y) : x) * osc;
      hi[e] = (rotate ? pj_rot_hi(x, y, t.x, t.y) : y) * osc;
    }
    if (p.out_fp32) {
      *(float4*)base = make_float4(lo[0], lo[1], lo[2], lo[3]);
      *(float4*)(base + 64 * 4) = make_float4(hi[0], hi[1], hi[2], hi[3]);
    } else {
      *(uint2*)base = make_uint2(pj_pack2(lo[0], lo[1]), pj_pack2(lo[2], lo[3]));
      *(uint2*)(base + 64 * 2) = make_uint2(pj_pack2(hi[0], hi[1]), pj_pack2(hi[2], hi[3]));
    }
  } else {
    const int row = blockIdx.x * 16 + 4 * j4;
    char* base = (char*)p.y + ((int64_t)tok * p.y_stride + row) * esz;
    if (row + 4 <= p.a_rows && p.y_stride % 4 == 0) {
      if (p.out_fp32) *(float4*)base = make_float4(v[0][0], v[0][1], v[0][2], v[0][3]);
      else *(uint2*)base = make_uint2(pj_pack2(v[0][0], v[0][1]), pj_pack2(v[0][2], v[0][3]));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (row + e < p.a_rows) {
          if (p.out_fp32) ((float*)base)[e] = v[0][e];
          else ((uint16_t*)base)[e] = float_to_bf16_bits(v[0][e]);
        }
    }
  }
}

// ---- one token (decode): the same two projections as matrix-vector products, bound by the HBM read of the weights.
// A wavefront takes pairs of weight rows (for Q/K/V: dimension i and i + 64 of a head, the two members of a rotary
// pair), each lane 16 bytes of every 1 KiB of the row against the matching 16 bytes of x, fp32 accumulation, one
// cross-lane reduction per row.
struct GemvArgs {
  const uint16_t* w;      // [rows][K] bf16
  const uint16_t* x;      // [K] bf16
  int rows, K;
  int mode, out_fp32;
  void* q_out; void* k_out; void* v_out; int n_q_heads, n_kv_heads;   // kPjQkv
  int64_t position; double log2_theta;                                // rotation angle position * 2^(-i/64 * log2_theta); < 0: none
  float q_scale;                                                      // kPjQkv: factor on the query heads' outputs
  void* y;                                                            // kPjOut
};

__device__ __forceinline__ uint4 gemv_load_stream(const uint16_t* p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ float gemv_dot8(uint4 a, uint4 b) {
  const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s = __builtin_fmaf(__uint_as_float(av[e] << 16), __uint_as_float(bv[e] << 16), s);
    s = __builtin_fmaf(__uint_as_float(av[e] & 0xFFFF0000u), __uint_as_float(bv[e] & 0xFFFF0000u), s);
  }
  return s;
}

constexpr int kGemvChunks = 8;
__global__ __launch_bounds__(256) void proj_gemv_kernel(GemvArgs g) {
  const int lane = lane_id();
  const int wave_global = blockIdx.x * 4 + wave_id();
  const int n_waves = gridDim.x * 4;
  const int n_pairs = g.mode == kPjQkv ? g.rows / 2 : (g.rows + 1) / 2;
  for (int pr = wave_global; pr < n_pairs; pr += n_waves) {
    int ra, rb;
    if (g.mode == kPjQkv) { ra = (pr >> 6) * kHeadDim + (pr & 63); rb = ra + 64; }
    else { ra = 2 * pr; rb = ra + 1 < g.rows ? ra + 1 : ra; }
    const uint16_t* wa = g.w + (int64_t)ra * g.K;
    const uint16_t* wb = g.w + (int64_t)rb * g.K;
    float sa = 0.f, sb = 0.f;
    // 8 x 512 contraction elements per round: both rows of a Llama-3-8B pair (4096 each) are in flight at once,
    // 16 loads of 16 bytes per lane, instead of two dependent rounds of 8
    for (int k0 = lane * 8; k0 < g.K; k0 += kGemvChunks * 512) {
      uint4 a[kGemvChunks], b[kGemvChunks], xv[kGemvChunks];
#pragma unroll
      for (int c = 0; c < kGemvChunks; ++c) {
        const int k = k0 + c * 512;
        const int kc = k < g.K ? k : 0;                  // in bounds; the product is dropped below
        a[c] = gemv_load_stream(wa + kc);                // the weights are read once: non-temporal
        b[c] = gemv_load_stream(wb + kc);
        xv[c] = *(const uint4*)(g.x + kc);
      }
#pragma unroll
      for (int c = 0; c < kGemvChunks; ++c)
        if (k0 + c * 512 < g.K) { sa += gemv_dot8(a[c], xv[c]); sb += gemv_dot8(b[c], xv[c]); }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { sa += __shfl_xor(sa, off); sb += __shfl_xor(sb, off); }
    if (lane != 0) continue;
    if (g.mode == kPjQkv) {
      const int head = pr >> 6, i = pr & 63;
      char* base;
      int hh;
      if (head < g.n_q_heads) { base = (char*)g.q_out; hh = head; }
      else if (head < g.n_q_heads + g.n_kv_heads) { base = (char*)g.k_out; hh = head - g.n_q_heads; }
      else { base = (char*)g.v_out; hh = head - g.n_q_heads - g.n_kv_heads; }
      float lo = sa, hi = sb;
      if (g.log2_theta >= 0 && head < g.n_q_heads + g.n_kv_heads) {
        double sn, cs;
        sincos((double)g.position * exp2(-(double)i / 64.0 * g.log2_theta), &sn, &cs);
        const float c = (float)cs, s = (float)sn;
        lo = sa * c - sb * s;
        hi = sb * c + sa * s;
      }
      if (head < g.n_q_heads) { lo *= g.q_scale; hi *= g.q_scale; }
      const int64_t at = (int64_t)hh * kHeadDim + i;
      if (g.out_fp32) { ((float*)base)[at] = lo; ((float*)base)[at + 64] = hi; }
      else { ((uint16_t*)base)[at] = float_to_bf16_bits(lo); ((uint16_t*)base)[at + 64] = float_to_bf16_bits(hi); }
    } else {
      if (g.out_fp32) { ((float*)g.y)[ra] = sa; if (rb != ra) ((float*)g.y)[rb] = sb; }
      else { ((uint16_t*)g.y)[ra] = float_to_bf16_bits(sa); if (rb != ra) ((uint16_t*)g.y)[rb] = float_to_bf16_bits(sb); }
    }
  }
}

static hi_status gemv_launch(void* stream, const GemvArgs& g) {
  const int n_pairs = (g.rows + 1) / 2;
  int wgs = (n_pairs + 3) / 4;              // at least one pair per wavefront
  if (wgs > 2048) wgs = 2048;
  hipLaunchKernelGGL(proj_gemv_kernel, dim3((unsigned)wgs), dim3(256), 0, (hipStream_t)stream, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error("projection (one token) launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

// table: room for the rotary table of the chunk, which the large tile reads (rope.on)
static hi_status pj_launch(void* stream, ProjArgs& p, int mode, const RopeChunk& rope, void* table) {
  static std::once_flag attr_once;      // the projections are stateless: any host thread may get here first
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [] {
    const void* kernels[6] = {(const void*)proj_gemm_kernel<kPjQkv, true>, (const void*)proj_gemm_kernel<kPjQkv, false>,
                              (const void*)proj_gemm_kernel<kPjOut, true>, (const void*)proj_gemm_kernel<kPjOut, false>,
                              (const void*)proj_gemm_small_kernel<kPjQkv, RopeChunk>, (const void*)proj_gemm_small_kernel<kPjOut, NoRope>};
    for (int i = 0; i < 6 && attr_err == hipSuccess; ++i)
      attr_err = hipFuncSetAttribute(kernels[i], hipFuncAttributeMaxDynamicSharedMemorySize, i < 4 ? kPjLdsBytes : kPsLdsBytes);
  });
  if (attr_err != hipSuccess) { set_last_error("hipFuncSetAttribute: %s", hipGetErrorString(attr_err)); return HI_ERR_HIP; }
  p.a_tiles = (int)ceil_div(p.a_rows, kPjTile);
  p.b_tiles = (int)ceil_div(p.b_rows, kPjTile);
  p.ga = p.a_tiles / 8 > 0 ? p.a_tiles / 8 : 1;
  const int total = p.a_tiles * p.b_tiles;
  const int per = (total + 7) / 8;
  // persistent workgroups: at most 32 per XCD (one per compute unit), each looping over its share of the tiles
  dim3 grid((unsigned)(8 * (per < kPjWgsPerXcd ? per : kPjWgsPerXcd)));
  // 16-byte stores need bf16 output, whole runs of 128 features per wavefront and an aligned row pitch
  const bool wide = !p.out_fp32 && p.a_rows % 128 == 0 && (mode == kPjQkv || (p.y_stride * 2) % 16 == 0);
  const dim3 block(kPjWaves * 64);
  // Which tile: at a contraction of 4096 a round of 256 small tiles takes 31 to 36 us; 256 large ones take 106, and a last round with
  // fewer of them 66 to 86 (a few, no power limit) to 108.  Measured with either tile forced (hidden size 4096, small / large):
  // Q/K/V of 1200 tokens 71 / 89 us, 1400 94 / 89, 1700 99 / 93, 2000 106 / 98, 2400 130 / 108, 2600 to 3300, where the large one starts
  // a second round, 136 / 178 to 167 / 190, 4000 199 / 198, 4600 227 / 205; output of 2000 65 / 70, 2600 89 / 84, 4000 126 / 108, 4600 153 / 179,
  // 5200 181 / 179.  Of 108 such pairs (500 to 6000 tokens, hidden sizes 1024, 4096, 8192) the sums below pick the slower one in 3, by
  // 1.8 % at most.
  const int64_t small_tiles = ceil_div(p.a_rows, kPsTile) * ceil_div(p.b_rows, kPsTile), rest = total % 256;
  const int64_t small_us = 35 * ceil_div(small_tiles, 256);
  const int64_t large_us = 106 * (total / 256) + (rest ? 72 + 36 * rest / 256 : 0);
  if (wide && p.K >= (kPsStages - 1) * kPjK && small_us < large_us) {
    p.a_tiles = (int)ceil_div(p.a_rows, kPsTile);
    p.b_tiles = (int)ceil_div(p.b_rows, kPsTile);
    p.ga = p.a_tiles / 8 > 0 ? p.a_tiles / 8 : 1;
    const dim3 sgrid((unsigned)(8 * ceil_div(small_tiles, 8)));
    if (mode == kPjQkv) hipLaunchKernelGGL((proj_gemm_small_kernel<kPjQkv, RopeChunk>), sgrid, block, kPsLdsBytes, (hipStream_t)stream, p, rope);
    else hipLaunchKernelGGL((proj_gemm_small_kernel<kPjOut, NoRope>), sgrid, block, kPsLdsBytes, (hipStream_t)stream, p, NoRope());
    hipError_t es = hipGetLastError();
    if (es != hipSuccess) { set_last_error("projection launch: %s", hipGetErrorString(es)); return HI_ERR_HIP; }
    return HI_OK;
  }
  if (rope.on) {
    hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)ceil_div(p.b_rows, kRopeRun)), dim3(64), 0, (hipStream_t)stream,
                       (float2*)table, rope.past, p.b_rows, rope.f);
    hipError_t er = hipGetLastError();
    if (er != hipSuccess) { set_last_error("rope table launch: %s", hipGetErrorString(er)); return HI_ERR_HIP; }
    p.rope = (const float2*)table;
  }
  if (mode == kPjQkv && wide) hipLaunchKernelGGL((proj_gemm_kernel<kPjQkv, true>), grid, block, kPjLdsBytes, (hipStream_t)stream, p);
  else if (mode == kPjQkv) hipLaunchKernelGGL((proj_gemm_kernel<kPjQkv, false>), grid, block, kPjLdsBytes, (hipStream_t)stream, p);
  else if (wide) hipLaunchKernelGGL((proj_gemm_kernel<kPjOut, true>), grid, block, kPjLdsBytes, (hipStream_t)stream, p);
  else hipLaunchKernelGGL((proj_gemm_kernel<kPjOut, false>), grid, block, kPjLdsBytes, (hipStream_t)stream, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error("projection launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

template <int MODE, int NT>
static hipError_t pj_few_go(void* stream, const ProjArgs& p, int64_t past, const RopeFreqs& f, int rotate_heads) {
  constexpr int lds = kPfwLdsBytes<MODE, NT>;
  static std::once_flag once;
  static hipError_t attr = hipSuccess;
  std::call_once(once, [] { attr = hipFuncSetAttribute((const void*)proj_few_kernel<MODE, NT>, hipFuncAttributeMaxDynamicSharedMemorySize, lds); });
  if (attr != hipSuccess) return attr;
  const unsigned wgs = (unsigned)ceil_div(p.a_rows, 16 * kPfwRowBlocks<MODE, NT>);
  hipLaunchKernelGGL((proj_few_kernel<MODE, NT>), dim3(wgs), dim3(256), lds, (hipStream_t)stream, p, past, f, rotate_heads);
  return hipGetLastError();
}

// rotate_heads: the leading heads (queries, then keys) that are rotated
template <int MODE>
static hi_status pj_few_launch(void* stream, const ProjArgs& p, int64_t past, const RopeFreqs& f, int rotate_heads) {
  const hipError_t e = p.b_rows <= 16 ? pj_few_go<MODE, 1>(stream, p, past, f, rotate_heads)
                     : p.b_rows <= 32 ? pj_few_go<MODE, 2>(stream, p, past, f, rotate_heads)
                                      : pj_few_go<MODE, 4>(stream, p, past, f, rotate_heads);
  if (e != hipSuccess) { set_last_error("projection (few tokens) launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

static bool pj_aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

#define HI_PJ_TRY(call)               \
  do {                                \
    hi_status s_ = (call);            \
    if (s_ != HI_OK) return s_;       \
  } while (0)

}  // namespace hi

using namespace hi;

extern "C" hi_status hi_proj_workspace_bytes(int32_t chunk, int64_t* bytes) {
  if (chunk < 1 || !bytes) { set_last_error("projection workspace: bad argument"); return HI_ERR_ARG; }
  // the table of the chunk plus a token block's worth of slack (see the epilogue of proj_gemm_kernel)
  *bytes = (int64_t)chunk * 64 * sizeof(float2) + kPjTile * 32;
  return HI_OK;
}

// hi_qkv_rope and its variant without a workspace argument; the rotary table goes to workspace_dev either way
static hi_status qkv_rope_impl(void* stream, const void* x_dev, const void* w_qkv_dev, int32_t d_model,
                               int32_t n_q_heads, int32_t n_kv_heads, int32_t chunk_len, int64_t past_len,
                               double rope_theta, int32_t out_fp32, void* q_out_dev, void* k_out_dev,
                               void* v_out_dev, void* workspace_dev, float q_scale) {
  if (!x_dev || !w_qkv_dev || !q_out_dev || !k_out_dev || !v_out_dev || (rope_theta > 0 && chunk_len > 1 && !workspace_dev)) {
    set_last_error("qkv projection: null buffer");
    return HI_ERR_ARG;
  }
  if (!pj_aligned16(x_dev) || !pj_aligned16(w_qkv_dev) || !pj_aligned16(q_out_dev) || !pj_aligned16(k_out_dev) ||
      !pj_aligned16(v_out_dev) || !pj_aligned16(workspace_dev)) {
    set_last_error("qkv projection: buffers must be 16-byte aligned");
    return HI_ERR_ARG;
  }
  if (n_q_heads < 1 || n_kv_heads < 1 || chunk_len < 1 || past_len < 0 || rope_theta < 0 || (out_fp32 != 0 && out_fp32 != 1) ||
      !(q_scale > 0.0f) || !(q_scale < 3.0e38f)) {
    set_last_error("qkv projection: bad shape");
    return HI_ERR_ARG;
  }
  const int64_t n_out = (int64_t)(n_q_heads + 2 * n_kv_heads) * kHeadDim;
  if (d_model < 2 * kPjK || d_model % (2 * kPjK) != 0 || n_out * d_model * 2 >= (1LL << 32) ||
      (int64_t)chunk_len * d_model * 2 >= (1LL << 32)) {
    set_last_error("qkv projection: d_model must be a multiple of %d and each operand smaller than 4 GiB", 2 * kPjK);
    return HI_ERR_UNSUPPORTED;
  }
  if (chunk_len == 1) {
    GemvArgs g = {};
    g.w = (const uint16_t*)w_qkv_dev; g.x = (const uint16_t*)x_dev;
    g.rows = (int)n_out; g.K = d_model;
    g.mode = kPjQkv; g.out_fp32 = out_fp32;
    g.q_out = q_out_dev; g.k_out = k_out_dev; g.v_out = v_out_dev;
    g.n_q_heads = n_q_heads; g.n_kv_heads = n_kv_heads;
    g.position = past_len;
    g.log2_theta = rope_theta > 0 ? log2(rope_theta) : -1.0;
    g.q_scale = q_scale;
    return gemv_launch(stream, g);
  }
  ProjArgs p = {};
  p.a = (const char*)w_qkv_dev; p.b = (const char*)x_dev;
  p.a_rows = (int)n_out; p.b_rows = chunk_len;
  p.a_stride = (uint32_t)d_model * 2; p.b_stride = (uint32_t)d_model * 2;
  p.K = d_model;
  p.out_fp32 = out_fp32;
  p.q_out = q_out_dev; p.k_out = k_out_dev; p.v_out = v_out_dev;
  p.n_q_heads = n_q_heads; p.n_kv_heads = n_kv_heads;
  p.rope = nullptr;
  p.q_scale = q_scale;
  RopeChunk rope = {};
  rope.past = past_len;
  rope.on = rope_theta > 0;
  if (rope.on)
    for (int i = 0; i < 64; ++i) rope.f.inv[i] = pow(rope_theta, -(double)i / 64.0);
  if (chunk_len <= kPfwMaxTokens) return pj_few_launch<kPjQkv>(stream, p, past_len, rope.f, rope.on ? n_q_heads + n_kv_heads : 0);
  return pj_launch(stream, p, kPjQkv, rope, workspace_dev);
}

extern "C" hi_status hi_qkv_rope(void* stream, const void* x_dev, const void* w_qkv_dev, int32_t d_model,
                                 int32_t n_q_heads, int32_t n_kv_heads, int32_t chunk_len, int64_t past_len,
                                 double rope_theta, int32_t out_fp32, void* q_out_dev, void* k_out_dev,
                                 void* v_out_dev, void* workspace_dev, float q_scale) {
  return qkv_rope_impl(stream, x_dev, w_qkv_dev, d_model, n_q_heads, n_kv_heads, chunk_len, past_len, rope_theta,
                       out_fp32, q_out_dev, k_out_dev, v_out_dev, workspace_dev, q_scale);
}

// ---- the variant for callers that cannot allocate: the chunk's rotary table lives in a file-scope device array.
// Every GPU holds its own copy of the array at its own address; in host code the array's name is only a stand-in,
// so the address is looked up once per device (with that device current) and only that pointer is handed to kernels.
constexpr int kQkvStaticMaxChunk = 16384;
constexpr int kQkvStaticMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[(size_t)kQkvStaticMaxChunk * 64 * sizeof(float2)];   // 8 MiB

static hi_status qkv_static_scratch(void** out) {
  static std::mutex mu;
  static void* ptr_of_device[kQkvStaticMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) { set_last_error("hipGetDevice: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  if (dev < 0 || dev >= kQkvStaticMaxDevices) { set_last_error("device index %d out of range", dev); return HI_ERR_UNSUPPORTED; }
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr_of_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) { set_last_error("hipGetSymbolAddress: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
    ptr_of_device[dev] = p;
  }
  *out = ptr_of_device[dev];
  return HI_OK;
}

extern "C" hi_status hi_qkv_rope_static(void* stream, const void* x_dev, const void* w_qkv_dev, int32_t d_model,
                                        int32_t n_q_heads, int32_t n_kv_heads, int32_t chunk_len, int64_t past_len,
                                        double rope_theta, int32_t out_fp32, void* q_out_dev, void* k_out_dev,
                                        void* v_out_dev, float q_scale) {
  if (chunk_len > kQkvStaticMaxChunk) {
    set_last_error("qkv projection without a workspace: chunk_len %d exceeds the built-in table of %d tokens", chunk_len,
                   kQkvStaticMaxChunk);
    return HI_ERR_RANGE;
  }
  void* table = nullptr;
  HI_PJ_TRY(qkv_static_scratch(&table));
  // the table is rewritten for tokens [0, chunk_len) by every call that rotates: nothing to clear
  return qkv_rope_impl(stream, x_dev, w_qkv_dev, d_model, n_q_heads, n_kv_heads, chunk_len, past_len, rope_theta,
                       out_fp32, q_out_dev, k_out_dev, v_out_dev, table, q_scale);
}

extern "C" hi_status hi_out_proj(void* stream, const void* attn_dev, const void* w_o_dev, int32_t n_q_heads,
                                 int32_t d_model, int32_t chunk_len, int32_t out_fp32, void* y_out_dev) {
  if (!attn_dev || !w_o_dev || !y_out_dev) { set_last_error("output projection: null buffer"); return HI_ERR_ARG; }
  if (!pj_aligned16(attn_dev) || !pj_aligned16(w_o_dev) || !pj_aligned16(y_out_dev)) {
    set_last_error("output projection: buffers must be 16-byte aligned");
    return HI_ERR_ARG;
  }
  if (n_q_heads < 1 || d_model < 1 || chunk_len < 1 || (out_fp32 != 0 && out_fp32 != 1)) {
    set_last_error("output projection: bad shape");
    return HI_ERR_ARG;
  }
  const int64_t K = (int64_t)n_q_heads * kHeadDim;
  if ((int64_t)d_model * K * 2 >= (1LL << 32) || (int64_t)chunk_len * kRowBytes >= (1LL << 32)) {
    set_last_error("output projection: each operand must be smaller than 4 GiB");
    return HI_ERR_UNSUPPORTED;
  }
  if (chunk_len == 1) {                      // one token: the head-major output is the concatenation itself
    GemvArgs g = {};
    g.w = (const uint16_t*)w_o_dev; g.x = (const uint16_t*)attn_dev;
    g.rows = d_model; g.K = (int)K;
    g.mode = kPjOut; g.out_fp32 = out_fp32;
    g.log2_theta = -1.0;
    g.y = y_out_dev;
    return gemv_launch(stream, g);
  }
  ProjArgs p = {};
  p.a = (const char*)w_o_dev; p.b = (const char*)attn_dev;
  p.a_rows = d_model; p.b_rows = chunk_len;
  p.a_stride = (uint32_t)K * 2; p.b_stride = kRowBytes;
  p.b_head_stride = (int64_t)chunk_len * kRowBytes;
  p.K = (int)K;
  p.out_fp32 = out_fp32;
  p.y = y_out_dev; p.y_stride = d_model;
  if (chunk_len <= kPfwMaxTokens) return pj_few_launch<kPjOut>(stream, p, 0, RopeFreqs(), 0);
  return pj_launch(stream, p, kPjOut, RopeChunk(), nullptr);
}
