// K2 (split-KV decode attention) and K3 (log-sum-exp combine) for gfx950.
//
// Algorithm 1, decode phase: one new query row per query head attends over the head's whole K/V history
// (Eq. 3 / Eq. 9).  The work is bandwidth bound (Section 5: decode intensity is O(1) flop per byte), so the
// kernel is organised around the memory pipeline: every wavefront streams its share of the 16-row
// K/V blocks through a private 4-stage LDS ring filled by direct-to-LDS 128-bit loads (24 KiB in flight per
// wavefront, nothing staged in VGPRs, no workgroup barriers in the loop).  The G <= 16 query heads ride along
// as the 16 columns of small MFMA tiles (S^T = K Q^T, O^T += V^T P^T), which keeps the vector ALU nearly idle;
// the matrix unit runs at a few percent of its rate and is not the bound.
#include <mutex>
#include <type_traits>
#include "hi_device.h"
#include "hi_internal.h"

namespace hi {

constexpr int kDecStages = 4;
constexpr int kDecBlockRows = 16;
constexpr int kDecTileBytes = kDecBlockRows * kRowBytes;         // 4 KiB of K (or V)
constexpr int kDecStageBytes = 2 * kDecTileBytes;                // K tile then V tile
constexpr int kDecWaveLds = kDecStages * kDecStageBytes;         // 32 KiB per wavefront
constexpr int kDecLdsBytes = 4 * kDecWaveLds;                    // 128 KiB per workgroup

// The 8 loads (4 K + 4 V) of a block as uniform base + lane offset: LDS chunk position p of row r holds chunk p ^ (r % 16) of a
// K row, p ^ 2 (r % 8) of a V row.  ok / ov: the lane's offset in the first four rows; load i lies i * 1024 bytes further on with the
// swizzle bits of its rows, which are bits of their own.  A block that ends beyond row n - 1 takes per-lane row numbers (rows past
// the end re-read row n - 1 and are masked later).
struct DecLane { uint32_t ok, ov; };
__device__ __forceinline__ DecLane dec_lane(int lane) {
  const int r = lane >> 4, p = lane & 15;       // row within the 4-row group of one load instruction, LDS chunk position
  return {(uint32_t)(r * kRowBytes + ((p ^ r) << 4)), (uint32_t)(r * kRowBytes + ((p ^ (2 * r)) << 4))};
}
__device__ __forceinline__ void dec_issue_block(const char* __restrict__ k, const char* __restrict__ v, int blk, int64_t n,
                                                uint32_t stage, int lane, const DecLane& dl) {
  const int64_t at = (int64_t)blk * kDecTileBytes;
  const int64_t left = n - (int64_t)blk * kDecBlockRows;
  if (left >= kDecBlockRows) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      g2lds16_s_stream(k + at, dl.ok ^ (uint32_t)(i * 1024 + i * 64), stage + i * 1024);
      g2lds16_s_stream(v + at, dl.ov ^ (uint32_t)(i * 1024 + (i & 1) * 128), stage + kDecTileBytes + i * 1024);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * i + (lane >> 4), p = lane & 15, row = r < (int)left ? r : (int)left - 1;
      g2lds16_s_stream(k + at, (uint32_t)(row * kRowBytes + ((p ^ r) << 4)), stage + i * 1024);
      g2lds16_s_stream(v + at, (uint32_t)(row * kRowBytes + ((p ^ ((r & 7) << 1)) << 4)), stage + kDecTileBytes + i * 1024);
    }
  }
}

struct NoLens {};        // every head of the launch has the same number of rows
template <class Lens> constexpr bool kRagged = std::is_same<Lens, DecodeLens>::value;

// partials that cross workgroups inside one launch: through the point all XCDs agree on, past the L2s
__device__ __forceinline__ void store_shared2(float* p, float2 x) {   // 8-byte aligned
  __hip_atomic_store((uint64_t*)p, (uint64_t)__float_as_uint(x.x) | ((uint64_t)__float_as_uint(x.y) << 32), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_shared2(const float* p) {      // 8-byte aligned
  const uint64_t v = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

// x of lane p (a constant)
__device__ __forceinline__ float from_lane(float x, int p) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), p)); }

// What decode_combine_kernel does, for all G query heads of one KV head, by the workgroup that finished its partial last, in
// that kernel's order of operations (at most one partition per lane there): the same bits, so that a captured step, which
// takes two launches, agrees with an eager one.
// Bound by the latency of its loads (the partials come from beyond the L2), so all of them are asked for at once: that is
// why a launch has to have few partitions for it.  lds: 2 * 8 * kTailMaxParts floats; k_lo, k_hi: dims lane and lane + 64 of
// the token's own K row; v2: dims 2 lane and 2 lane + 1 of its V row.
__device__ __forceinline__ void decode_tail(int kv, const uint16_t* q, int G, const float* part, int n_part, const DecodeTail& tl,
                                            int64_t append_off, float c, float* lds, uint16_t k_lo, uint16_t k_hi, uint32_t v2) {
#pragma clang fp contract(off)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float* w = lds;                                  // [n_part][G] maxima of the partials
  float* sum = lds + 8 * kTailMaxParts;            // [n_part][G] sums
  const int64_t part_pitch = (int64_t)G * kPartialFloats;
  const int dim = 2 * lane;                        // a wavefront takes query heads wave and wave + 4, a lane two dims
  uint16_t q_lo[2] = {0, 0}, q_hi[2] = {0, 0};     // asked for first: the scores are formed while the partials arrive
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int g = wave + 4 * h;
    if (g < G) {
      q_lo[h] = q[g * kHeadDim + lane];
      q_hi[h] = q[g * kHeadDim + 64 + lane];
    }
  }
  float2 ml = make_float2(0.f, 0.f);
  if (tid < n_part * G) ml = load_shared2(part + (int64_t)tid * kPartialFloats + kHeadDim);
  float2 o[2][kTailMaxParts];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int g = wave + 4 * h;
    if (g < G) {
#pragma unroll
      for (int p = 0; p < kTailMaxParts; ++p) {    // (past the last partial: zeros, as the combine kernel adds there)
        o[h][p] = make_float2(0.f, 0.f);
        if (p < n_part) o[h][p] = load_shared2(part + p * part_pitch + g * kPartialFloats + dim);
      }
    }
  }
  if (tl.k_append != nullptr && wave == 0) {
    uint16_t* const k_row = (uint16_t*)((char*)tl.k_append + append_off);
    k_row[lane] = k_lo;
    k_row[lane + 64] = k_hi;
    *(uint32_t*)((char*)tl.v_append + append_off + 2 * dim) = v2;
  }
  // (the products of two bf16 numbers are exact: these are the combine kernel's dot products, fused or not)
  float score[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    score[h] = bf16_bits_to_float(q_lo[h]) * bf16_bits_to_float(k_lo) + bf16_bits_to_float(q_hi[h]) * bf16_bits_to_float(k_hi);
    if (4 * h < G) score[h] = over_wave(score[h], op_add);
  }
  if (tid < n_part * G) {
    w[tid] = ml.x;
    sum[tid] = ml.y;
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int g = wave + 4 * h;
    if (g >= G) break;
    const float d = score[h];
    const float m = lane < n_part ? w[lane * G + g] : kNegBig;
    const float mx = over_wave(fmaxf(d, m), op_max);
    const float wp = lane < n_part ? fast_exp2((m - mx) * c) : 0.f;
    const float lp = lane < n_part ? wp * sum[lane * G + g] : 0.f;
    const float p_new = fast_exp2((d - mx) * c);
    float2 acc = make_float2(0.f, 0.f);
    float total = 0.f;
#pragma unroll
    for (int p = 0; p < kTailMaxParts; ++p) {
      const float x = from_lane(wp, p), l = from_lane(lp, p);
      acc.x += x * o[h][p].x;
      acc.y += x * o[h][p].y;
      total += l;
    }
    acc.x = __builtin_fmaf(p_new, __uint_as_float(v2 << 16), acc.x);
    acc.y = __builtin_fmaf(p_new, __uint_as_float(v2 & 0xFFFF0000u), acc.y);
    total += p_new;
    acc.x /= total;
    acc.y /= total;
    const int64_t at = ((int64_t)kv * G + g) * kHeadDim + dim;
    if (tl.out_fp32) *(float2*)((float*)tl.out + at) = acc;
    else *(uint32_t*)((uint16_t*)tl.out + at) = (uint32_t)float_to_bf16_bits(acc.x) | ((uint32_t)float_to_bf16_bits(acc.y) << 16);
  }
}

// Lens = DecodeLens: the heads of the launch have their own numbers of rows (sequences of different lengths served as
// more KV heads), and partitions in proportion or the same number each (see decode_cut).
// TAIL: this launch writes all partials of its heads, few enough of them (kTailMaxParts) for one workgroup to combine: the
// workgroup of a head that finishes last does so, and no combine launch follows.
// Over a short history this is a chain of latencies in which every instruction of a lone wavefront counts 7 cycles.  By time stamps
// of 8 heads of 1000 rows: arguments 0.45 us, addresses and loads out 0.5, rows and queries here 1.2, the block 0.6, wavefronts merged
// 0.5, partials out and counted 0.9, combined 1.7.  With 64-bit divisions and row addresses per lane, sums and maxima by __shfl
// (an LDS round trip a step) and accumulators in AGPRs (64 moves a block, as the compiler has it for a kernel that may use more than 256
// registers) it was 7.4 us instead of 6.1; a call, back to back with others of its kind: 8 heads of 60 / 1000 / 6003 / 20 thousand /
// 130 thousand rows 8.2 / 9.3 / 13.8 / 21.2 / 86 -> 6.9 / 7.5 / 11.9 / 19.4 / 83.6 us, a million 621 -> 616.
template <class Lens, bool TAIL>
__global__ __launch_bounds__(256, 2) void decode_partial_kernel(const uint16_t* __restrict__ q, int G,
                                                             const char* __restrict__ k, const char* __restrict__ v,
                                                             int64_t n, float* partials, int part0,
                                                             float c, int64_t kv_head_stride,
                                                             int64_t part_head_stride, int64_t skip_row,
                                                             DecodeTail tail, Lens lens) {
  // group launches: blockIdx.y is the head; partitions in proportion (rows_per_wg > 0) lie one head after the other along x,
  // so that the hardware deals the workgroups evenly to the XCDs
  int head_i = blockIdx.y, part = blockIdx.x, n_part = gridDim.x;
  if constexpr (kRagged<Lens>) {
    if (lens.rows_per_wg > 0) {
      // The head of this workgroup, eight by eight.  The cache lines of all that is looked up are asked for at once, so that the
      // later look-ups do not wait for the argument memory again (all in all it costs about 0.9 us: see decode_cut).
      static_assert(kDecodeMaxRagged == 64, "eight groups of eight");
      uint32_t lines = lens.first[0] ^ lens.first[32];
#pragma unroll
      for (int j = 0; j < kDecodeMaxRagged; j += 16) lines ^= lens.n[j];
      asm volatile("" : : "s"(lines));
      int oct = 0;
#pragma unroll
      for (int j = 1; j < 8; ++j) oct += blockIdx.x >= lens.first[8 * j] ? 1 : 0;
      oct = __builtin_amdgcn_readfirstlane(oct);
      head_i = 8 * oct;
#pragma unroll
      for (int j = 1; j < 8; ++j) head_i += blockIdx.x >= lens.first[8 * oct + j] ? 1 : 0;
      head_i = __builtin_amdgcn_readfirstlane(head_i);
      part = (int)blockIdx.x - lens.first[head_i];
      n_part = decode_parts(lens.n[head_i], lens.rows_per_wg);
    }
    n = lens.n[head_i];
  }
  q += (int64_t)head_i * G * kHeadDim;
  k += head_i * kv_head_stride;
  v += head_i * kv_head_stride;
  partials += head_i * part_head_stride;
  extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
  const int lane = lane_id();
  const int wave = wave_id();
  const uint32_t wlds = (uint32_t)(uintptr_t)(lds_char*)lds_raw + wave * kDecWaveLds;

  const int head = lane & 15;
  const int g4 = lane >> 4;

  // 16-row blocks are dealt round-robin to the wavefronts of the grid, so at any moment the whole chip reads one
  // compact window of the K and V streams (friendlier to HBM pages and TLBs than one far-apart range per wave)
  const int n_blocks = (int)((n + kDecBlockRows - 1) / kDecBlockRows);       // (an HBM-resident head has far fewer than 2^31)
  const int n_waves = n_part * 4;
  const int wid = part * 4 + wave;
  const int skip_blk = skip_row >= 0 ? (int)(skip_row / kDecBlockRows) : -1;
  const DecLane dl = dec_lane(lane);

  // prologue: up to three blocks in flight, before the queries are asked for (one wait for both: over a short history
  // two memory latencies in a row were a third of the kernel)
  for (int s = 0; s < kDecStages - 1; ++s)
    if (wid + s * n_waves < n_blocks) dec_issue_block(k, v, wid + s * n_waves, n, wlds + s * kDecStageBytes, lane, dl);

  // Q^T as the B operand of S^T = K Q^T: lane holds q[head][32*kk + 8*g4 .. +7]; heads >= G are zero columns
  bf16x8 qf[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    uint4 raw = make_uint4(0, 0, 0, 0);
    if (head < G) raw = *(const uint4*)(q + head * kHeadDim + 32 * kk + 8 * g4);
    qf[kk] = __builtin_bit_cast(bf16x8, raw);
  }
  // the token's own row, for the tail: asked for now, so that a cold first touch is not a latency of its own there
  uint32_t k_lo = 0, k_hi = 0, v2 = 0;
  if constexpr (TAIL) {
    const uint16_t* const k_row = (const uint16_t*)tail.k_new + head_i * kHeadDim;
    k_lo = k_row[lane];
    k_hi = k_row[lane + 64];
    v2 = *(const uint32_t*)((const uint16_t*)tail.v_new + head_i * kHeadDim + 2 * lane);
  }
  asm volatile("" : "+v"(k_lo), "+v"(k_hi), "+v"(v2));
  // make the compiler wait for these loads here, not inside the loop (a vmcnt(0) there would drain the ring)
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(qf[kk]));

  float m = kNegBig, l = 0.f;
  f32x4 o[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // lane-constant LDS offsets of the operand reads
  const int k_tok = lane & 15;
  const int v_row = 4 * g4 + ((lane & 15) >> 2);
  const int v_sub = lane & 3;      // which 8-byte quarter of the 32-byte column group

  int stage = 0;
  for (int b = wid; b < n_blocks; b += n_waves) {
    const int ahead = b + (kDecStages - 1) * n_waves;
    if (ahead < n_blocks) {
      dec_issue_block(k, v, ahead, n, wlds + ((stage + kDecStages - 1) & (kDecStages - 1)) * kDecStageBytes, lane, dl);
      wait_vmcnt<24>();   // everything but the 3 newest blocks has landed
    } else {
      wait_vmcnt<0>();
    }
    lds_char* kt = (lds_char*)(uintptr_t)(wlds + stage * kDecStageBytes);
    lds_char* vt = kt + kDecTileBytes;
    stage = (stage + 1) & (kDecStages - 1);

    // V^T operands: lane receives dim 16*db + (lane & 15) of rows 4*g4 .. 4*g4+3 (read here, so that their latency passes under the
    // scores)
    bf16x4 vop[8];
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const int chunk = (2 * db + (v_sub >> 1)) ^ ((v_row & 7) << 1);
      vop[db] = lds_read_tr8(vt + v_row * kRowBytes + (chunk << 4) + ((v_sub & 1) << 3));
    }
    f32x4 s = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8 a = lds_read16(kt + k_tok * kRowBytes + (((4 * kk + g4) ^ k_tok) << 4));
      s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[kk], s, 0, 0, 0);
    }
    // register r of lane (g4, head) is the score of row 16*b + 4*g4 + r
    // hidden rows: beyond the end, or the one row a streaming head's token is about to replace
    const bool hides = (int64_t)(b + 1) * kDecBlockRows > n || b == skip_blk;
    if (hides) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = (int64_t)b * kDecBlockRows + 4 * g4 + r;
        if (row >= n || row == skip_row) s[r] = kNegBig;
      }
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = over_rows16(mx, op_max);
    const float m_new = fmaxf(m, mx);
    if (__builtin_amdgcn_ballot_w64(m_new > m) != 0) {
      const float alpha = fast_exp2((m - m_new) * c);
      l *= alpha;
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] *= alpha;
      m = m_new;
    }
    const float mc = m * c;
    float p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = fast_exp2(__builtin_fmaf(s[r], c, -mc));
    if (hides) {   // exactly zero even while nothing visible has been seen (m still at its initial value)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (s[r] == kNegBig) p[r] = 0.f;
    }
    l += (p[0] + p[1]) + (p[2] + p[3]);
    bf16x4 pb;
#pragma unroll
    for (int r = 0; r < 4; ++r) pb[r] = (__bf16)p[r];
    const short4v pbs = __builtin_bit_cast(short4v, pb);
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      o[db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, vop[db]), pbs, o[db], 0, 0, 0);
    }
    asm volatile("" ::: "memory");
  }

  // per-lane-group partial sums -> per-head sums
  l = over_rows16(l, op_add);

  // merge the four wavefronts through LDS (the ring is idle now)
  __syncthreads();
  float* red = (float*)lds_raw;                 // [4 waves][16 heads][130]
  if (head < G) {
    float* mine = red + (wave * 16 + head) * kPartialFloats;
#pragma unroll
    for (int db = 0; db < 8; ++db)
#pragma unroll
      for (int r = 0; r < 4; r += 2) *(float2*)(mine + 16 * db + 4 * g4 + r) = make_float2(o[db][r], o[db][r + 1]);
    if (g4 == 0) *(float2*)(mine + kHeadDim) = make_float2(m, l);
  }
  __syncthreads();
  // a thread takes two dims of a query head; every read of it is asked for at once
  float* dst = partials + (int64_t)(part0 + part) * G * kPartialFloats;
  for (int idx = threadIdx.x; idx < G * kHeadDim / 2; idx += blockDim.x) {
    const int h = idx >> 6, dim = 2 * (idx & 63);
    float2 ml[4], x[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float* src = red + (w * 16 + h) * kPartialFloats;
      ml[w] = *(const float2*)(src + kHeadDim);
      x[w] = *(const float2*)(src + dim);
    }
    float M = kNegBig;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, ml[w].x);
    float2 acc = make_float2(0.f, 0.f);
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float wgt = fast_exp2((ml[w].x - M) * c);
      acc.x += wgt * x[w].x;
      acc.y += wgt * x[w].y;
      L += wgt * ml[w].y;
    }
    auto put = [&](float* p, float2 y) { if (TAIL) store_shared2(p, y); else *(float2*)p = y; };
    put(dst + h * kPartialFloats + dim, acc);
    if (dim == 0) put(dst + h * kPartialFloats + kHeadDim, make_float2(M, L));
  }
  if constexpr (TAIL) {
    // Every wavefront's partials have arrived before the count goes up; the last workgroup of the head resets it.  The
    // partials are written and read by device-scope accesses that no L2 keeps a copy of, so that the wait for the stores,
    // the barrier and the count order them; a release or acquire of everything else would walk the whole L2 once per
    // workgroup (measured: 2 us more at 128 workgroups, 3 at 256).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* flag = (int*)lds_raw;
    if (threadIdx.x == 0) {
      const int before = __hip_atomic_fetch_add(tail.counters + head_i, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int last = before == n_part - 1;
      if (last) __hip_atomic_store(tail.counters + head_i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *flag = last;
    }
    __syncthreads();
    const bool last = *flag != 0;
    __syncthreads();
    if (!last) return;
    int64_t off = head_i * tail.append_head_stride;
    if constexpr (kRagged<Lens>) off += n * kRowBytes;      // (k_append / v_append point at row 0 of the first head)
    decode_tail(head_i, q, G, partials, n_part, tail, off, c, (float*)lds_raw, (uint16_t)k_lo, (uint16_t)k_hi, v2);
  }
}

// K3: out[g][:] = (sum_s O_s w_s + p_new v_new) / (sum_s l_s w_s + p_new),  w_s = 2^{(m_s - M) c},
// p_new = 2^{(q_g . k_new - M) c}, M = max(max_s m_s, q_g . k_new).   grid (G, 8): one query head, 16 dims;
// thread = (one of 16 partition lanes, one dim), several independent loads in flight per thread.
constexpr int kCombDims = 16;
constexpr int kCombLanes = 256 / kCombDims;

template <class Lens>
__global__ __launch_bounds__(256) void decode_combine_kernel(const uint16_t* __restrict__ q, int G,
                                                             const uint16_t* __restrict__ k_new,
                                                             const uint16_t* __restrict__ v_new,
                                                             const float* __restrict__ partials, int n_part,
                                                             void* __restrict__ out, int out_fp32, float c,
                                                             uint16_t* __restrict__ k_append,
                                                             uint16_t* __restrict__ v_append,
                                                             int64_t part_head_stride, int64_t append_head_stride,
                                                             Lens lens) {
  // group launches: blockIdx.z is the head
  if constexpr (kRagged<Lens>)
    if (lens.rows_per_wg > 0 && n_part > 0) n_part = decode_parts(lens.n[blockIdx.z], lens.rows_per_wg);
  q += (int64_t)blockIdx.z * G * kHeadDim;
  k_new += blockIdx.z * kHeadDim;
  v_new += blockIdx.z * kHeadDim;
  partials += blockIdx.z * part_head_stride;
  out = (char*)out + (int64_t)blockIdx.z * G * kHeadDim * (out_fp32 ? 4 : 2);
  if (k_append != nullptr) {
    // (ragged: k_append / v_append point at row 0 of the first head; each head appends at its own length)
    int64_t row_off = 0;
    if constexpr (kRagged<Lens>) row_off = (int64_t)lens.n[blockIdx.z] * kRowBytes;
    k_append = (uint16_t*)((char*)k_append + blockIdx.z * append_head_stride + row_off);
    v_append = (uint16_t*)((char*)v_append + blockIdx.z * append_head_stride + row_off);
  }
  __shared__ float red[4];
  __shared__ float red_o[kCombLanes][kCombDims + 1];
  __shared__ float bc;
  const int g = blockIdx.x;
  const int tid = threadIdx.x;
  const float* base = partials + (int64_t)g * kPartialFloats;
  const int64_t stride = (int64_t)G * kPartialFloats;

  // HBM-resident cache: the token's K/V row is appended here instead of by two tiny device copies
  if (k_append != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && tid < kHeadDim) {
    k_append[tid] = k_new[tid];
    v_append[tid] = v_new[tid];
  }

  // score of the token's own row (first wavefront), and the maximum over all partitions
  float mx = kNegBig;
  for (int p = tid; p < n_part; p += 256) mx = fmaxf(mx, base[p * stride + kHeadDim]);
  if (tid < 64) {
    float d = bf16_bits_to_float(q[g * kHeadDim + tid]) * bf16_bits_to_float(k_new[tid]) +
              bf16_bits_to_float(q[g * kHeadDim + 64 + tid]) * bf16_bits_to_float(k_new[64 + tid]);
    d = over_wave(d, op_add);
    if (tid == 0) bc = d;
  }
  mx = over_wave(mx, op_max);
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  const float s_new = bc;
  const float M = fmaxf(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])), s_new);

  const int pl = tid / kCombDims;
  const int dim = blockIdx.y * kCombDims + (tid % kCombDims);
  float acc = 0.f, L = 0.f;
#pragma unroll 4
  for (int p = pl; p < n_part; p += kCombLanes) {
    const float* src = base + p * stride;
    const float w = fast_exp2((src[kHeadDim] - M) * c);
    acc = __builtin_fmaf(w, src[dim], acc);
    L = __builtin_fmaf(w, src[kHeadDim + 1], L);
  }
  red_o[pl][tid % kCombDims] = acc;
  if ((tid % kCombDims) == 0) red_o[pl][kCombDims] = L;
  __syncthreads();
  if (tid < kCombDims) {
    float a = 0.f, lsum = 0.f;
#pragma unroll
    for (int i = 0; i < kCombLanes; ++i) { a += red_o[i][tid]; lsum += red_o[i][kCombDims]; }
    const float p_new = fast_exp2((s_new - M) * c);
    a = __builtin_fmaf(p_new, bf16_bits_to_float(v_new[dim]), a);
    lsum += p_new;
    const float r = a / lsum;
    if (out_fp32) ((float*)out)[g * kHeadDim + dim] = r;
    else ((uint16_t*)out)[g * kHeadDim + dim] = float_to_bf16_bits(r);
  }
}


// Counters of contexts: a slot each of a built-in array, all zero whenever no launch of their context is in flight.  A slot
// that is given back keeps the event of its context's last unit, which the next owner's stream waits for (no query: one from
// a thread beside a stream capture would break the capture).
constexpr int kTailSlots = 64, kTailDevices = 64;
static __device__ int tail_counters[kTailSlots * kTailMaxHeads];
namespace {
std::mutex tail_mu;
struct TailSlot { bool taken; hipEvent_t busy_until; } tail_slots[kTailSlots];

// the array on the current device (tail_mu held); looking it up takes half a millisecond: once per device
void* tail_array() {
  static void* address[kTailDevices] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kTailDevices) { (void)hipGetLastError(); return nullptr; }
  void*& base = address[dev];
  if (!base && (hipGetSymbolAddress(&base, HIP_SYMBOL(tail_counters)) != hipSuccess || !base)) {
    (void)hipGetLastError();
    base = nullptr;
  }
  return base;
}
}  // namespace

void tail_counters_prepare() {
  std::lock_guard<std::mutex> lock(tail_mu);
  (void)tail_array();
}

int* tail_counters_take(void* stream, int* slot) {
  std::lock_guard<std::mutex> lock(tail_mu);
  void* const base = tail_array();
  if (!base) return nullptr;
  for (int i = 0; i < kTailSlots; ++i) {
    TailSlot& s = tail_slots[i];
    if (s.taken) continue;
    if (s.busy_until) {
      if (hipStreamWaitEvent((hipStream_t)stream, s.busy_until, 0) != hipSuccess) { (void)hipGetLastError(); continue; }
      (void)hipEventDestroy(s.busy_until);
      s.busy_until = nullptr;
    }
    s.taken = true;
    *slot = i;
    return (int*)base + i * kTailMaxHeads;
  }
  return nullptr;
}

void tail_counters_give(int slot, void* busy_until) {
  std::lock_guard<std::mutex> lock(tail_mu);
  tail_slots[slot].busy_until = (hipEvent_t)busy_until;
  tail_slots[slot].taken = false;
}

hi_status launch_decode_partial(void* stream, const void* q, int G, const void* k, const void* v, int64_t n,
                                int n_split, void* partials, int part0, bool q_prescaled, int n_heads,
                                int64_t kv_head_stride, int64_t part_head_stride, int64_t skip_row,
                                const DecodeLens* lens, const DecodeTail* tail, int n_wgs, void* done) {
  if (n <= 0 || n_split <= 0 || n_heads < 1 || (lens && (n_heads > kDecodeMaxRagged || (lens->rows_per_wg > 0 && n_wgs < n_heads)))) { set_last_error("decode partial: empty launch"); return HI_ERR_ARG; }
  if (tail && (part0 != 0 || n_split > kTailMaxParts || n_heads > kTailMaxHeads || !tail->counters)) { set_last_error("decode partial: too many partials to combine in the launch"); return HI_ERR_ARG; }
  static std::once_flag attr_once;      // contexts on different host threads may get here together
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [] {
    const void* kernels[4] = {(const void*)decode_partial_kernel<NoLens, false>, (const void*)decode_partial_kernel<NoLens, true>,
                              (const void*)decode_partial_kernel<DecodeLens, false>, (const void*)decode_partial_kernel<DecodeLens, true>};
    for (int i = 0; i < 4 && attr_err == hipSuccess; ++i)
      attr_err = hipFuncSetAttribute(kernels[i], hipFuncAttributeMaxDynamicSharedMemorySize, kDecLdsBytes);
  });
  if (attr_err != hipSuccess) { set_last_error("hipFuncSetAttribute: %s", hipGetErrorString(attr_err)); return HI_ERR_HIP; }
  auto go = [&](auto kernel, auto lens_arg) {
    launch_kernel(kernel, lens && lens->rows_per_wg > 0 ? dim3(n_wgs) : dim3(n_split, n_heads), dim3(256), kDecLdsBytes, stream,
                  done, (const uint16_t*)q, G, (const char*)k, (const char*)v, n, (float*)partials, part0,
                  softmax_scale_log2(q_prescaled), kv_head_stride, part_head_stride, skip_row, tail ? *tail : DecodeTail(), lens_arg);
  };
  if (lens && tail) go(decode_partial_kernel<DecodeLens, true>, *lens);
  else if (lens) go(decode_partial_kernel<DecodeLens, false>, *lens);
  else if (tail) go(decode_partial_kernel<NoLens, true>, NoLens());
  else go(decode_partial_kernel<NoLens, false>, NoLens());
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error("decode_partial launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

hi_status launch_decode_combine(void* stream, const void* q, int G, const void* k_new, const void* v_new,
                                const void* partials, int n_part, void* out, int out_fp32, void* k_append,
                                void* v_append, bool q_prescaled, int n_heads, int64_t part_head_stride,
                                int64_t append_head_stride, const DecodeLens* lens, void* done) {
  if (lens && n_heads > kDecodeMaxRagged) { set_last_error("decode combine: too many heads of their own length"); return HI_ERR_ARG; }
  auto go = [&](auto kernel, auto lens_arg) {
    launch_kernel(kernel, dim3(G, kHeadDim / kCombDims, n_heads), dim3(256), 0, stream, done, (const uint16_t*)q, G,
                  (const uint16_t*)k_new, (const uint16_t*)v_new, (const float*)partials, n_part, out, out_fp32,
                  softmax_scale_log2(q_prescaled), (uint16_t*)k_append, (uint16_t*)v_append, part_head_stride, append_head_stride,
                  lens_arg);
  };
  if (lens) go(decode_combine_kernel<DecodeLens>, *lens);
  else go(decode_combine_kernel<NoLens>, NoLens());
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_error("decode_combine launch: %s", hipGetErrorString(e)); return HI_ERR_HIP; }
  return HI_OK;
}

}  // namespace hi
