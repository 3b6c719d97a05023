// Device-side building blocks shared by the prefill and decode kernels (gfx950 only).
//
// K/V tiles travel HBM -> LDS with direct-to-LDS 128-bit loads (no VGPR staging).  The hardware writes lane i's
// 16 bytes at (uniform LDS base) + 16*i, so the LDS image is "lane order"; bank conflicts of the later MFMA
// operand reads are avoided by choosing WHICH global 16-byte chunk each lane fetches: LDS chunk position p of
// row r holds global chunk p ^ swz(r).
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <cstdint>

namespace hi {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(1))) const char glb_char;

constexpr float kNegBig = -1.0e30f;   // finite stand-in for -inf: exp2 of (kNegBig - m) * c underflows to 0

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// 16 bytes per lane, global -> LDS at lds_uniform + 16 * lane (M0 carries the wave-uniform LDS byte address).
// Issued as opaque assembly on purpose: the compiler then keeps no record of an asynchronous LDS write, so it
// never guards later LDS reads with a full vmcnt(0) drain; the kernels place their own `s_waitcnt vmcnt(N)`
// before touching a tile, which is what lets several tiles stay in flight.  M0 is written without being declared
// (the compiler rejects it as a clobber); nothing else in these kernels uses M0: no dynamic register indexing,
// no compiler-issued LDS-DMA.
//
// Addressed as (64-bit scalar base) + (32-bit per-lane byte offset): no vector ALU work per load.  Non-temporal: the decode kernel
// reads every K/V byte exactly once; keeping the stream from displacing the L2's contents measured 5.9 -> 6.6 TB/s over a million rows.
__device__ __forceinline__ void g2lds16_s_stream(const char* sbase, uint32_t voff, uint32_t lds_uniform_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
               :
               : "s"(lds_uniform_addr), "v"(voff), "s"(sbase)
               : "memory");
}

// Same without the hint, and with an immediate.
// The instruction's immediate offset is added to the global address and to the LDS address alike.
template <int IMM>
__device__ __forceinline__ void g2lds16_s(const char* sbase, uint32_t voff, uint32_t lds_uniform_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
               :
               : "s"(lds_uniform_addr), "v"(voff), "s"(sbase), "n"(IMM)
               : "memory");
}

// The same in two steps, so that an instruction in between (an MFMA) covers the wait state that the load needs behind a write of M0.
__device__ __forceinline__ void set_m0(uint32_t lds_uniform_addr) { asm volatile("s_mov_b32 m0, %0" : : "s"(lds_uniform_addr) : "memory"); }
__device__ __forceinline__ void g2lds16_m0(const char* sbase, uint32_t voff) {
  asm volatile("global_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(sbase) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ bf16x8 lds_read16(lds_char* p) {
  return *(__attribute__((address_space(3))) bf16x8*)p;
}

// LDS transpose read: within each group of 16 lanes, lane s supplies the address of 4 consecutive bf16 (one
// row of a 4-row x 16-column block: row s/4, columns 4*(s%4)..+3); lane L receives column L of the 4 rows.
__device__ __forceinline__ bf16x4 lds_read_tr8(lds_char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)p);
}

// Sums and maxima over lanes without a trip through LDS (over 100 cycles a step with __shfl_xor, about 10 here): halves and rows of
// 16 lanes change places inside the register file, and within a row of 16 the other operand is a rotation.  The order is that of
// a butterfly from lane ^ 32 down to lane ^ 1 (a rotation by OFF is lane ^ OFF where the values repeat every 2 OFF lanes).
template <int OFF>
__device__ __forceinline__ float row_ror(float x) {
  const int u = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(u, u, 0x120 + OFF, 0xf, 0xf, false));
}
template <class Op>
__device__ __forceinline__ float over_rows16(float x, Op op) {          // lanes ^ 16 and ^ 32
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
template <class Op>
__device__ __forceinline__ float over_wave(float x, Op op) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(s[0]), __uint_as_float(s[1]));
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  x = op(x, row_ror<8>(x));
  x = op(x, row_ror<4>(x));
  x = op(x, row_ror<2>(x));
  return op(x, row_ror<1>(x));
}
__device__ __forceinline__ float op_add(float a, float b) { return a + b; }
__device__ __forceinline__ float op_max(float a, float b) { return fmaxf(a, b); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even fp32 -> bf16 bits (finite inputs)
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// two floats to two bf16 in a word, round-to-nearest-even: one instruction, where the integer form takes four per value
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  return __builtin_bit_cast(uint32_t, (bf16x2){(__bf16)lo, (__bf16)hi});
}

// A launch, and an event (hipEvent_t, may be null) that marks its end.  The event is the launch's own completion signal: recorded
// behind the launch it is a packet of its own, which holds the next kernel back by 2.8 us and costs the host 0.5 us more
// (kernels of 3 us back to back: 7.8 us each with a record, 5.0 without or with the signal).  Not for streams being captured.
// The arguments convert to the kernel's parameters as in a call.
template <class T> struct AsGiven { using type = T; };
template <class... P>
inline void launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds, void* stream, void* done,
                          typename AsGiven<P>::type... args) {
  if (done) hipExtLaunchKernelGGL(kernel, grid, block, lds, (hipStream_t)stream, nullptr, (hipEvent_t)done, 0, args...);
  else hipLaunchKernelGGL(kernel, grid, block, lds, (hipStream_t)stream, args...);
}

}  // namespace hi
