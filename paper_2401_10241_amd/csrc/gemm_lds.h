// What the bf16 GEMM kernels share between global memory and the matrix cores: direct-to-LDS loads, the wait for them
// and the fragment reads of the two LDS tile layouts (gemm_mfma.hip describes both).
#pragma once
#include "zb_common.h"

namespace zb {
namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// s_waitcnt immediate that waits for vmcnt <= n and nothing else (gfx9 encoding)
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// 16 bytes per lane to consecutive LDS addresses from s on (one 1 KB run per wave)
__device__ __forceinline__ void dma16(const void* g, bf16_t* s) {
  __builtin_amdgcn_global_load_lds((gptr_t)g, (lptr_t)s, 16, 0, 0);
}

// the same with an address that is a part common to the wave plus a byte offset per lane
__device__ __forceinline__ void dma16_at(const bf16_t* base, unsigned lane_off, bf16_t* s) {
  typedef const __attribute__((address_space(1))) char* cptr;
  cptr p = (cptr)(gptr_t)base;
  asm volatile("" : "+s"(p));  // keeps the common part in scalar registers
  __builtin_amdgcn_global_load_lds((gptr_t)(p + (size_t)lane_off), (lptr_t)s, 16, 0, 0);
}

// Operands of v_mfma_f32_16x16x32_bf16 are 16 rows of 32 k: lane l holds row (l & 15), k = 8 * (l >> 4)
// and the seven after it.  A [k][R] tile is read 32 bytes from each of eight k-lines (0-3 and 8-11, then 4-7 and 12-15,
// then 16 more) by half a wave at a time; its swizzle puts those in different eighths of the banks (R = 64: a line is half
// of the banks, so k & 1 already separates two).
template <int R> __device__ __forceinline__ int swz16_tr(int k) {
  return R >= 128 ? ((k & 3) | ((k >> 1) & 4)) << 1 : (((k >> 1) & 1) | ((k >> 2) & 2)) << 1;
}
// rows rb..rb+15, k = k0 .. k0+31 of a [k][R] tile
template <int R> __device__ __forceinline__ bf16x8 frag16_tr(const bf16_t* __restrict__ s, int rb, int k0, int lane) {
  const int a = lane & 15;
  const int row = rb + ((a & 3) << 2);
  const int k = k0 + ((lane >> 4) << 3) + (a >> 2);
  typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
  const bf16_t* p0 = s + k * R + ((((row >> 3) ^ swz16_tr<R>(k)) << 3) | (row & 7));
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p0));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p0 + 4 * R));  // k + 4: same swizzle
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// rows rb..rb+15, k = kk*32 .. kk*32+31 of a [R][64] tile
__device__ __forceinline__ bf16x8 frag16_rows(const bf16_t* __restrict__ s, int rb, int kk, int lane) {
  const int r = rb + (lane & 15);
  const int chunk = kk * 4 + (lane >> 4);
  return *reinterpret_cast<const bf16x8*>(s + r * 64 + ((chunk ^ ((r >> 1) & 7)) << 3));
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace
}  // namespace zb
