// Per-element GEMM epilogues shared by the generic and the MFMA GEMM kernels.
#pragma once
#include "zb_common.h"

namespace zb {

struct EpiParams {
  int mode;
  int N;  // row stride of the outputs, aux and outf (elements)
  void* out0;
  void* out1;
  float* outf;
  const float* bias;
  const void* aux;
};

__host__ inline EpiParams make_epi(const GemmArgs& g) {
  EpiParams e;
  e.mode = g.epilogue; e.N = g.N; e.out0 = g.out0; e.out1 = g.out1; e.outf = g.outf; e.bias = g.bias; e.aux = g.aux;
  return e;
}

// one output element (m, n) with fp32 accumulator value acc
template <typename T, int MODE>
__device__ __forceinline__ void epilogue_one(const EpiParams& e, int m, int n, float acc) {
  const size_t idx = (size_t)m * e.N + n;
  if (MODE == EPI_STORE) {
    ((T*)e.out0)[idx] = from_f32<T>(acc);
  } else if (MODE == EPI_BIAS) {
    ((T*)e.out0)[idx] = from_f32<T>(acc + e.bias[n]);
  } else if (MODE == EPI_BIAS_RESID) {
    ((T*)e.out0)[idx] = from_f32<T>(acc + e.bias[n] + to_f32(((const T*)e.aux)[idx]));
  } else if (MODE == EPI_BIAS_GELU) {
    const float f = acc + e.bias[n];
    ((T*)e.out0)[idx] = from_f32<T>(f);
    ((T*)e.out1)[idx] = from_f32<T>(gelu<T>(f));
  } else if (MODE == EPI_DGELU) {
    ((T*)e.out0)[idx] = from_f32<T>(acc * gelu_grad<T>(to_f32(((const T*)e.aux)[idx])));
  } else {  // EPI_ACCUM_F32
    e.outf[idx] += acc;
  }
}

// Two accumulators of v_mfma_f32_16x16x32_bf16 side by side (columns 0-15 and 16-31 of a 16 x 32 block; lane l holds
// column l & 15 and rows 4 (l >> 4) .. + 3 of each) -> column l & 31 and rows 8 (l >> 5) .. + 7, so that a wave's memory
// access covers 128 bytes of two rows and not 64 of four (32 of sixteen with the block transposed: a W pass over 256 tokens
// of hidden 1024 took 65 us so, 52 like this).  The exchange is its own inverse.
typedef float f32x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ void swap_rows16(float* x, float* y) {  // lanes 16-31 and 48-63 of x with 0-15 and 32-47 of y
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, *x), __builtin_bit_cast(unsigned, *y), false, false);
  const unsigned lo = r[0], hi = r[1];
  *x = __builtin_bit_cast(float, lo);
  *y = __builtin_bit_cast(float, hi);
}
__device__ __forceinline__ f32x8 rows8(const f32x4& a, const f32x4& b) {
  f32x8 c;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    float x = a[v], y = b[v];
    swap_rows16(&x, &y);
    c[v] = x;
    c[4 + v] = y;
  }
  return c;
}
__device__ __forceinline__ void from_rows8(const f32x8& c, f32x4* a, f32x4* b) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    float x = c[v], y = c[4 + v];
    swap_rows16(&x, &y);
    (*a)[v] = x;
    (*b)[v] = y;
  }
}

// this lane's offset (in elements) from the first element of such a 16 x 32 block with rows ld apart
__device__ __forceinline__ unsigned rows8_lane_off(int ld, int lane) { return (unsigned)((lane >> 5) * 8 * ld + (lane & 31)); }
// element off of an array whose address is the same for the whole wave: kept in scalar registers, the offset in one vector
// register, so that an access needs no vector arithmetic
template <typename T> __device__ __forceinline__ __attribute__((address_space(1))) T* at_lane(T* base, unsigned off) {
  typedef __attribute__((address_space(1))) T* gptr;
  typedef __attribute__((address_space(1))) const char* cptr;
  gptr p = (gptr)base;
  asm volatile("" : "+s"(p));
  return (gptr)(__attribute__((address_space(1))) char*)((cptr)p + (size_t)(unsigned)(off * (unsigned)sizeof(T)));
}

// The 16 MT x 16 NT block at (m0, n0) (both the same for the whole wave: the addresses are scalar but for one lane offset).
// All reads of 16 rows are issued before any of their writes, so they overlap instead of each waiting for a store.
// (The fp32 accumulate of a wgrad GEMM is not an epilogue here: its kernels start the accumulators from C.)
template <int MODE, int MT, int NT>
__device__ __forceinline__ void epilogue_wave(const EpiParams& e, int m0, int n0, int lane, const f32x4 (&acc)[MT][NT]) {
  const unsigned off = rows8_lane_off(e.N, lane);
  float b[NT / 2];
#pragma unroll
  for (int q = 0; q < NT / 2; ++q)
    b[q] = MODE == EPI_BIAS || MODE == EPI_BIAS_RESID || MODE == EPI_BIAS_GELU ? e.bias[n0 + q * 32 + (lane & 31)] : 0.f;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const size_t row = (size_t)(m0 + i * 16) * e.N + n0;
    float a[NT / 2][8];
    if (MODE == EPI_BIAS_RESID || MODE == EPI_DGELU) {
#pragma unroll
      for (int q = 0; q < NT / 2; ++q)
#pragma unroll
        for (int v = 0; v < 8; ++v) a[q][v] = to_f32(*at_lane((const bf16_t*)e.aux + row + (size_t)v * e.N + q * 32, off));
    }
#pragma unroll
    for (int q = 0; q < NT / 2; ++q) {
      const f32x8 c = rows8(acc[i][2 * q], acc[i][2 * q + 1]);
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const size_t at = row + (size_t)v * e.N + q * 32;
        const float f = c[v] + b[q];
        if (MODE == EPI_PARTIAL) *at_lane(e.outf + at, off) = c[v];  // e.outf already points at this K slice's [M,N] plane
        else if (MODE == EPI_DGELU) *at_lane((bf16_t*)e.out0 + at, off) = (bf16_t)(c[v] * gelu_grad<bf16_t>(a[q][v]));
        else *at_lane((bf16_t*)e.out0 + at, off) = (bf16_t)(MODE == EPI_BIAS_RESID ? f + a[q][v] : MODE == EPI_STORE ? c[v] : f);
        if (MODE == EPI_BIAS_GELU) *at_lane((bf16_t*)e.out1 + at, off) = (bf16_t)gelu<bf16_t>(f);
      }
    }
  }
}

}  // namespace zb
