// Causal attention row by row on the vector ALUs, one wavefront per row, head sizes up to 128: the exact path of the
// matrix-core kernels that take any sequence length.
//
// A matrix product multiplies masked entries too, and a probability that is exactly zero times an infinity or NaN is NaN:
// a later token's V would reach the queries before it that share its tile (an earlier token's dO the keys behind it).
// So the kernels test what they are about to store and take rows that are not finite from here, where masked entries are
// skipped.  On finite data this costs the test only (128 tokens of 4 fp32 heads: the iteration 893 -> 900 us).  Rows whose
// softmax itself is NaN (masked scores have no part in its sum) are not taken again, so data full of NaN costs little more; one
// such token among 777 of 16 heads costs 2.6 ms in the forward, once.
#pragma once
#include "zb_common.h"

namespace zb {

// What a softmax subtracts from the scores whose maximum is m: nothing if there is none but -infinity so far (weights of 0)
__device__ __forceinline__ float softmax_ref(float m) { return m == -INFINITY ? 0.f : m; }

template <typename T> __device__ __forceinline__ float row_dot(const T* __restrict__ x, const T* __restrict__ y, int d) {
  float t = 0.f;
#pragma unroll 8
  for (int e = 0; e < d; ++e) t = fmaf(to_f32(x[e]), to_f32(y[e]), t);
  return t;
}
// acc[c] += weight of row r * column lane + 64 c of it, for the n rows from p on; lane r holds row r's weight
template <typename T>
__device__ __forceinline__ void row_add(float (&acc)[2], float w, const T* __restrict__ p, long ld, int n, int d, int lane) {
  for (int r = 0; r < n; ++r) {
    const float wr = __shfl(w, r, 64);
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (lane + 64 * c < d) acc[c] = fmaf(wr, to_f32(p[r * ld + lane + 64 * c]), acc[c]);
  }
}
template <typename T> __device__ __forceinline__ void row_store(T* __restrict__ p, const float (&acc)[2], float f, int d, int lane) {
#pragma unroll
  for (int c = 0; c < 2; ++c)
    if (lane + 64 * c < d) p[lane + 64 * c] = from_f32<T>(acc[c] * f);
}

template <typename T>
__device__ __forceinline__ void attn_row_fwd(int i, int head, int bi, const T* __restrict__ qkv, T* __restrict__ out,
                                             float* __restrict__ lse, int s, int a, int d, float scale) {
  const int h = a * d, lane = threadIdx.x & 63;
  const long ld = 3L * h, tok0 = (long)bi * s;
  const T* base = qkv + tok0 * ld + head * d;
  float m = -INFINITY, l = 0.f, o[2] = {0.f, 0.f};
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const bool in = j0 + lane <= i;
    const float sc = row_dot(base + i * ld, base + h + min(j0 + lane, i) * ld, d) * scale;
    const float m_new = fmaxf(m, wave_max(in ? sc : -INFINITY));
    const float ref = softmax_ref(m_new), p = in ? expf(sc - ref) : 0.f, alpha = expf(m - ref);
    l = l * alpha + wave_sum(p);
    o[0] *= alpha;
    o[1] *= alpha;
    m = m_new;
    row_add(o, p, base + 2 * h + j0 * ld, ld, min(64, i + 1 - j0), d, lane);
  }
  row_store(out + (tok0 + i) * h + head * d, o, 1.0f / l, d, lane);
  if (lane == 0) lse[((long)bi * a + head) * s + i] = m + logf(l);
}

template <typename T>
__device__ __forceinline__ void attn_row_dq(int i, int head, int bi, const T* __restrict__ qkv, const T* __restrict__ o,
                                            const T* __restrict__ dout, const float* __restrict__ lse, T* __restrict__ dqkv,
                                            int s, int a, int d, float scale) {
  const int h = a * d, lane = threadIdx.x & 63;
  const long ld = 3L * h, tok0 = (long)bi * s;
  const T* base = qkv + tok0 * ld + head * d;
  const T* dorow = dout + (tok0 + i) * h + head * d;
  const float D = row_dot(dorow, o + (tok0 + i) * h + head * d, d), li = lse[((long)bi * a + head) * s + i];
  float dq[2] = {0.f, 0.f};
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const T* k = base + h + min(j0 + lane, i) * ld;
    const float p = expf(row_dot(base + i * ld, k, d) * scale - li);
    row_add(dq, p * (row_dot(dorow, k + h, d) - D), base + h + j0 * ld, ld, min(64, i + 1 - j0), d, lane);
  }
  row_store(dqkv + (tok0 + i) * ld + head * d, dq, scale, d, lane);
}

template <typename T>
__device__ __forceinline__ void attn_row_dkv(int j, int head, int bi, const T* __restrict__ qkv, const T* __restrict__ o,
                                             const T* __restrict__ dout, const float* __restrict__ lse, T* __restrict__ dqkv,
                                             int s, int a, int d, float scale) {
  const int h = a * d, lane = threadIdx.x & 63;
  const long ld = 3L * h, tok0 = (long)bi * s;
  const T* base = qkv + tok0 * ld + head * d;
  const T* k = base + h + j * ld;
  const T* dobase = dout + tok0 * h + head * d;
  float dk[2] = {0.f, 0.f}, dv[2] = {0.f, 0.f};
  bool lost = false;  // a query without a softmax, or an output gradient without a number: every entry here is NaN
  for (int i = j + lane; i < s && !lost; i += 64) {
    lost = true;
    for (int e = 0; e < d && lost; ++e) lost = isnan(to_f32(dobase[(long)i * h + e]));
    lost = lost || isnan(lse[((long)bi * a + head) * s + i]);
  }
  if (__any(lost)) dk[0] = dk[1] = dv[0] = dv[1] = NAN;
  else for (int i0 = j; i0 < s; i0 += 64) {
    const int i = min(i0 + lane, s - 1), n = min(64, s - i0);
    const float p = expf(row_dot(base + i * ld, k, d) * scale - lse[((long)bi * a + head) * s + i]);
    const T* dorow = dobase + (long)i * h;
    const float D = row_dot(dorow, o + (tok0 + i) * h + head * d, d);
    row_add(dk, p * (row_dot(dorow, k + h, d) - D), base + i0 * ld, ld, n, d, lane);
    row_add(dv, p, dobase + (long)i0 * h, h, n, d, lane);
  }
  T* op = dqkv + (tok0 + j) * ld + h + head * d;
  row_store(op, dk, scale, d, lane);
  row_store(op + h, dv, 1.0f, d, lane);
}

}  // namespace zb
