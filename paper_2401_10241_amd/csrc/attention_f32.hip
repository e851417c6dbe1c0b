// Causal attention in fp32 on the matrix cores (v_mfma_f32_32x32x2_f32), forward and backward, head sizes that are
// multiples of 4 up to 128, any sequence length.
//
// A workgroup owns 32 queries (forward, dQ) or 32 keys (dK / dV) of one head; its four waves take the 32-row blocks
// of the other side in turn, each with its own state, and the states are merged through LDS in wave order.  As in
// the bf16 kernels all products are formed so that a lane owns one query (or key):
//   forward  S^T = K Q^T,  O^T += V^T P^T;   dQ  dP^T = V dO^T,  dQ^T += K^T dS^T;   dK/dV  dV^T += dO^T P,  dK^T += Q^T dS
// A 32 x 32 accumulator holds in lane l, element v, row 8 (v/4) + 4 (l>>5) + v%4 and column l&31, and one MFMA
// contracts the two rows that a lane pair holds in element v: P and dS go into the next product as they are, in
// fp32, and the other operand is one float per lane, 32 consecutive columns of a row at a time, from memory.
// Columns past the head size are zeros in the products over them; rows past the end of the sequence are fetched
// from the last row and masked.  Rows whose result is not finite are taken again from attention_rows.h.
//
// What bounds it: latency.  The fp32 stages are small (128 tokens of 4 heads: 512 rows), one wavefront per row
// walked up to 128 dependent steps; here a wave has one 32 x 32 block.  Both halves of the backward are one launch
// and D = rowsum(dO * O) is formed where it is used.  Measured (rocprof, 4 heads of 64, 128 tokens): forward 14.5 -> 11.6 us,
// backward 13.4 + 20.3 -> 16.9 us; the iteration 1.07 -> 0.90 ms.
#include "attention_rows.h"

namespace zb {

template <typename T> hipError_t launch_attention_fwd_mfma(const AttnArgs& a, hipStream_t s, bool* taken);
template <typename T> hipError_t launch_attention_bwd_mfma(const AttnArgs& a, hipStream_t s, bool* taken);

namespace {

constexpr int NW = 4;

template <int D> struct Frag { f32x4 c[D / 32][4]; };  // a row: element 4q + j of chunk i is column 32 i + 8 q + 4 (lane>>5) + j

template <int D> __device__ __forceinline__ void load_row(Frag<D>& f, const float* __restrict__ row, int hi, int d) {
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = i * 32 + q * 8 + hi * 4;
      f.c[i][q] = *reinterpret_cast<const f32x4*>(row + min(e, d - 4));
      if (e >= d) f.c[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}
// 32 x 32 products of rows: out = a b^T
template <int D> __device__ __forceinline__ f32x16 dot_rows(const Frag<D>& a, const Frag<D>& b) {
  f32x16 r;
#pragma unroll
  for (int v = 0; v < 16; ++v) r[v] = 0.f;
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) r = __builtin_amdgcn_mfma_f32_32x32x2f32(a.c[i][q][e], b.c[i][q][e], r, 0, 0, 0);
  return r;
}
template <int D> __device__ __forceinline__ float dot_self(const Frag<D>& a, const Frag<D>& b) {
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) t = fmaf(a.c[i][q][e], b.c[i][q][e], t);
  return t + __shfl_xor(t, 32, 64);
}
// out^T += (rows r0 .. r0+31 of p, columns) * w, w an accumulator whose rows are the same 32 rows; rows >= s: zero
template <int D>
__device__ __forceinline__ void add_rows(f32x16 (&out)[D / 32], const float* __restrict__ p, long ld, int r0, int s, int d,
                                         const f32x16& w, int lane) {
  float x[D / 32][16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = r0 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
    const float* row = p + (long)min(r, s - 1) * ld;
#pragma unroll
    for (int i = 0; i < D / 32; ++i) {
      x[i][v] = row[min(i * 32 + (lane & 31), d - 1)];
      if (r >= s) x[i][v] = 0.f;
    }
  }
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) out[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][v], w[v], out[i], 0, 0, 0);
}
template <int D> __device__ __forceinline__ void clear(f32x16 (&o)[D / 32]) {
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
}

constexpr int P = 65;  // LDS pitch of an accumulator register's 64 lanes
template <int D> constexpr int kState = (D / 32) * 16 * P;
template <int D> __device__ __forceinline__ void put(float* sm, const f32x16 (&o)[D / 32], int wave, int lane) {
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) sm[wave * kState<D> + (i * 16 + v) * P + lane] = o[i][v];
}
// where column e of row r (0..31) of a transposed accumulator lies
__device__ __forceinline__ int at(int r, int e) {
  return ((e >> 5) * 16 + ((e & 31) >> 3) * 4 + (e & 3)) * P + r + ((e >> 2) & 1) * 32;
}
// Rows whose result is not finite (attention_rows.h); cleared before the barrier that precedes the results
__device__ __forceinline__ void clear_flags(int* bad) {
  if (threadIdx.x < 32) bad[threadIdx.x] = 0;
}
// rows [0, min(32, rows)) x d columns = scale * (sum over the waves, in order); ends with a barrier
template <int D>
__device__ __forceinline__ void sum_out(float* sm, const f32x16 (&o)[D / 32], float* __restrict__ out, long ld, int rows, int d,
                                        float scale, int wave, int lane, int* bad) {
  put<D>(sm, o, wave, lane);
  __syncthreads();
  for (int t = threadIdx.x; t < 32 * d; t += 64 * NW) {
    const int r = t / d, e = t % d;
    if (r >= rows) break;
    float x = sm[at(r, e)];
#pragma unroll
    for (int w = 1; w < NW; ++w) x += sm[w * kState<D> + at(r, e)];
    out[(long)r * ld + e] = x * scale;
    if (!isfinite(x * scale)) bad[r] = 1;
  }
  __syncthreads();
}

template <int D>
__global__ __launch_bounds__(64 * NW) void attn_fwd_f32_kernel(const float* __restrict__ qkv, float* __restrict__ out,
                                                               float* __restrict__ lse, int s, int a, int d, float scale) {
  extern __shared__ float sm[];           // [NW] states, then [NW][2][32] maxima and sums
  __shared__ int bad[32];
  float* xm = sm + NW * kState<D>;
  const int qb = gridDim.z - 1 - blockIdx.z, head = blockIdx.x, bi = blockIdx.y;  // longest rows first
  const int h = a * d, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, hi = lane >> 5, l31 = lane & 31;
  const long ld = 3L * h;
  const float* base = qkv + (long)bi * s * ld + head * d;
  const int q = qb * 32 + l31;
  Frag<D> qf;
  load_row<D>(qf, base + (long)min(q, s - 1) * ld, hi, d);
  f32x16 o[D / 32];
  clear<D>(o);
  float m = -INFINITY, l = 0.f;
  for (int kb = wave; kb <= qb; kb += NW) {
    const int k0 = kb * 32;
    Frag<D> kf;
    load_row<D>(kf, base + h + (long)min(k0 + l31, s - 1) * ld, hi, d);
    f32x16 st = dot_rows<D>(kf, qf);
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = k0 + (v >> 2) * 8 + hi * 4 + (v & 3);
      st[v] = key > q ? -INFINITY : st[v] * scale;
      mx = fmaxf(mx, st[v]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m, mx), ref = softmax_ref(m_new), alpha = expf(m - ref);
    float rs = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      st[v] = expf(st[v] - ref);
      rs += st[v];
    }
    l = l * alpha + rs + __shfl_xor(rs, 32, 64);
    m = m_new;
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[i][v] *= alpha;
    add_rows<D>(o, base + 2 * h, ld, k0, s, d, st, lane);
  }
  put<D>(sm, o, wave, lane);
  clear_flags(bad);
  if (hi == 0) { xm[wave * 64 + l31] = m; xm[wave * 64 + 32 + l31] = l; }
  __syncthreads();
  // a wave without a block has m = -inf, l = 0, o = 0: its factor is 0 (wave 0 always has key 0)
  float* op = out + ((long)bi * s + qb * 32) * h + head * d;
  for (int t = threadIdx.x; t < 32 * d; t += 64 * NW) {
    const int r = t / d, e = t % d;
    if (qb * 32 + r >= s) break;
    float mm = xm[r];
#pragma unroll
    for (int w = 1; w < NW; ++w) mm = fmaxf(mm, xm[w * 64 + r]);
    float x = 0.f, sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = expf(xm[w * 64 + r] - mm);
      x += f * sm[w * kState<D> + at(r, e)];
      sum += f * xm[w * 64 + 32 + r];
    }
    op[(long)r * h + e] = x / sum;
    if (!isfinite(x / sum) && sum == sum) bad[r] = 1;
    if (e == 0) lse[((long)bi * a + head) * s + qb * 32 + r] = mm + logf(sum);
  }
  __syncthreads();
  for (int r = wave; r < 32; r += NW)
    if (bad[r]) attn_row_fwd<float>(qb * 32 + r, head, bi, qkv, out, lse, s, a, d, scale);
}

template <int D>
__device__ __forceinline__ void dq_body(float* sm, int* bad, int qb, int head, int bi, const float* __restrict__ qkv,
                                        const float* __restrict__ o, const float* __restrict__ dout,
                                        const float* __restrict__ lse, float* __restrict__ dqkv, int s, int a, int d,
                                        float scale) {
  const int h = a * d, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, hi = lane >> 5, l31 = lane & 31;
  const long ld = 3L * h, tok0 = (long)bi * s;
  const float* base = qkv + tok0 * ld + head * d;
  const int q = qb * 32 + l31, rq = min(q, s - 1);
  Frag<D> qf, dof;
  load_row<D>(qf, base + (long)rq * ld, hi, d);
  load_row<D>(dof, dout + (tok0 + rq) * h + head * d, hi, d);
  float Dq;
  {
    Frag<D> of;
    load_row<D>(of, o + (tok0 + rq) * h + head * d, hi, d);
    Dq = dot_self<D>(dof, of);
  }
  const float lq = lse[((long)bi * a + head) * s + rq];
  f32x16 dq[D / 32];
  clear<D>(dq);
  for (int kb = wave; kb <= qb; kb += NW) {
    const int k0 = kb * 32;
    const float* krow = base + h + (long)min(k0 + l31, s - 1) * ld;
    Frag<D> kf, vf;
    load_row<D>(kf, krow, hi, d);
    load_row<D>(vf, krow + h, hi, d);
    const f32x16 st = dot_rows<D>(kf, qf), dp = dot_rows<D>(vf, dof);
    f32x16 ds;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = k0 + (v >> 2) * 8 + hi * 4 + (v & 3);
      ds[v] = key > q ? 0.f : expf(st[v] * scale - lq) * (dp[v] - Dq);
    }
    add_rows<D>(dq, base + h, ld, k0, s, d, ds, lane);
  }
  clear_flags(bad);
  const bool lost = lq != lq || Dq != Dq;  // no weight or no gradient is a number: neither is the row
  sum_out<D>(sm, dq, dqkv + (tok0 + qb * 32) * ld + head * d, ld, s - qb * 32, d, scale, wave, lane, bad);
  for (int r = wave; r < 32; r += NW)
    if (bad[r] && !__shfl((int)lost, r, 64)) attn_row_dq<float>(qb * 32 + r, head, bi, qkv, o, dout, lse, dqkv, s, a, d, scale);
}

template <int D>
__device__ __forceinline__ void dkv_body(float* sm, int* bad, int kb, int head, int bi, const float* __restrict__ qkv,
                                         const float* __restrict__ o, const float* __restrict__ dout,
                                         const float* __restrict__ lse, float* __restrict__ dqkv, int s, int a, int d,
                                         float scale) {
  const int h = a * d, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, hi = lane >> 5, l31 = lane & 31;
  const long ld = 3L * h, tok0 = (long)bi * s;
  const float* base = qkv + tok0 * ld + head * d;
  const int key = kb * 32 + l31;
  const float* krow = base + h + (long)min(key, s - 1) * ld;
  Frag<D> kf, vf;
  load_row<D>(kf, krow, hi, d);
  load_row<D>(vf, krow + h, hi, d);
  f32x16 dk[D / 32], dv[D / 32];
  clear<D>(dk);
  clear<D>(dv);
  const int nb = (s + 31) / 32;
  for (int qb = kb + wave; qb < nb; qb += NW) {
    const int q0 = qb * 32, rq = min(q0 + l31, s - 1);
    const float* dorow = dout + (tok0 + rq) * h + head * d;
    Frag<D> dof;
    load_row<D>(dof, dorow, hi, d);
    float Dl;
    {
      Frag<D> of;
      load_row<D>(of, o + (tok0 + rq) * h + head * d, hi, d);
      Dl = dot_self<D>(dof, of);
    }
    const float ll = lse[((long)bi * a + head) * s + rq];
    const f32x16 dp = dot_rows<D>(dof, vf);
    Frag<D> qf;
    load_row<D>(qf, base + (long)rq * ld, hi, d);
    const f32x16 st = dot_rows<D>(qf, kf);
    f32x16 p, ds;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = (v >> 2) * 8 + hi * 4 + (v & 3);
      const float lr = __shfl(ll, r, 64), dr = __shfl(Dl, r, 64);
      const bool in = q0 + r < s && key <= q0 + r;
      p[v] = in ? expf(st[v] * scale - lr) : 0.f;
      ds[v] = in ? p[v] * (dp[v] - dr) : 0.f;
    }
    add_rows<D>(dv, dout + tok0 * h + head * d, h, q0, s, d, p, lane);
    add_rows<D>(dk, base, ld, q0, s, d, ds, lane);
  }
  float* op = dqkv + (tok0 + kb * 32) * ld + h + head * d;
  clear_flags(bad);
  sum_out<D>(sm, dk, op, ld, s - kb * 32, d, scale, wave, lane, bad);
  sum_out<D>(sm, dv, op + h, ld, s - kb * 32, d, 1.0f, wave, lane, bad);
  for (int r = wave; r < 32; r += NW)
    if (bad[r]) attn_row_dkv<float>(kb * 32 + r, head, bi, qkv, o, dout, lse, dqkv, s, a, d, scale);
}

template <int D>
__global__ __launch_bounds__(64 * NW) void attn_bwd_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ o,
                                                               const float* __restrict__ dout, const float* __restrict__ lse,
                                                               float* __restrict__ dqkv, int s, int a, int d, float scale) {
  extern __shared__ float sm[];
  __shared__ int bad[32];
  const int blk = blockIdx.z >> 1, nb = gridDim.z >> 1;  // the blocks with the longest walks first
  if (blockIdx.z & 1) dq_body<D>(sm, bad, nb - 1 - blk, blockIdx.x, blockIdx.y, qkv, o, dout, lse, dqkv, s, a, d, scale);
  else dkv_body<D>(sm, bad, blk, blockIdx.x, blockIdx.y, qkv, o, dout, lse, dqkv, s, a, d, scale);
}

template <typename K> hipError_t set_smem(K kern, size_t smem, bool* done) {
  if (*done) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e == hipSuccess) *done = true;
  return e;
}

template <int D> hipError_t fwd_f32(const AttnArgs& a, hipStream_t s) {
  static bool done = false;
  constexpr size_t smem = (size_t)NW * (kState<D> + 64) * sizeof(float);
  hipError_t e = set_smem(attn_fwd_f32_kernel<D>, smem, &done);
  if (e != hipSuccess) return e;
  attn_fwd_f32_kernel<D><<<dim3(a.a, a.b, (a.s + 31) / 32), 64 * NW, smem, s>>>((const float*)a.qkv, (float*)a.out, a.lse, a.s,
                                                                               a.a, a.d, 1.0f / sqrtf((float)a.d));
  return hipGetLastError();
}
template <int D> hipError_t bwd_f32(const AttnArgs& a, hipStream_t s) {
  static bool done = false;
  constexpr size_t smem = (size_t)NW * kState<D> * sizeof(float);
  hipError_t e = set_smem(attn_bwd_f32_kernel<D>, smem, &done);
  if (e != hipSuccess) return e;
  attn_bwd_f32_kernel<D><<<dim3(a.a, a.b, 2 * ((a.s + 31) / 32)), 64 * NW, smem, s>>>(
      (const float*)a.qkv, (const float*)a.o, (const float*)a.dout, a.lse, (float*)a.dqkv, a.s, a.a, a.d,
      1.0f / sqrtf((float)a.d));
  return hipGetLastError();
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
// rows of a head at 16-byte addresses; b and the row blocks (two per 32 rows in the backward) are grid dimensions of 16 bits
inline bool takes(const AttnArgs& a) {
  return a.d % 4 == 0 && a.d <= 128 && a.b < 65536 && 2 * ((a.s + 31) / 32) < 65536 && aligned16(a.qkv);
}

}  // namespace

template <> hipError_t launch_attention_fwd_mfma<float>(const AttnArgs& a, hipStream_t s, bool* taken) {
  *taken = takes(a);
  if (!*taken) return hipSuccess;
  return a.d <= 32 ? fwd_f32<32>(a, s) : a.d <= 64 ? fwd_f32<64>(a, s) : a.d <= 96 ? fwd_f32<96>(a, s) : fwd_f32<128>(a, s);
}
template <> hipError_t launch_attention_bwd_mfma<float>(const AttnArgs& a, hipStream_t s, bool* taken) {
  *taken = takes(a) && aligned16(a.o) && aligned16(a.dout);
  if (!*taken) return hipSuccess;
  return a.d <= 32 ? bwd_f32<32>(a, s) : a.d <= 64 ? bwd_f32<64>(a, s) : a.d <= 96 ? bwd_f32<96>(a, s) : bwd_f32<128>(a, s);
}

}  // namespace zb
