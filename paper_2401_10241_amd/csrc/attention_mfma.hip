// Causal multi-head attention on the gfx950 matrix cores (bf16 in, fp32 accumulate), forward and
// backward, for head sizes from 8 to 128 and any sequence length.
//
// All products are formed "transposed" so that a lane owns one query (forward, dQ) or one key
// (dK/dV) and softmax statistics never cross lanes except for one exchange between lane l and l+32:
//   forward   S^T = K Q^T           (32 keys x 32 queries per MFMA tile; lane = query)
//             O^T += V^T P^T        (P taken straight from the S^T accumulators as an MFMA operand)
//   dQ pass   S^T, dP^T = V dO^T,   dS^T = P^T o (dP^T - D),   dQ^T += K^T dS^T
//   dK/dV     S = Q K^T, dP = dO V^T (lane = key),  dV^T += dO^T P,  dK^T += Q^T dS
// dQ and dK/dV are separate workgroups of one launch (each recomputes S), so no floating-point atomics are
// needed and results do not depend on scheduling.
//
// Two forms of every kernel.  EDGE = false: head size 64, whole 128-row blocks.  EDGE = true: a head of d columns
// is padded with zeros to D = 32 / 64 / 96 / 128 on its way into registers and LDS, rows past the end of the
// sequence are zeros as well (a zero query or output gradient adds nothing; a key past the end is always behind
// the diagonal), and P and dS, fp32 values, go into their products as three bf16 terms, which hold all 24 bits of
// their mantissas (the whole-tile form rounds them to one).  Rows whose result is not finite are taken
// again from attention_rows.h.
//
// What bounds them: a workgroup is a chain of dependent tiles (LDS read -> MFMA -> exponentials -> MFMA), and
// the shapes that come here have few heads, so most of the chip is idle.  Where it is, two groups of waves share a
// workgroup's rows and take its tiles in turn (the rule and figures at `Fwd`).
// Measured: 16 heads of 75 columns, 777 tokens 315 us forward and 1292 us backward on the vector ALUs, 65 and 93 here
// with one group, 44 and 60 with two.
//
// A 32x32 accumulator tile holds, in lane l and element v, row 8*(v/4) + 4*(l>>5) + v%4 and column
// l&31.  Used directly as the k-operand of the next MFMA (16 rows per instruction: elements 0-7,
// then 8-15), lane l's slots j = 0..7 carry rows 16*kk' + 8*(j/4) + 4*(l>>5) + j%4; the other operand
// is fetched from LDS with the transposing load ds_read_b64_tr_b16 using the same row order.
//
// LDS tiles are [64 rows][D + 16] bf16 (rows = keys or queries, D contiguous); the 16-byte chunk c of
// row r sits at chunk position c ^ ((r >> 2) & 1), which keeps both the 16-byte row reads and the
// transposing reads free of bank conflicts.
#include "attention_rows.h"

namespace zb {

hipError_t launch_attention_fwd_d128(const AttnArgs& a, hipStream_t s);  // attention_mfma128.hip
hipError_t launch_attention_bwd_d128(const AttnArgs& a, hipStream_t s);

namespace {

constexpr int KB = 64;   // rows of the inner-loop tile
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

template <int D, int NW = 4> struct AT {
  static constexpr int PITCH = D + 16;
  static constexpr int CH = KB * D / 8 / (64 * NW);  // 16-byte chunks per thread per tile
  static constexpr int TILE = KB * PITCH;      // elements
};

// Columns c0 .. c0+7 of a row of d columns (d >= 8): read inside the row only, at any even address; then, when
// the load has arrived, zeros from column d on (`valid` false: all zeros).  Two steps so that a tile's loads are
// all in flight before the first is waited for.
typedef u32x4 __attribute__((aligned(2))) u32x4_any;
__device__ __forceinline__ u32x4 load_chunk(const bf16_t* __restrict__ row, int c0, int d) {
  return *reinterpret_cast<const u32x4_any*>(row + min(c0, d - 8));
}
__device__ __forceinline__ u32x4 trim_chunk(u32x4 v, int c0, int d, bool valid) {
  const int sh = valid ? c0 - min(c0, d - 8) : 8;
  if (sh) {  // a tail chunk was read from column d - 8: move it down
    unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v);
    x = sh < 8 ? x >> (16 * sh) : 0;
    v = __builtin_bit_cast(u32x4, x);
  }
  return v;
}

// A workgroup is NG groups of NW waves that own the same rows and take the tiles of the other side in turn, each
// with its own LDS stages; the second hands its sums to the first at the end.
template <int NW> __device__ __forceinline__ int group_thread() { return threadIdx.x & (64 * NW - 1); }
template <int NW> __device__ __forceinline__ int group_of() { return __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * NW)); }
// this lane's place for n floats of its wave, 64 apart
__device__ __forceinline__ float* hand_over(unsigned char* smem, int wave, int n, int lane) {
  return reinterpret_cast<float*>(smem) + wave * n * 64 + lane;
}
template <int N> __device__ __forceinline__ void put(float* x, const f32x16 (&t)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) x[(i * 16 + v) * 64] = t[i][v];
}
template <int N> __device__ __forceinline__ void add(f32x16 (&t)[N], const float* x) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) t[i][v] += x[(i * 16 + v) * 64];
}

// rows [0, KB) of a tile whose first `rows` exist, NW * 64 threads
template <int D, int NW, bool EDGE, int CH>
__device__ __forceinline__ void gload_tile(u32x4 (&reg)[CH], const bf16_t* __restrict__ base, long ld, int rows, int d) {
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int c = group_thread<NW>() + 64 * NW * j;
    const int row = c / (D / 8), dc = c % (D / 8);
    if constexpr (EDGE) reg[j] = load_chunk(base + (long)min(row, rows - 1) * ld, dc * 8, d);
    else reg[j] = *reinterpret_cast<const u32x4*>(base + (long)row * ld + dc * 8);
  }
}
template <int D, int NW, bool EDGE, int CH>
__device__ __forceinline__ void lstore_tile(const u32x4 (&reg)[CH], bf16_t* __restrict__ s, int rows, int d) {
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int c = group_thread<NW>() + 64 * NW * j;
    const int row = c / (D / 8), dc = c % (D / 8);
    *reinterpret_cast<u32x4*>(s + row * AT<D>::PITCH + ((dc ^ ((row >> 2) & 1)) << 3)) =
        EDGE ? trim_chunk(reg[j], dc * 8, d, row < rows) : reg[j];
  }
}
// the row's k-operand fragments (columns kk*16 + hi*8 ..) straight from memory
template <int D, bool EDGE>
__device__ __forceinline__ void load_row_frags(bf16x8 (&f)[D / 16], const bf16_t* __restrict__ row, int hi, bool valid, int d) {
  if constexpr (EDGE) {
    u32x4 v[D / 16];
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) v[kk] = load_chunk(row, kk * 16 + hi * 8, d);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) f[kk] = __builtin_bit_cast(bf16x8, trim_chunk(v[kk], kk * 16 + hi * 8, d, valid));
  } else {
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) f[kk] = *reinterpret_cast<const bf16x8*>(row + kk * 16 + hi * 8);
  }
}

// operand fragment with rows = tile rows rb..rb+31 and k = D-columns kk*16..kk*16+15
template <int D> __device__ __forceinline__ bf16x8 frag_rowk(const bf16_t* __restrict__ s, int rb, int kk, int lane) {
  const int row = rb + (lane & 31);
  const int chunk = kk * 2 + (lane >> 5);
  return *reinterpret_cast<const bf16x8*>(s + row * AT<D>::PITCH + ((chunk ^ ((row >> 2) & 1)) << 3));
}

// operand fragment with rows = D-columns eb..eb+31 and k = tile rows, in accumulator row order:
// slots 0-3 = rows kl0 + 4*(lane>>5) + 0..3, slots 4-7 = the same + 8
template <int D> __device__ __forceinline__ bf16x8 frag_tr(const bf16_t* __restrict__ s, int eb, int kl0, int lane) {
  const int blk = lane >> 4, a = lane & 15;
  const int e = eb + ((blk & 1) << 4) + ((a & 3) << 2);
  const int kl = kl0 + ((blk >> 1) << 2) + (a >> 2);
  const int sw = (kl >> 2) & 1;  // same for kl and kl + 8
  const bf16_t* p = s + kl * AT<D>::PITCH + ((((e >> 3) ^ sw) << 3) | (e & 7));
  typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 8 * AT<D>::PITCH));
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// elements 8*half .. 8*half+7 of an accumulator tile as a bf16 k-operand
__device__ __forceinline__ bf16x8 pack_half(const f32x16& t, int half) {
  bf16x8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = (bf16_t)t[half * 8 + j];
  return r;
}

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Elements 8*half .. 8*half+7 of an accumulator tile as a k-operand: rounded to bf16 or, with edges, all of them in
// three terms (x - hi and x - hi - mid are exact)
template <bool EDGE> struct Weights { bf16x8 t[EDGE ? 3 : 1]; };
template <bool EDGE> __device__ __forceinline__ Weights<EDGE> weights(const f32x16& t, int half) {
  Weights<EDGE> w;
  w.t[0] = pack_half(t, half);
  if constexpr (EDGE) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float r = t[half * 8 + j] - (float)w.t[0][j];
      w.t[1][j] = (bf16_t)r;
      w.t[2][j] = (bf16_t)(r - (float)w.t[1][j]);
    }
  }
  return w;
}
template <bool EDGE> __device__ __forceinline__ f32x16 mfma(bf16x8 a, const Weights<EDGE>& w, f32x16 c) {
#pragma unroll
  for (const bf16x8& t : w.t) c = mfma(a, t, c);
  return c;
}
// The softmax: in powers of two on whole tiles, in powers of e with edges
template <bool EDGE> __device__ __forceinline__ float exp_of(float x) { return EDGE ? expf(x) : __builtin_amdgcn_exp2f(x); }
template <bool EDGE> __device__ __forceinline__ float units(float x) { return EDGE ? x : x * kLog2e; }

__device__ __forceinline__ void store4(bf16_t* p, float a, float b, float c, float d) {
  bf16x4 t;
  t[0] = (bf16_t)a; t[1] = (bf16_t)b; t[2] = (bf16_t)c; t[3] = (bf16_t)d;
  *reinterpret_cast<bf16x4*>(p) = t;
}
// one of this lane's 16 x N values is infinite or NaN
template <int N> __device__ __forceinline__ bool not_finite(const f32x16 (&t)[N]) {
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) z = fmaf(t[i][v], 0.f, z);
  return z != 0.f;
}
// bit r: the row of lanes r and r + 32 is one that either lane calls bad
__device__ __forceinline__ unsigned bad_rows(bool bad) {
  const unsigned long long b = __ballot(bad);
  return (unsigned)(b | (b >> 32));
}
// columns e .. e+3 of a row of d columns
template <bool EDGE>
__device__ __forceinline__ void store4_row(bf16_t* row, int e, int d, float a, float b, float c, float f) {
  if (!EDGE || (d % 4 == 0 && e < d)) {
    store4(row + e, a, b, c, f);
  } else {
    if (e < d) row[e] = (bf16_t)a;
    if (e + 1 < d) row[e + 1] = (bf16_t)b;
    if (e + 2 < d) row[e + 2] = (bf16_t)c;
    if (e + 3 < d) row[e + 3] = (bf16_t)f;
  }
}

// ------------------------------------------------------------------------------------------------
// forward
// ------------------------------------------------------------------------------------------------
template <int D, int NW, int NG, bool EDGE>
__global__ __launch_bounds__(64 * NW * NG) void attn_fwd_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ out,
                                                           float* __restrict__ lse, int s, int a, int d, float scale) {
  constexpr int QB = 32 * NW;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int grp = NG > 1 ? group_of<NW>() : 0;
  bf16_t* sK = reinterpret_cast<bf16_t*>(smem_raw) + grp * 4 * AT<D>::TILE;  // [2][TILE]
  bf16_t* sV = sK + 2 * AT<D>::TILE;
  const int qb = gridDim.z - 1 - blockIdx.z, head = blockIdx.x, bi = blockIdx.y;  // heaviest blocks first
  if (!EDGE) d = D;
  const int h = a * d;
  const long ld = 3L * h;
  const long tok0 = (long)bi * s;
  const int wave = group_thread<NW>() >> 6, lane = threadIdx.x & 63;
  const int hi = lane >> 5, lq = lane & 31;
  const int qw0 = qb * QB + wave * 32;  // first query of this wave
  const float su = units<EDGE>(scale);

  const bool mine = !EDGE || qw0 + lq < s;  // this lane's query exists
  const int row_q = mine ? qw0 + lq : s - 1;
  bf16x8 qf[D / 16];
  load_row_frags<D, EDGE>(qf, qkv + (tok0 + row_q) * ld + head * d, hi, mine, d);
  f32x16 o[D / 32];
#pragma unroll
  for (int et = 0; et < D / 32; ++et)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[et][v] = 0.f;
  float m = -INFINITY, l = 0.f;

  const int nkb = EDGE ? (min((qb + 1) * QB, s) + KB - 1) / KB : (qb + 1) * QB / KB;
  const bf16_t* kbase = qkv + tok0 * ld + h + head * d;
  const bf16_t* vbase = kbase + h;
  u32x4 rk[AT<D, NW>::CH], rv[AT<D, NW>::CH];
  auto gload = [&](int jb) {
    gload_tile<D, NW, EDGE>(rk, kbase + (long)jb * KB * ld, ld, s - jb * KB, d);
    gload_tile<D, NW, EDGE>(rv, vbase + (long)jb * KB * ld, ld, s - jb * KB, d);
  };
  auto lstore = [&](int jb, int stage) {
    lstore_tile<D, NW, EDGE>(rk, sK + stage * AT<D>::TILE, s - jb * KB, d);
    lstore_tile<D, NW, EDGE>(rv, sV + stage * AT<D>::TILE, s - jb * KB, d);
  };
  if (grp < nkb) {
    gload(grp);
    lstore(grp, 0);
  }
  if (grp + NG < nkb) gload(grp + NG);
  __syncthreads();

  for (int it = 0; it * NG < nkb; ++it) {
    const int jb = it * NG + grp;  // this group's tile (none in the last step if past the end)
    const bf16_t* kc = sK + (it & 1) * AT<D>::TILE;
    const bf16_t* vc = sV + (it & 1) * AT<D>::TILE;
    const int key0 = jb * KB;
    if (jb < nkb && key0 <= qw0 + 31) {  // this wave still has unmasked keys in the tile
      const bool act1 = key0 + 32 <= qw0 + 31;
      f32x16 st[2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) st[t][v] = 0.f;
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        st[0] = mfma(frag_rowk<D>(kc, 0, kk, lane), qf[kk], st[0]);
        if (act1) st[1] = mfma(frag_rowk<D>(kc, 32, kk, lane), qf[kk], st[1]);
      }
      const bool diag = key0 + KB - 1 > qw0;
      const int myq = qw0 + lq;
      float mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          float x = st[t][v] * su;
          if (diag) {
            const int key = key0 + t * 32 + (v >> 2) * 8 + hi * 4 + (v & 3);
            if (key > myq) x = -INFINITY;
          }
          st[t][v] = x;
          mx = fmaxf(mx, x);
        }
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m, mx), ref = softmax_ref(m_new);
      const float alpha = exp_of<EDGE>(m - ref);
      float rs = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float p = exp_of<EDGE>(st[t][v] - ref);
          st[t][v] = p;
          rs += p;
        }
      rs += __shfl_xor(rs, 32, 64);
      l = l * alpha + rs;
      m = m_new;
#pragma unroll
      for (int et = 0; et < D / 32; ++et)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[et][v] *= alpha;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (kk < 2 || act1) {
          const Weights<EDGE> pf = weights<EDGE>(st[kk >> 1], kk & 1);
#pragma unroll
          for (int et = 0; et < D / 32; ++et) {
            const bf16x8 vf = frag_tr<D>(vc, et * 32, kk * 16, lane);
            o[et] = mfma(vf, pf, o[et]);
          }
        }
      }
    }
    if (jb + NG < nkb) lstore(jb + NG, (it + 1) & 1);
    __syncthreads();
    if (jb + 2 * NG < nkb) gload(jb + 2 * NG);
  }

  if constexpr (NG > 1) {
    float* x = hand_over(smem_raw, wave, D / 2 + 2, lane);
    if (grp) {
      x[0] = m;
      x[64] = l;
      put(x + 128, o);
    }
    __syncthreads();
    if (grp) return;
    const float m1 = x[0], m_new = fmaxf(m, m1), ref = softmax_ref(m_new);
    const float a0 = exp_of<EDGE>(m - ref), a1 = exp_of<EDGE>(m1 - ref);
    l = l * a0 + x[64] * a1;
    m = m_new;
#pragma unroll
    for (int et = 0; et < D / 32; ++et)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[et][v] = o[et][v] * a0 + x[(2 + et * 16 + v) * 64] * a1;
  }
  const float inv = 1.0f / l;
#pragma unroll
  for (int et = 0; et < D / 32; ++et)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[et][v] *= inv;
  unsigned bad = 0;
  if constexpr (EDGE) bad = bad_rows(mine && l == l && not_finite(o));
  if (mine && !(bad >> lq & 1)) {
    bf16_t* op = out + (tok0 + qw0 + lq) * h + head * d;
#pragma unroll
    for (int et = 0; et < D / 32; ++et)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        store4_row<EDGE>(op, et * 32 + g * 8 + hi * 4, d, o[et][4 * g], o[et][4 * g + 1], o[et][4 * g + 2], o[et][4 * g + 3]);
    if (hi == 0) lse[((long)bi * a + head) * s + qw0 + lq] = EDGE ? m + logf(l) : (m + __builtin_amdgcn_logf(l)) * kLn2;
  }
  if constexpr (EDGE)
    for (; bad; bad &= bad - 1) attn_row_fwd<bf16_t>(qw0 + __builtin_ctz(bad), head, bi, qkv, out, lse, s, a, d, scale);
}

// ------------------------------------------------------------------------------------------------
// backward, step 0: D_i = dO_i . O_i     (16 lanes per (row, head), 16 rows per workgroup)
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void attn_bwd_prep_kernel(const bf16_t* __restrict__ o, const bf16_t* __restrict__ dout,
                                                            float* __restrict__ dvec, int s, int a, int d) {
  const int i = blockIdx.x * 16 + (threadIdx.x >> 4), head = blockIdx.y, bi = blockIdx.z;
  const int l16 = threadIdx.x & 15;
  const long off = ((long)bi * s + min(i, s - 1)) * a * d + head * d;
  float acc = 0.f;
#pragma unroll 8
  for (int e = l16; e < d; e += 16) acc += (float)o[off + e] * (float)dout[off + e];
#pragma unroll
  for (int x = 8; x > 0; x >>= 1) acc += __shfl_xor(acc, x, 64);
  if (l16 == 0 && i < s) dvec[((long)bi * a + head) * s + i] = acc;
}

// ------------------------------------------------------------------------------------------------
// backward, dQ: workgroup = 32 NW queries, loop over key tiles up to the diagonal
// ------------------------------------------------------------------------------------------------
template <int D, int NW, int NG, bool EDGE>
__device__ __forceinline__ void attn_bwd_dq_body(unsigned char* smem_raw, int qb, int head, int bi,
                                                 const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                                 const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                 const float* __restrict__ dvec, bf16_t* __restrict__ dqkv, int s, int a, int d, float scale) {
  constexpr int QB = 32 * NW;
  const int grp = NG > 1 ? group_of<NW>() : 0;
  bf16_t* sK = reinterpret_cast<bf16_t*>(smem_raw) + grp * 4 * AT<D>::TILE;
  bf16_t* sV = sK + 2 * AT<D>::TILE;
  if (!EDGE) d = D;
  const int h = a * d;
  const long ld = 3L * h;
  const long tok0 = (long)bi * s;
  const int wave = group_thread<NW>() >> 6, lane = threadIdx.x & 63;
  const int hi = lane >> 5, lq = lane & 31;
  const int qw0 = qb * QB + wave * 32;
  const float su = units<EDGE>(scale);

  const bool mine = !EDGE || qw0 + lq < s;
  const int row_q = mine ? qw0 + lq : s - 1;
  bf16x8 qf[D / 16], dof[D / 16];
  load_row_frags<D, EDGE>(qf, qkv + (tok0 + row_q) * ld + head * d, hi, mine, d);
  load_row_frags<D, EDGE>(dof, dout + (tok0 + row_q) * h + head * d, hi, mine, d);
  const long srow = ((long)bi * a + head) * s + row_q;
  const float lse_u = units<EDGE>(lse[srow]);
  const float Dq = dvec[srow];
  f32x16 dq[D / 32];
#pragma unroll
  for (int et = 0; et < D / 32; ++et)
#pragma unroll
    for (int v = 0; v < 16; ++v) dq[et][v] = 0.f;

  const int nkb = EDGE ? (min((qb + 1) * QB, s) + KB - 1) / KB : (qb + 1) * QB / KB;
  const bf16_t* kbase = qkv + tok0 * ld + h + head * d;
  const bf16_t* vbase = kbase + h;
  u32x4 rk[AT<D, NW>::CH], rv[AT<D, NW>::CH];
  auto gload = [&](int jb) {
    gload_tile<D, NW, EDGE>(rk, kbase + (long)jb * KB * ld, ld, s - jb * KB, d);
    gload_tile<D, NW, EDGE>(rv, vbase + (long)jb * KB * ld, ld, s - jb * KB, d);
  };
  auto lstore = [&](int jb, int stage) {
    lstore_tile<D, NW, EDGE>(rk, sK + stage * AT<D>::TILE, s - jb * KB, d);
    lstore_tile<D, NW, EDGE>(rv, sV + stage * AT<D>::TILE, s - jb * KB, d);
  };
  if (grp < nkb) {
    gload(grp);
    lstore(grp, 0);
  }
  if (grp + NG < nkb) gload(grp + NG);
  __syncthreads();

  for (int it = 0; it * NG < nkb; ++it) {
    const int jb = it * NG + grp;  // this group's tile (none in the last step if past the end)
    const bf16_t* kc = sK + (it & 1) * AT<D>::TILE;
    const bf16_t* vc = sV + (it & 1) * AT<D>::TILE;
    const int key0 = jb * KB;
    if (jb < nkb && key0 <= qw0 + 31) {
      const bool act1 = key0 + 32 <= qw0 + 31;
      f32x16 st[2], dpt[2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) st[t][v] = dpt[t][v] = 0.f;
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        st[0] = mfma(frag_rowk<D>(kc, 0, kk, lane), qf[kk], st[0]);
        dpt[0] = mfma(frag_rowk<D>(vc, 0, kk, lane), dof[kk], dpt[0]);
        if (act1) {
          st[1] = mfma(frag_rowk<D>(kc, 32, kk, lane), qf[kk], st[1]);
          dpt[1] = mfma(frag_rowk<D>(vc, 32, kk, lane), dof[kk], dpt[1]);
        }
      }
      const bool diag = key0 + KB - 1 > qw0;
      const int myq = qw0 + lq;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          float p = exp_of<EDGE>(st[t][v] * su - lse_u);
          if (diag) {
            const int key = key0 + t * 32 + (v >> 2) * 8 + hi * 4 + (v & 3);
            if (key > myq) p = 0.f;
          }
          st[t][v] = p * (dpt[t][v] - Dq);
        }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (kk < 2 || act1) {
          const Weights<EDGE> dsf = weights<EDGE>(st[kk >> 1], kk & 1);
#pragma unroll
          for (int et = 0; et < D / 32; ++et) {
            const bf16x8 kf = frag_tr<D>(kc, et * 32, kk * 16, lane);
            dq[et] = mfma(kf, dsf, dq[et]);
          }
        }
      }
    }
    if (jb + NG < nkb) lstore(jb + NG, (it + 1) & 1);
    __syncthreads();
    if (jb + 2 * NG < nkb) gload(jb + 2 * NG);
  }
  if constexpr (NG > 1) {
    float* x = hand_over(smem_raw, wave, D / 2, lane);
    if (grp) put(x, dq);
    __syncthreads();
    if (grp) return;
    add(dq, x);
  }
  unsigned bad = 0;
  if constexpr (EDGE) bad = bad_rows(mine && lse_u == lse_u && Dq == Dq && not_finite(dq));  // else every term is NaN
  if (mine && !(bad >> lq & 1)) {
    bf16_t* op = dqkv + (tok0 + qw0 + lq) * ld + head * d;
#pragma unroll
    for (int et = 0; et < D / 32; ++et)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        store4_row<EDGE>(op, et * 32 + g * 8 + hi * 4, d, dq[et][4 * g] * scale, dq[et][4 * g + 1] * scale,
                         dq[et][4 * g + 2] * scale, dq[et][4 * g + 3] * scale);
  }
  if constexpr (EDGE)
    for (; bad; bad &= bad - 1)
      attn_row_dq<bf16_t>(qw0 + __builtin_ctz(bad), head, bi, qkv, o, dout, lse, dqkv, s, a, d, scale);
}

// ------------------------------------------------------------------------------------------------
// backward, dK and dV: workgroup = 32 NW keys, loop over query tiles from the diagonal to the end
// ------------------------------------------------------------------------------------------------
template <int D, int NW, int NG, bool EDGE>
__device__ __forceinline__ void attn_bwd_dkv_body(unsigned char* smem_raw, int kb, int head, int bi,
                                                  const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                                  const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                  const float* __restrict__ dvec, bf16_t* __restrict__ dqkv, int s, int a, int d, float scale) {
  constexpr int QB = 32 * NW;
  const int grp = NG > 1 ? group_of<NW>() : 0;
  bf16_t* sQ = reinterpret_cast<bf16_t*>(smem_raw) + grp * 4 * AT<D>::TILE;  // [2][TILE]
  bf16_t* sO = sQ + 2 * AT<D>::TILE;                                         // dO tiles
  float* sL = reinterpret_cast<float*>(smem_raw + NG * 4 * AT<D>::TILE * sizeof(bf16_t)) + grp * 4 * KB;  // [2][64] lse in units of the softmax
  float* sD = sL + 2 * KB;                                     // [2][64] D
  if (!EDGE) d = D;
  const int h = a * d;
  const long ld = 3L * h;
  const long tok0 = (long)bi * s;
  const int wave = group_thread<NW>() >> 6, lane = threadIdx.x & 63;
  const int hi = lane >> 5, lk = lane & 31;
  const int kw0 = kb * QB + wave * 32;  // first key of this wave
  const float su = units<EDGE>(scale);

  const bool mine = !EDGE || kw0 + lk < s;
  const int row_k = mine ? kw0 + lk : s - 1;
  bf16x8 kf[D / 16], vf[D / 16];
  load_row_frags<D, EDGE>(kf, qkv + (tok0 + row_k) * ld + h + head * d, hi, mine, d);
  load_row_frags<D, EDGE>(vf, qkv + (tok0 + row_k) * ld + 2 * h + head * d, hi, mine, d);
  f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
  for (int et = 0; et < D / 32; ++et)
#pragma unroll
    for (int v = 0; v < 16; ++v) dk[et][v] = dv[et][v] = 0.f;

  const int ib0 = kb * (QB / KB), nib = (s + KB - 1) / KB;
  const bf16_t* qbase = qkv + tok0 * ld + head * d;
  const bf16_t* obase = dout + tok0 * h + head * d;
  const float* lbase = lse + ((long)bi * a + head) * s;
  const float* dbase = dvec + ((long)bi * a + head) * s;
  u32x4 rq[AT<D, NW>::CH], ro[AT<D, NW>::CH];
  float rs = 0.f;  // threads 0..63 stage lse, 64..127 stage D
  const int tid = group_thread<NW>();
  auto gload = [&](int ib) {
    gload_tile<D, NW, EDGE>(rq, qbase + (long)ib * KB * ld, ld, s - ib * KB, d);
    gload_tile<D, NW, EDGE>(ro, obase + (long)ib * KB * h, h, s - ib * KB, d);
    const int r = ib * KB + (tid & (KB - 1));
    if (EDGE && r >= s) rs = tid < KB ? INFINITY : 0.f;  // exp(-inf): no weight
    else if (tid < KB) rs = units<EDGE>(lbase[r]);
    else if (tid < 2 * KB) rs = dbase[r];
  };
  auto lstore = [&](int ib, int stage) {
    lstore_tile<D, NW, EDGE>(rq, sQ + stage * AT<D>::TILE, s - ib * KB, d);
    lstore_tile<D, NW, EDGE>(ro, sO + stage * AT<D>::TILE, s - ib * KB, d);
    if (tid < KB) sL[stage * KB + tid] = rs;
    else if (tid < 2 * KB) sD[stage * KB + tid - KB] = rs;
  };
  if (ib0 + grp < nib) {
    gload(ib0 + grp);
    lstore(ib0 + grp, 0);
  }
  if (ib0 + grp + NG < nib) gload(ib0 + grp + NG);
  __syncthreads();

  for (int it = 0; ib0 + it * NG < nib; ++it) {
    const int ib = ib0 + it * NG + grp;  // this group's tile (none in the last step if past the end)
    const int stage = it & 1;
    const bf16_t* qc = sQ + stage * AT<D>::TILE;
    const bf16_t* oc = sO + stage * AT<D>::TILE;
    const float* lc = sL + stage * KB;
    const float* dc = sD + stage * KB;
    const int q0 = ib * KB;
    if (ib < nib && q0 + KB - 1 >= kw0) {  // some query of the tile can see this wave's keys
      const bool act0 = q0 + 31 >= kw0;
      f32x16 st[2], dpt[2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) st[t][v] = dpt[t][v] = 0.f;
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        if (act0) {
          st[0] = mfma(frag_rowk<D>(qc, 0, kk, lane), kf[kk], st[0]);
          dpt[0] = mfma(frag_rowk<D>(oc, 0, kk, lane), vf[kk], dpt[0]);
        }
        st[1] = mfma(frag_rowk<D>(qc, 32, kk, lane), kf[kk], st[1]);
        dpt[1] = mfma(frag_rowk<D>(oc, 32, kk, lane), vf[kk], dpt[1]);
      }
      const bool diag = q0 < kw0 + 31;
      const int mykey = kw0 + lk;
      f32x16 pt[2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int qi = t * 32 + g * 8 + hi * 4;
          const f32x4 l4 = *reinterpret_cast<const f32x4*>(lc + qi);
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(dc + qi);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int v = g * 4 + i;
            float p = exp_of<EDGE>(st[t][v] * su - l4[i]);
            if (diag && mykey > q0 + qi + i) p = 0.f;
            if (t == 0 && !act0) p = 0.f;
            pt[t][v] = p;
            st[t][v] = p * (dpt[t][v] - d4[i]);
          }
        }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (kk >= 2 || act0) {
          const Weights<EDGE> pf = weights<EDGE>(pt[kk >> 1], kk & 1), dsf = weights<EDGE>(st[kk >> 1], kk & 1);
#pragma unroll
          for (int et = 0; et < D / 32; ++et) {
            const bf16x8 of = frag_tr<D>(oc, et * 32, kk * 16, lane), qf = frag_tr<D>(qc, et * 32, kk * 16, lane);
            dv[et] = mfma(of, pf, dv[et]);
            dk[et] = mfma(qf, dsf, dk[et]);
          }
        }
      }
    }
    if (ib + NG < nib) lstore(ib + NG, stage ^ 1);
    __syncthreads();
    if (ib + 2 * NG < nib) gload(ib + 2 * NG);
  }
  if constexpr (NG > 1) {
    float* x = hand_over(smem_raw, wave, D, lane);
    if (grp) {
      put(x, dk);
      put(x + D / 2 * 64, dv);
    }
    __syncthreads();
    if (grp) return;
    add(dk, x);
    add(dv, x + D / 2 * 64);
  }
  unsigned bad = 0;
  if constexpr (EDGE) bad = bad_rows(mine && (not_finite(dk) || not_finite(dv)));
  if (mine && !(bad >> lk & 1)) {
    bf16_t* kp = dqkv + (tok0 + kw0 + lk) * ld + h + head * d;
#pragma unroll
    for (int et = 0; et < D / 32; ++et)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int e = et * 32 + g * 8 + hi * 4;
        store4_row<EDGE>(kp, e, d, dk[et][4 * g] * scale, dk[et][4 * g + 1] * scale, dk[et][4 * g + 2] * scale,
                         dk[et][4 * g + 3] * scale);
        store4_row<EDGE>(kp + h, e, d, dv[et][4 * g], dv[et][4 * g + 1], dv[et][4 * g + 2], dv[et][4 * g + 3]);
      }
  }
  if constexpr (EDGE)
    for (; bad; bad &= bad - 1)
      attn_row_dkv<bf16_t>(kw0 + __builtin_ctz(bad), head, bi, qkv, o, dout, lse, dqkv, s, a, d, scale);
}

// Both halves of the backward in one launch: they are independent, and each alone leaves most of the chip idle.
// Even workgroups are key blocks, odd ones query blocks, those with the most tiles first.
template <int D, int NW, int NG, bool EDGE>
__global__ __launch_bounds__(64 * NW * NG) void attn_bwd_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                                           const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                           const float* __restrict__ dvec, bf16_t* __restrict__ dqkv, int s, int a, int d, float scale) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int blk = blockIdx.z >> 1, nblk = gridDim.z >> 1, head = blockIdx.x, bi = blockIdx.y;
  if (blockIdx.z & 1)
    attn_bwd_dq_body<D, NW, NG, EDGE>(smem_raw, nblk - 1 - blk, head, bi, qkv, o, dout, lse, dvec, dqkv, s, a, d, scale);
  else
    attn_bwd_dkv_body<D, NW, NG, EDGE>(smem_raw, blk, head, bi, qkv, o, dout, lse, dvec, dqkv, s, a, d, scale);
}

template <typename K> hipError_t set_smem(K kern, size_t smem, bool* done) {
  if (*done) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)smem);
  if (e == hipSuccess) *done = true;
  return e;
}

template <int D, int NW, int NG, bool EDGE> hipError_t run_fwd(const AttnArgs& a, hipStream_t s) {
  static bool done = false;
  constexpr size_t smem = (size_t)NG * 4 * AT<D>::TILE * sizeof(bf16_t);
  static_assert(smem <= 160 * 1024 && (NG == 1 || smem >= (size_t)NW * (D / 2 + 2) * 64 * sizeof(float)), "stages; what a group hands over");
  hipError_t e = set_smem(attn_fwd_kernel<D, NW, NG, EDGE>, smem, &done);
  if (e != hipSuccess) return e;
  dim3 grid(a.a, a.b, (a.s + 32 * NW - 1) / (32 * NW));  // the last index is the slowest: heaviest blocks of all heads first
  attn_fwd_kernel<D, NW, NG, EDGE><<<grid, 64 * NW * NG, smem, s>>>((const bf16_t*)a.qkv, (bf16_t*)a.out, a.lse, a.s, a.a, a.d,
                                                          1.0f / sqrtf((float)a.d));
  return hipGetLastError();
}

template <int D, int NW, int NG, bool EDGE> hipError_t run_bwd(const AttnArgs& a, hipStream_t s) {
  static bool done = false;
  constexpr size_t smem = (size_t)NG * (4 * AT<D>::TILE * sizeof(bf16_t) + 4 * KB * sizeof(float));
  static_assert(smem <= 160 * 1024 && (NG == 1 || smem >= (size_t)NW * D * 64 * sizeof(float)), "stages; what a group hands over");
  hipError_t e = set_smem(attn_bwd_kernel<D, NW, NG, EDGE>, smem, &done);
  if (e != hipSuccess) return e;
  dim3 grid1((a.s + 15) / 16, a.a, a.b);
  attn_bwd_prep_kernel<<<grid1, 256, 0, s>>>((const bf16_t*)a.o, (const bf16_t*)a.dout, a.dvec, a.s, a.a, a.d);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 grid(a.a, a.b, 2 * ((a.s + 32 * NW - 1) / (32 * NW)));
  attn_bwd_kernel<D, NW, NG, EDGE><<<grid, 64 * NW * NG, smem, s>>>((const bf16_t*)a.qkv, (const bf16_t*)a.o, (const bf16_t*)a.dout, a.lse,
                                                          a.dvec, (bf16_t*)a.dqkv, a.s, a.a, a.d, 1.0f / sqrtf((float)a.d));
  return hipGetLastError();
}

// whole tiles: head sizes 96 and 128 go to attention_mfma128.hip, 64 to the kernels above without edges
inline bool whole_tiles(const AttnArgs& a) { return a.s % 128 == 0 && (a.d == 64 || a.d == 96 || a.d == 128); }
// sizes the kernels above take (b and the row blocks are grid dimensions of 16 bits)
inline bool mfma_shape(const AttnArgs& a) { return a.d >= 8 && a.d <= 128 && a.b < 65536 && a.a < 65536 && a.s <= (1 << 20); }
// Rows per workgroup: 128 (four waves) or 64 (two), and one or two groups of that many waves.  Two groups halve the chain
// of tiles and put a second wave on each SIMD where the launch leaves the chip room for them; two waves share the staging
// of a tile between fewer rows but leave less idle at the diagonal and pack the CUs more evenly.  Measured, us with 64 rows /
// 128 rows / 64 rows, two groups / 128 rows, two groups (heads x tokens x samples; blocks = 128-row blocks of the launch):
//   forward, whole tiles  16 x 256 (32) 10.6 / 11.2 / 7.5 / 8.2, 12 x 512 (48) 18.6 / 19.2 / 11.7 / 11.9, 12 x 1024 (96) 34.4 / 34.9 /
//                         20.5 / 19.8, 16 x 256 x 8 (256) 11.7 / 11.8 / 8.6 / 8.8, 16 x 1024 x 3 (384) 37.1 / 35.6 / 25.5 / 21.3,
//                         32 x 512 x 4 (512) 22.6 / 21.2 / 21.4 / 18.0, but 64 x 128 x 8 (512) 10.3 / 10.4 / 12.3 / 12.4, 64 x 1024 x 2
//                         (1024) 59 / 50 / 61 / 52
//   forward, edges        head 75: 16 x 130 (32) 20.2 / 18.9 / 16.5 / 16.5, 16 x 777 (112) 73 / 65 / 45 / 44, 16 x 777 x 4 (448) 77 / 68 /
//                         94 / 61, 96 x 777 (672) 119 / 86 / 139 / 91; head 40: 16 x 500 x 4 (256) 35 / 33 / 21 / 22; head 128: 64 x
//                         257 x 2 (384) 33 / 39 / 40 / 30; head 96: 64 x 130 x 3 (384) 18.6 / 18.6 / 25.8 / 22.7
//   backward, whole tiles 16 x 256 (32) 15.7 / 17.1 / 12.0 / 15.5, 12 x 512 (48) 26.0 / 27.3 / 17.8 / 22.5, 8 x 2048 (128) 90 / 87 / 56 /
//                         63, 12 x 512 x 3 (144) 29.1 / 28.4 / 27.1 / 24.4, 16 x 256 x 8 (256) 23.5 / 25.8 / 31.1 / 24.7, 64 x 512 (256)
//                         34.2 / 36.0 / 42.3 / 32.6, 64 x 1024 x 2 (1024) 198 / 208 / 242 / 159
//   backward, edges       head 75: 16 x 130 (32) 30 / 34 / 25 / -, 16 x 777 (112) 96 / 93 / 60 / -, 16 x 777 x 2 (224) 99 / 96 / 106 / -;
//                         head 128: 18 x 1100 (162) 135 / 125 / 99 / -, 16 x 257 x 4 (192) 44.9 / 44.3 / 47.5 / -; one group: 128 x
//                         257 (384) 74 / 93, 96 x 777 (672) 253 / 273, 64 x 1500 (768) 500 / 483, head 40 96 x 256 (192) 29 / 31
//                         (- : 128 rows and two groups do not fit the registers)
// With edges the second group also doubles the staging (zeros past the columns are put in on the way) or the LDS of wide heads,
// which costs where other launches want the chip: three stages at once, us per iteration with one and two groups: 16 heads
// of 75, 777 tokens 2340 / 2308 with a forward in two, / 2390 with the backward as well; 16 of 40, 178 tokens 1161 / 1184; 4 of
// 48, 945 tokens 1168 / 1004.  So two groups from 256 tokens on, and in the backward of heads up to 64 columns.
// Where launches of two groups come near filling the chip the second only shares it (heads x tokens x samples, us with one
// group / two): forward, whole tiles 40 x 1024 x 3 (960) 46 / 51, 16 x 2048 x 3 (768) 71 / 65; backward 40 x 128 x 3 (120) 12.4 /
// 14.8, 16 x 128 x 3 (48) 10.9 / 9.6; forward of heads whose columns are staged singly, head 75 40 x 257 x 3 (360) 30 / 35, but
// 16 x 257 x 3 (144) 28 / 22, 40 x 257 x 3 of head 96 26 / 25.
inline long blocks128(const AttnArgs& a) { return (long)((a.s + 127) / 128) * a.a * a.b; }
template <int D, bool EDGE> struct Fwd {
  static hipError_t run(const AttnArgs& a, hipStream_t s) {
    const long n = blocks128(a);
    if constexpr (!EDGE) {
      if (n < 96) return run_fwd<D, 2, 2, EDGE>(a, s);
      if (n < 512 || (n < 896 && a.s >= 512)) return run_fwd<D, 4, 2, EDGE>(a, s);
    } else {
      if (n < 512 && a.s >= (n >= 256 && a.d % 8 != 0 ? 512 : 256)) return run_fwd<D, D <= 64 ? 2 : 4, 2, EDGE>(a, s);
      if constexpr (D == 128)
        if (a.s < 1024 && n >= 352) return run_fwd<D, 2, 1, EDGE>(a, s);
    }
    return run_fwd<D, 4, 1, EDGE>(a, s);
  }
};
template <int D, bool EDGE> struct Bwd {
  static hipError_t run(const AttnArgs& a, hipStream_t s) {
    const long n = blocks128(a);
    if (EDGE ? n <= 128 && D <= 64 && a.s >= 256 : n <= (a.s >= 256 ? 128 : 64)) return run_bwd<D, 2, 2, EDGE>(a, s);
    if constexpr (!EDGE) {
      return a.s >= 512 ? run_bwd<D, 4, 2, EDGE>(a, s) : run_bwd<D, 2, 1, EDGE>(a, s);
    } else {
      const bool narrow = (a.s < 1024 && n >= 192) || (D == 96 && a.s <= 256);
      return narrow ? run_bwd<D, 2, 1, EDGE>(a, s) : run_bwd<D, 4, 1, EDGE>(a, s);
    }
  }
};

template <template <int, bool> class Run> hipError_t run_shape(const AttnArgs& a, hipStream_t s) {
  if (whole_tiles(a)) return Run<64, false>::run(a, s);
  if (a.d <= 32) return Run<32, true>::run(a, s);
  if (a.d <= 64) return Run<64, true>::run(a, s);
  if (a.d <= 96) return Run<96, true>::run(a, s);
  return Run<128, true>::run(a, s);
}

}  // namespace

// fp32: attention_f32.hip
template <typename T> hipError_t launch_attention_fwd_mfma(const AttnArgs& a, hipStream_t s, bool* taken);
template <typename T> hipError_t launch_attention_bwd_mfma(const AttnArgs& a, hipStream_t s, bool* taken);
template <> hipError_t launch_attention_fwd_mfma<bf16_t>(const AttnArgs& a, hipStream_t s, bool* taken) {
  *taken = mfma_shape(a);
  if (!*taken) return hipSuccess;
  return whole_tiles(a) && a.d != 64 ? launch_attention_fwd_d128(a, s) : run_shape<Fwd>(a, s);
}
template <> hipError_t launch_attention_bwd_mfma<bf16_t>(const AttnArgs& a, hipStream_t s, bool* taken) {
  *taken = mfma_shape(a);
  if (!*taken) return hipSuccess;
  return whole_tiles(a) && a.d != 64 ? launch_attention_bwd_d128(a, s) : run_shape<Bwd>(a, s);
}

}  // namespace zb
