// fp32 GEMMs on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and sums, nothing rounded below fp32),
// all three operand forms: forward X*W, dgrad dY*W^T (W as stored, K-contiguous), wgrad X^T*dY.
//
// A workgroup owns one output tile and its waves split K between them, 32 k at a time in turn; fragments come
// straight from memory into registers, and the waves' partial tiles are added through LDS in wave order.  What bounds
// the products that come here (hundreds of tokens, widths up to a few thousand) is latency, so a wave has the loads of four
// (16 x 16 tiles) or two (32 x 32) of its blocks in flight before the first product: with one block ahead of the products 128 x
// 256 x 1024 took 22.5 us (dgrad 12.3).  Small products take 16 x 16 tiles, four times the workgroups: 5.9 us.  The 64 x 64 tiles of the
// largest, which other workgroups' loads keep busy, and the W of four waves, which have one block each, load one at a time.  The
// rules are at `kSmallTiles` and `four_waves`.
#include <algorithm>

#include "gemm_epilogue.h"

namespace zb {

template <typename T> hipError_t launch_gemm_mfma(const GemmArgs& g, hipStream_t s, bool* taken);
template <typename T> hipError_t launch_wgrad_multi_mfma(const WgradMultiArgs& w, hipStream_t s, bool* taken);
template <typename T> hipError_t launch_gemm_generic(const GemmArgs& g, hipStream_t s);

namespace {

constexpr int KB = 32;  // k per block

// An MFMA tile is T x T: 32 x 32 (v_mfma_f32_32x32x2_f32) or 16 x 16 (v_mfma_f32_16x16x4_f32), the same rate.
template <int T> struct Mfma;
template <> struct Mfma<32> {
  using Acc = f32x16;
  static __device__ __forceinline__ void mac(float a, float b, Acc& c) { c = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
};
template <> struct Mfma<16> {
  using Acc = f32x4;
  static __device__ __forceinline__ void mac(float a, float b, Acc& c) { c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};
template <int T> using Acc = typename Mfma<T>::Acc;
template <int T> using Frag = f32x4[KB * T / 256];

// One operand's row (or column) r of this lane (lane % T), k0 .. k0+31: element 4q + j is k = k0 + (256 / T) q + 4 hi + j,
// hi = lane / T.  KC: element (r, k) at p[r * ld + k], K and ld multiples of 4; else at p[k * ld + r].  k >= K: zero.
template <int T, bool KC>
__device__ __forceinline__ void load_frag(Frag<T>& f, const float* __restrict__ p, long ld, int r, int k0, int K, int hi) {
#pragma unroll
  for (int q = 0; q < KB * T / 256; ++q) {
    const int k = k0 + q * (256 / T) + hi * 4;
    if constexpr (KC) {
      f[q] = *reinterpret_cast<const f32x4*>(p + (long)r * ld + min(k, K - 4));
      if (k >= K) f[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = p[(long)min(k + j, K - 1) * ld + r];
        f[q][j] = k + j < K ? v : 0.f;
      }
    }
  }
}

// ND blocks of a wave's share of a tile, `step` apart in k: all their loads are in flight before the first product
template <int T, int MT, int NT, int ND, bool AKC, bool BKC>
__device__ __forceinline__ void wave_blocks(Acc<T> (&acc)[MT][NT], const float* __restrict__ A, const float* __restrict__ B,
                                            int K, long lda, long ldb, const int (&rm)[MT], const int (&rn)[NT], int k0,
                                            int step, int hi) {
  Frag<T> a[ND][MT], b[ND][NT];
#pragma unroll
  for (int d = 0; d < ND; ++d) {
#pragma unroll
    for (int i = 0; i < MT; ++i) load_frag<T, AKC>(a[d][i], A, lda, rm[i], k0 + d * step, K, hi);
#pragma unroll
    for (int j = 0; j < NT; ++j) load_frag<T, BKC>(b[d][j], B, ldb, rn[j], k0 + d * step, K, hi);
  }
#pragma unroll
  for (int d = 0; d < ND; ++d)
#pragma unroll
    for (int q = 0; q < KB * T / 256; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j) Mfma<T>::mac(a[d][i][q][e], b[d][j][q][e], acc[i][j]);
}

// This wave's share of the TM x TN tile at (m0, n0), ND (1, 2 or 4) blocks at a time
template <int T, int TM, int TN, int NW, int ND, bool AKC, bool BKC>
__device__ __forceinline__ void wave_tile(Acc<T> (&acc)[TM / T][TN / T], const float* __restrict__ A,
                                          const float* __restrict__ B, int M, int N, int K, long lda, long ldb, int m0,
                                          int n0, int wave, int lane) {
  constexpr int MT = TM / T, NT = TN / T, step = NW * KB;
  const int hi = lane / T;
  int rm[MT], rn[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) rm[i] = min(m0 + i * T + lane % T, M - 1);
#pragma unroll
  for (int j = 0; j < NT; ++j) rn[j] = min(n0 + j * T + lane % T, N - 1);
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < T * T / 64; ++v) acc[i][j][v] = 0.f;
  int k0 = wave * KB;
  for (; k0 + (ND - 1) * step < K; k0 += ND * step)
    wave_blocks<T, MT, NT, ND, AKC, BKC>(acc, A, B, K, lda, ldb, rm, rn, k0, step, hi);
  if constexpr (ND > 2)
    if (k0 + step < K) {
      wave_blocks<T, MT, NT, 2, AKC, BKC>(acc, A, B, K, lda, ldb, rm, rn, k0, step, hi);
      k0 += 2 * step;
    }
  if constexpr (ND > 1)
    if (k0 < K) wave_blocks<T, MT, NT, 1, AKC, BKC>(acc, A, B, K, lda, ldb, rm, rn, k0, step, hi);
}

// The waves' partial tiles into LDS, then element `e` of this thread = the sum over the waves in order.
// Element id x = tile (i, j), register v, lane, as the MFMA leaves them.
template <int T, int TM, int TN, int NW>
__device__ __forceinline__ void put_partial(float* red, const Acc<T> (&acc)[TM / T][TN / T], int wave, int lane) {
  constexpr int R = T * T / 64;
#pragma unroll
  for (int i = 0; i < TM / T; ++i)
#pragma unroll
    for (int j = 0; j < TN / T; ++j)
#pragma unroll
      for (int v = 0; v < R; ++v) red[wave * TM * TN + ((i * (TN / T) + j) * R + v) * 64 + lane] = acc[i][j][v];
}
template <int TM, int TN, int NW> __device__ __forceinline__ float sum_partial(const float* red, int x) {
  float t = red[x];
#pragma unroll
  for (int w = 1; w < NW; ++w) t += red[w * TM * TN + x];
  return t;
}
template <int T, int TN> __device__ __forceinline__ void where(int x, int* m, int* n) {
  constexpr int R = T * T / 64;
  const int lane = x & 63, v = x / 64 % R, t = x / 64 / R;
  *m = (t / (TN / T)) * T + (v >> 2) * 8 + lane / T * 4 + (v & 3);
  *n = (t % (TN / T)) * T + lane % T;
}

template <int T, int TM, int TN, int NW, int ND, bool BKC, int MODE>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ B, int M,
                                                           int N, int K, long lda, long ldb, EpiParams epi) {
  __shared__ float red[NW * TM * TN];
  const int tiles_m = (M + TM - 1) / TM;
  const int m0 = ((int)blockIdx.x % tiles_m) * TM, n0 = ((int)blockIdx.x / tiles_m) * TN;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  Acc<T> acc[TM / T][TN / T];
  wave_tile<T, TM, TN, NW, ND, true, BKC>(acc, A, B, M, N, K, lda, ldb, m0, n0, wave, lane);
  put_partial<T, TM, TN, NW>(red, acc, wave, lane);
  __syncthreads();
#pragma unroll
  for (int e = 0; e < (TM * TN + 64 * NW - 1) / (64 * NW); ++e) {
    const int x = threadIdx.x + e * 64 * NW;
    if (x >= TM * TN) break;  // 16 x 16 tiles have fewer elements than threads
    int m, n;
    where<T, TN>(x, &m, &n);
    if (m0 + m < M && n0 + n < N) epilogue_one<float, MODE>(epi, m0 + m, n0 + n, sum_partial<TM, TN, NW>(red, x));
  }
}

struct F32WgradTable {
  int nprob, ngroup, ntiles;
  int tile0[kWgradMaxProblems + 1];
  int strip0[kWgradMaxProblems + 1];  // 64-column strips of the bias gradients; equal entries: no bias
  int M[kWgradMaxProblems], N[kWgradMaxProblems];
  float* outf[kWgradMaxProblems];
  float* bias[kWgradMaxProblems];
  const float* a[kWgradMaxPairs];
  const float* b[kWgradMaxPairs];
};

// All gradients of a W pass in one launch: C += A_0^T B_0, then += A_1^T B_1, ...  (each pair's product is
// finished before it is added, so several pairs in one launch give the bits of one launch each), and the bias
// gradients (column sums of the B operands, rows in a fixed order) in the workgroups after the tiles.
template <int T, int TM, int TN, int NW, int ND>
__global__ __launch_bounds__(64 * NW) void gemm_f32_wgrad_kernel(F32WgradTable tb, int K) {
  __shared__ float red[NW * TM * TN];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int pid = blockIdx.x, q = 0;
  const bool strip = pid >= tb.ntiles;
  if (strip) pid -= tb.ntiles;
#pragma unroll
  for (int i = 1; i < kWgradMaxProblems; ++i) q += (i < tb.nprob && pid >= (strip ? tb.strip0[i] : tb.tile0[i])) ? 1 : 0;
  pid -= strip ? tb.strip0[q] : tb.tile0[q];
  const int M = tb.M[q], N = tb.N[q], ngroup = tb.ngroup;
  if (strip) {
    const int n = pid * 64 + lane;
    float run = wave == 0 && n < N ? tb.bias[q][n] : 0.f;
    for (int g = 0; g < ngroup; ++g) {
      const float* __restrict__ b = tb.b[q * ngroup + g] + min(n, N - 1);
      float t = 0.f;
#pragma unroll 8
      for (int r = wave; r < K; r += NW) t += b[(long)r * N];
      red[wave * 64 + lane] = t;
      __syncthreads();
      if (wave == 0) {
        float u = red[lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) u += red[w * 64 + lane];
        run += u;
      }
      __syncthreads();
    }
    if (wave == 0 && n < N) tb.bias[q][n] = run;
    return;
  }
  const int tiles_m = (M + TM - 1) / TM;
  const int m0 = (pid % tiles_m) * TM, n0 = (pid / tiles_m) * TN;
  constexpr int PER = TM * TN / (64 * NW);
  float c[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    int m, n;
    where<T, TN>(threadIdx.x + e * 64 * NW, &m, &n);
    c[e] = tb.outf[q][(size_t)min(m0 + m, M - 1) * N + min(n0 + n, N - 1)];
  }
  for (int g = 0; g < ngroup; ++g) {
    Acc<T> acc[TM / T][TN / T];
    wave_tile<T, TM, TN, NW, ND, false, false>(acc, tb.a[q * ngroup + g], tb.b[q * ngroup + g], M, N, K, M, N, m0, n0, wave, lane);
    put_partial<T, TM, TN, NW>(red, acc, wave, lane);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) c[e] += sum_partial<TM, TN, NW>(red, threadIdx.x + e * 64 * NW);
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    int m, n;
    where<T, TN>(threadIdx.x + e * 64 * NW, &m, &n);
    if (m0 + m < M && n0 + n < N) tb.outf[q][(size_t)(m0 + m) * N + n0 + n] = c[e];
  }
}

inline long tiles_of(int M, int N, int t) { return (long)((M + t - 1) / t) * ((N + t - 1) / t); }

// Forward / dgrad: 16 x 16 tiles up to half a 32 x 32 tile per CU, 64 x 64 tiles with four waves from eight of them on.
// Measured, us with 16 x 16 / 32 x 32 / 64 x 64 tiles, weights as stored (dgrad in brackets), tokens x N x K:
// 128 x 256 x 1024 (32 tiles of 32 x 32) 5.9 / 9.7 / 28 (5.8 / 10.4 / 28), 128 x 1024 x 256 (128) 3.7 / 4.2 / 11 (4.1 / 4.5 / 12),
// 512 x 256 x 1024 (128) 8.4 / 10.0 / 31 (9.3 / 10.5 / 29), 200 x 1024 x 256 (224) 5.3 / 4.3 / 12 (5.8 / 4.8 / 12), 512 x 1024 x 1024
// (512) 26 / 18 / 34 (31 / 23 / 33), 512 x 2048 x 512 (1024) 25 / 18 / 23 (32 / 20 / 22), 1024 x 1024 x 4096 (1024) 168 / 113 / 111
// (225 / 123 / 101), 1024 x 2048 x 512 (2048) 47 / 31 / 32 (60 / 35 / 31), 1024 x 4096 x 1024 (4096) 184 / 113 / 98 (227 / 128 / 94).
constexpr long kSmallTiles = 128, kWideTiles = 2048;

// W: 32 x 32 tiles with eight waves, or with four where they have at most one 32-k block each (the idle four of eight
// would only add zeros: the same bits) and the gradients fill half the chip.  Above that the two would add in different
// orders, so the choice may rest only on what is the same in every launch of a stage - the tokens and the largest gradient of a layer
// - and not on how many layers share the launch (nor may `valu_wgrad`): the gradients keep their bits in every grouping.
// Measured with the bias sums, us with eight waves / four / 64 x 64 tiles with four, hidden h, ffn 4 h, 128 tokens: h 128
// (largest gradient 64 tiles) one layer 4.2 / 4.3 / 7.9, four 7.6 / 6.7 / 8.2; h 192 (144) one 5.1 / 5.2 / 8.0, two 7.8 / 7.3 / 8.3; h 256
// (256) one 6.5 / 6.4 / 8.1, two 10.4 / 9.5 / 11.2, four 20 / 17 / 18; h 1024 60 / 51 / 55; 17 tokens: h 256, four 16 / 12 / 15, h 1024
// 46 / 31 / 50.  136 tokens: h 256, one 7.4 / 7.4 / 10.4.
inline long largest_tiles(const WgradMultiArgs& w) {
  long most = 0;
  for (int q = 0; q < w.nprob; ++q) most = std::max(most, tiles_of(w.M[q], w.N[q], 32));
  return most;
}
inline bool four_waves(const WgradMultiArgs& w) { return w.K <= 4 * KB && largest_tiles(w) >= 128; }

// Large gradients are bound by their own turn-around, and these tiles, whose waves wait for each other's partial sums,
// keep too few loads in flight for it: the vector-ALU kernel takes the products there, one launch each, and only the
// strips stay here.  Measured with the bias sums, us of one layer, matrix cores / vector ALUs (hidden h, ffn 4 h; the
// largest gradient is h^2 / 256 tiles): h 768 17 tokens 45 / 50, h 1024 17: 77 / 58, 64: 76 / 73, 128: 82 / 110, 136: 148 /
// 116, 220: 152 / 158 (four layers 668 / 628), 256: 153 / 180; h 1536 64: 160 / 124, 128: 172 / 187, 220: 335 / 286, 512: 523 /
// 580; h 2048 17: 277 / 128, 128: 304 / 253, 256: 600 / 440, 1024: 1607 / 1560.
inline bool valu_wgrad(const WgradMultiArgs& w) {
  const long most = largest_tiles(w);
  return most >= 16384 || (most >= 4096 && (w.K <= 64 || (w.K > 4 * KB && w.K < 224)));
}

template <bool BKC, int MODE> hipError_t run_f32(const GemmArgs& g, long lda, long ldb, hipStream_t s) {
  const long small = tiles_of(g.M, g.N, 32);
  if (small >= (1L << 31)) return hipErrorInvalidValue;
  const float *A = (const float*)g.A, *B = (const float*)g.B;
  const EpiParams epi = make_epi(g);
  if (small <= kSmallTiles)
    gemm_f32_kernel<16, 16, 16, 8, 4, BKC, MODE><<<(unsigned)tiles_of(g.M, g.N, 16), 512, 0, s>>>(A, B, g.M, g.N, g.K, lda, ldb, epi);
  else if (small < kWideTiles)
    gemm_f32_kernel<32, 32, 32, 8, 2, BKC, MODE><<<(unsigned)small, 512, 0, s>>>(A, B, g.M, g.N, g.K, lda, ldb, epi);
  else
    gemm_f32_kernel<32, 64, 64, 4, 1, BKC, MODE><<<(unsigned)tiles_of(g.M, g.N, 64), 256, 0, s>>>(A, B, g.M, g.N, g.K, lda, ldb, epi);
  return hipGetLastError();
}

template <bool BKC> hipError_t run_f32_mode(const GemmArgs& g, long lda, long ldb, hipStream_t s) {
  switch (g.epilogue) {
    case EPI_STORE: return run_f32<BKC, EPI_STORE>(g, lda, ldb, s);
    case EPI_BIAS: return run_f32<BKC, EPI_BIAS>(g, lda, ldb, s);
    case EPI_BIAS_RESID: return run_f32<BKC, EPI_BIAS_RESID>(g, lda, ldb, s);
    case EPI_BIAS_GELU: return run_f32<BKC, EPI_BIAS_GELU>(g, lda, ldb, s);
    case EPI_DGELU: return run_f32<BKC, EPI_DGELU>(g, lda, ldb, s);
  }
  return hipErrorInvalidValue;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

template <> hipError_t launch_wgrad_multi_mfma<float>(const WgradMultiArgs& w, hipStream_t s, bool* taken) {
  *taken = false;
  if (w.nprob < 1 || w.nprob > kWgradMaxProblems || w.ngroup < 1 || w.ngroup > kGemmGroupMax ||
      w.nprob * w.ngroup > kWgradMaxPairs || w.K <= 0)
    return hipSuccess;
  F32WgradTable tb{};
  tb.nprob = w.nprob;
  tb.ngroup = w.ngroup;
  long small = 0;
  for (int q = 0; q < w.nprob; ++q) {
    if (w.M[q] <= 0 || w.N[q] <= 0) return hipSuccess;
    small += tiles_of(w.M[q], w.N[q], 32);
  }
  if (small >= (1L << 30)) return hipSuccess;
  const bool valu = valu_wgrad(w), four = !valu && four_waves(w);
  int tiles = 0, strips = 0;
  for (int q = 0; q < w.nprob; ++q) {
    tb.M[q] = w.M[q]; tb.N[q] = w.N[q]; tb.outf[q] = w.outf[q];
    tb.bias[q] = w.bias_done ? w.bias[q] : nullptr;
    tb.tile0[q] = tiles;
    tb.strip0[q] = strips;
    if (!valu) tiles += (int)tiles_of(w.M[q], w.N[q], 32);
    if (tb.bias[q]) strips += (w.N[q] + 63) / 64;
    for (int g = 0; g < w.ngroup; ++g) {
      tb.a[q * w.ngroup + g] = (const float*)w.a[q * w.ngroup + g];
      tb.b[q * w.ngroup + g] = (const float*)w.b[q * w.ngroup + g];
    }
  }
  for (int q = w.nprob; q <= kWgradMaxProblems; ++q) { tb.tile0[q] = tiles; tb.strip0[q] = strips; }
  tb.ntiles = tiles;
  *taken = true;
  if (w.bias_done) *w.bias_done = true;
  if (valu)
    for (int i = 0; i < w.nprob * w.ngroup; ++i) {
      const int q = i / w.ngroup;
      GemmArgs g{};
      g.A = w.a[i]; g.B = w.b[i]; g.M = w.M[q]; g.N = w.N[q]; g.K = w.K;
      g.a_sm = 1; g.a_sk = g.M; g.b_sk = g.N; g.b_sn = 1; g.epilogue = EPI_ACCUM_F32; g.outf = w.outf[q];
      hipError_t e = launch_gemm_generic<float>(g, s);
      if (e != hipSuccess) return e;
    }
  if (tiles + strips == 0) return hipSuccess;
  if (four) gemm_f32_wgrad_kernel<32, 32, 32, 4, 1><<<tiles + strips, 256, 0, s>>>(tb, w.K);
  else gemm_f32_wgrad_kernel<32, 32, 32, 8, 2><<<tiles + strips, 512, 0, s>>>(tb, w.K);
  return hipGetLastError();
}

template <> hipError_t launch_gemm_mfma<float>(const GemmArgs& g, hipStream_t s, bool* taken) {
  *taken = false;
  if (g.epilogue == EPI_ACCUM_F32 || g.a_sk != 1) return hipSuccess;
  const long lda = g.a_sm;
  if (g.K % 4 != 0 || lda % 4 != 0 || !aligned16(g.A)) return hipSuccess;
  if (g.b_sn == 1 && g.b_sk != 1) {
    *taken = true;
    return run_f32_mode<false>(g, lda, g.b_sk, s);
  }
  if (g.b_sk == 1 && g.b_sn % 4 == 0 && aligned16(g.B)) {
    *taken = true;
    return run_f32_mode<true>(g, lda, g.b_sn, s);
  }
  return hipSuccess;
}

}  // namespace zb
