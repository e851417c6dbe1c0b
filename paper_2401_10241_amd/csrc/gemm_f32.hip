// fp32 GEMMs on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and sums, nothing rounded below fp32),
// all three operand forms: forward X*W, dgrad dY*W^T (W as stored, K-contiguous), wgrad X^T*dY.
//
// A workgroup owns one output tile and its waves split K between them, 32 k at a time in turn; fragments come
// straight from memory into registers (one block of 32 k ahead), and the waves' partial tiles are added through
// LDS in wave order.  What bounds the products that come here (hundreds of tokens, widths up to a few thousand)
// is latency: with the K range walked in steps of 16 through LDS by a 64 x 64 tile, 128 x 256 x 1024 took 64
// dependent steps on 8 CUs; here it is 4 on 32.  Tiles are 32 x 32 with eight waves or 64 x 64 with four (half the
// reads per product, twice the chain); the rules are at `kWideTiles` and `wide_wgrad`.  Measured on
// the stage of hidden 256 with 128 tokens: N = 256 products 103-111 us -> 10-15 us, a W pass 215 us in eight
// launches plus column sums -> 17 us in one, the iteration 4.97 -> 1.09 ms.
#include <algorithm>

#include "gemm_epilogue.h"

namespace zb {

template <typename T> hipError_t launch_gemm_mfma(const GemmArgs& g, hipStream_t s, bool* taken);
template <typename T> hipError_t launch_wgrad_multi_mfma(const WgradMultiArgs& w, hipStream_t s, bool* taken);
template <typename T> hipError_t launch_gemm_generic(const GemmArgs& g, hipStream_t s);

namespace {

constexpr int KB = 32;  // k per block

// One operand's rows (or columns) r0 + (lane & 31), k0 .. k0+31: element 4q + j is k = k0 + 8q + 4 (lane >> 5) + j.
// KC: element (r, k) at p[r * ld + k], K and ld multiples of 4; else at p[k * ld + r].  k >= K: zero.
template <bool KC>
__device__ __forceinline__ void load_frag(f32x4 (&f)[4], const float* __restrict__ p, long ld, int r, int k0, int K, int hi) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = k0 + q * 8 + hi * 4;
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

// This wave's share of the tile at (m0, n0)
template <int TM, int TN, int NW, bool AKC, bool BKC>
__device__ __forceinline__ void wave_tile(f32x16 (&acc)[TM / 32][TN / 32], const float* __restrict__ A,
                                          const float* __restrict__ B, int M, int N, int K, long lda, long ldb, int m0,
                                          int n0, int wave, int lane) {
  constexpr int MT = TM / 32, NT = TN / 32;
  const int hi = lane >> 5;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  f32x4 a[MT][4], b[NT][4];
  auto load = [&](f32x4 (&x)[MT][4], f32x4 (&y)[NT][4], int k0) {
#pragma unroll
    for (int i = 0; i < MT; ++i) load_frag<AKC>(x[i], A, lda, min(m0 + i * 32 + (lane & 31), M - 1), k0, K, hi);
#pragma unroll
    for (int j = 0; j < NT; ++j) load_frag<BKC>(y[j], B, ldb, min(n0 + j * 32 + (lane & 31), N - 1), k0, K, hi);
  };
  int k0 = wave * KB;
  if (k0 < K) load(a, b, k0);
  for (; k0 < K; k0 += NW * KB) {
    f32x4 a1[MT][4], b1[NT][4];
    const bool more = k0 + NW * KB < K;
    if (more) load(a1, b1, k0 + NW * KB);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][q][e], b[j][q][e], acc[i][j], 0, 0, 0);
    if (more) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int i = 0; i < MT; ++i) a[i][q] = a1[i][q];
#pragma unroll
        for (int j = 0; j < NT; ++j) b[j][q] = b1[j][q];
      }
    }
  }
}

// The waves' partial tiles into LDS, then element `e` of this thread = the sum over the waves in order.
// Element id x = tile (i, j), register v, lane, as the MFMA leaves them.
template <int TM, int TN, int NW>
__device__ __forceinline__ void put_partial(float* red, const f32x16 (&acc)[TM / 32][TN / 32], int wave, int lane) {
#pragma unroll
  for (int i = 0; i < TM / 32; ++i)
#pragma unroll
    for (int j = 0; j < TN / 32; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[wave * TM * TN + ((i * (TN / 32) + j) * 16 + v) * 64 + lane] = acc[i][j][v];
}
template <int TM, int TN, int NW> __device__ __forceinline__ float sum_partial(const float* red, int x) {
  float t = red[x];
#pragma unroll
  for (int w = 1; w < NW; ++w) t += red[w * TM * TN + x];
  return t;
}
template <int TN> __device__ __forceinline__ void where(int x, int* m, int* n) {
  const int lane = x & 63, v = (x >> 6) & 15, t = x >> 10;
  *m = (t / (TN / 32)) * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
  *n = (t % (TN / 32)) * 32 + (lane & 31);
}

template <int TM, int TN, int NW, bool BKC, int MODE>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ B, int M,
                                                           int N, int K, long lda, long ldb, EpiParams epi) {
  __shared__ float red[NW * TM * TN];
  const int tiles_m = (M + TM - 1) / TM;
  const int m0 = ((int)blockIdx.x % tiles_m) * TM, n0 = ((int)blockIdx.x / tiles_m) * TN;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  f32x16 acc[TM / 32][TN / 32];
  wave_tile<TM, TN, NW, true, BKC>(acc, A, B, M, N, K, lda, ldb, m0, n0, wave, lane);
  put_partial<TM, TN, NW>(red, acc, wave, lane);
  __syncthreads();
#pragma unroll
  for (int e = 0; e < TM * TN / (64 * NW); ++e) {
    const int x = threadIdx.x + e * 64 * NW;
    int m, n;
    where<TN>(x, &m, &n);
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
template <int TM, int TN, int NW>
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
    where<TN>(threadIdx.x + e * 64 * NW, &m, &n);
    c[e] = tb.outf[q][(size_t)min(m0 + m, M - 1) * N + min(n0 + n, N - 1)];
  }
  for (int g = 0; g < ngroup; ++g) {
    f32x16 acc[TM / 32][TN / 32];
    wave_tile<TM, TN, NW, false, false>(acc, tb.a[q * ngroup + g], tb.b[q * ngroup + g], M, N, K, M, N, m0, n0, wave, lane);
    put_partial<TM, TN, NW>(red, acc, wave, lane);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) c[e] += sum_partial<TM, TN, NW>(red, threadIdx.x + e * 64 * NW);
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    int m, n;
    where<TN>(threadIdx.x + e * 64 * NW, &m, &n);
    if (m0 + m < M && n0 + n < N) tb.outf[q][(size_t)(m0 + m) * N + n0 + n] = c[e];
  }
}

inline long tiles_of(int M, int N, int t) { return (long)((M + t - 1) / t) * ((N + t - 1) / t); }

// Forward / dgrad: 64 x 64 tiles with four waves from four 32 x 32 tiles per CU on.  Measured, us with 32 x 32 / 64 x 64
// tiles: 512 x 1024 x 256 (512 tiles) 7.6 / 10.5, 512 x 1536 x 512 (768) 20.9 / 16.5, 512 x 2048 x 512 (1024) 29.2 /
// 18.6, 600 x 2048 x 512 (1216) 36.8 / 29.3, its dgrad 28.3 / 32.8, 1024 x 4096 x 1024 (4096) 220 / 98.
constexpr long kWideTiles = 1024;

// W: the two forms split K over eight and four waves, i.e. add in different orders, so the choice may rest only on what
// is the same in every launch of a stage - the tokens and the largest gradient of a layer - and not on how many layers
// share the launch (nor may `valu_wgrad`): the gradients keep their bits in every grouping.  The wide form pays with at most one 32-k block
// per wave and gradients that fill half the chip.  Measured, us with 32 x 32 / 64 x 64 tiles, hidden h, ffn 4 h: 128 tokens
// h 128 (largest gradient 64 tiles of 32 x 32) one layer 4.4 / 8.3, four 12.8 / 8.8; h 192 (144) one 6.9 / 8.5, two 12.7 / 8.9;
// h 256 (256) one 10.9 / 8.7, four 41 / 27; h 1024 128 / 88; h 256, two layers 64 tokens 18.7 / 15.4, 136 tokens 23.6 / 26.4,
// 512 tokens 39 / 104; h 1024, 512 tokens 256 / 531.
inline long largest_tiles(const WgradMultiArgs& w) {
  long most = 0;
  for (int q = 0; q < w.nprob; ++q) most = std::max(most, tiles_of(w.M[q], w.N[q], 32));
  return most;
}
inline bool wide_wgrad(const WgradMultiArgs& w) { return w.K <= 4 * KB && largest_tiles(w) >= 128; }

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
  if (small < kWideTiles)
    gemm_f32_kernel<32, 32, 8, BKC, MODE><<<(unsigned)small, 512, 0, s>>>(A, B, g.M, g.N, g.K, lda, ldb, make_epi(g));
  else
    gemm_f32_kernel<64, 64, 4, BKC, MODE><<<(unsigned)tiles_of(g.M, g.N, 64), 256, 0, s>>>(A, B, g.M, g.N, g.K, lda, ldb,
                                                                                          make_epi(g));
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
  const bool valu = valu_wgrad(w), wide = !valu && wide_wgrad(w);
  int tiles = 0, strips = 0;
  for (int q = 0; q < w.nprob; ++q) {
    tb.M[q] = w.M[q]; tb.N[q] = w.N[q]; tb.outf[q] = w.outf[q];
    tb.bias[q] = w.bias_done ? w.bias[q] : nullptr;
    tb.tile0[q] = tiles;
    tb.strip0[q] = strips;
    if (!valu) tiles += (int)tiles_of(w.M[q], w.N[q], wide ? 64 : 32);
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
  if (wide) gemm_f32_wgrad_kernel<64, 64, 4><<<tiles + strips, 256, 0, s>>>(tb, w.K);
  else gemm_f32_wgrad_kernel<32, 32, 8><<<tiles + strips, 512, 0, s>>>(tb, w.K);
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
