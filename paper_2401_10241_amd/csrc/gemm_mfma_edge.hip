// bf16 GEMMs on the matrix cores for what the 256-column tiles of gemm_mfma.hip do not take or do not fill the
// chip with: any M, N and K that are multiples of 8 in their contiguous direction (forward / dgrad: K and N;
// wgrad: M and N, any number of tokens), and small products.
//
//   forward / dgrad  A [m][k] K-contiguous, B [k][n] row-contiguous, 64 k per step, tiles 128 x 128 (8 waves,
//                    2 x 4) or 64 x 64 (4 waves, 2 x 2), optionally cut into K slices
//   wgrad            both operands row-contiguous ([k][m], [k][n]), 32 k per step, tile 128 x 128 (4 waves), the
//                    accumulators start from the old gradient as in gemm_mfma.hip
//
// Tiles travel global memory -> LDS directly, four stages deep.  Nothing out of range is ever read: rows and
// columns past the edge are fetched from the last valid one (their products are never stored), and 16-byte
// chunks whose k lies past the end are fetched from a chunk of zeros, so that the last step adds exact zeros
// whatever the neighbouring memory holds (infinities and NaN included).  Which chunk a lane fetches also
// implements the LDS swizzle.
//
// What bounds them: at these sizes a GEMM is a chain of K / 64 steps on a chip that is filled once or less, so
// the latency of a step (global -> LDS -> fragments -> MFMA, with three later steps in flight) times the number
// of steps is the time; smaller tiles and K slices shorten the chain or use more CUs (the rule is at
// `edge_cost`).  Measured (M x N x K with a bias epilogue, us per launch back to back, the launch that adds K slices
// included; before: the vector ALUs or the 256-column tiles): 777 x 4808 x 1200 245 -> 26, 777 x 1200 x 4808 1041 -> 28,
// 777 x 1200 x 1200 264 -> 10, 256 x 1024 x 1024 15.6 -> 7.5, 512 x 768 x 3072 25.7 -> 12.9, 512 x 2048 x 2048 25.6 -> 13.6.
#include <type_traits>

#include "gemm_epilogue.h"
#include "gemm_lds.h"

namespace zb {

double split_cost(int M, int N, int slices, bool rides);

namespace {

__device__ const uint4 kZeroChunk = {0, 0, 0, 0};

// XCD-aware renumbering (ids go round the 8 XCDs) and bands of G tile rows, M fastest within a band
__device__ __forceinline__ void tile_of(int pid, int tiles_m, int tiles_n, int G, int* tm, int* tn) {
  const int band = pid / (G * tiles_n);
  const int rows = min(tiles_m - band * G, G);
  const int in = pid - band * G * tiles_n;
  *tm = band * G + in % rows;
  *tn = in / rows;
}
// Workgroup ids that share (id & 7) run on one XCD: XCD x gets the contiguous run of tiles that starts after
// those of the XCDs before it (the first nblk & 7 of them have one more).
__device__ __forceinline__ int xcd_run(int id, int nblk) {
  const int x = id & 7, per = nblk >> 3, rem = nblk & 7;
  return x * per + min(x, rem) + (id >> 3);
}

constexpr int ST = 4;  // LDS stages

// epilogue_tile for a tile that the last row cuts: all reads first (from the last row where a row does not exist), or
// every row would wait for a read of its own behind the store before it
template <int MODE>
__device__ __forceinline__ void epilogue_edge(const EpiParams& e, int m0, int M, int n, const f32x16& acc) {
  size_t idx[16];
  float a[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) idx[v] = (size_t)min(m0 + (v >> 2) * 8 + (v & 3), M - 1) * e.N + n;
  if (MODE == EPI_BIAS_RESID || MODE == EPI_DGELU) {
#pragma unroll
    for (int v = 0; v < 16; ++v) a[v] = to_f32(((const bf16_t*)e.aux)[idx[v]]);
  }
  const float b = MODE == EPI_BIAS || MODE == EPI_BIAS_RESID || MODE == EPI_BIAS_GELU ? e.bias[n] : 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    if (m0 + (v >> 2) * 8 + (v & 3) >= M) continue;
    const float f = acc[v] + b;
    if (MODE == EPI_PARTIAL) {
      e.outf[idx[v]] = acc[v];
    } else if (MODE == EPI_DGELU) {
      ((bf16_t*)e.out0)[idx[v]] = (bf16_t)(acc[v] * gelu_grad<bf16_t>(a[v]));
    } else {
      ((bf16_t*)e.out0)[idx[v]] = (bf16_t)(MODE == EPI_BIAS_RESID ? f + a[v] : f);
      if (MODE == EPI_BIAS_GELU) ((bf16_t*)e.out1)[idx[v]] = (bf16_t)gelu<bf16_t>(f);
    }
  }
}

template <int BM, int BN, int NWM, int NWN, int MODE>
__global__ __launch_bounds__(64 * NWM * NWN) void gemm_edge_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                                  int M, int N, int K, long lda, long ldb, EpiParams epi,
                                                                  int slices) {
  constexpr int NW = NWM * NWN;
  constexpr int WM = BM / NWM, WN = BN / NWN, MT = WM / 32, NT = WN / 32;
  constexpr int LA = BM / 8 / NW;        // 1 KB runs (8 rows of 64 k) per wave per A tile
  constexpr int CPL = BN / 8, LPB = 64 / CPL;  // chunks per k-line of B, k-lines per run
  constexpr int LB = 64 / LPB / NW;
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* sA = reinterpret_cast<bf16_t*>(smem_raw);
  bf16_t* sB = sA + ST * BM * 64;

  int pid = xcd_run(blockIdx.x, gridDim.x);
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  if constexpr (MODE == EPI_PARTIAL) {  // slice s of the K range (whole 64-k blocks) goes to plane s
    const int slice = pid / (tiles_m * tiles_n);
    pid -= slice * tiles_m * tiles_n;
    const int blocks64 = (K + 63) / 64, per = (blocks64 + slices - 1) / slices;
    const int k0 = slice * per * 64;
    A += k0;
    B += (long)k0 * ldb;
    K = min(K - k0, per * 64);
    epi.outf += (size_t)slice * M * N;
  }
  int tm, tn;
  tile_of(pid, tiles_m, tiles_n, 8, &tm, &tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = (wave / NWN) * WM, wn = (wave % NWN) * WN;

  const bf16_t* pa[LA];  // this lane's chunk of each run, at k = 0
  int ka[LA];
  const bf16_t* pb[LB];
  int kb[LB];
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const int r = (j * NW + wave) * 8 + (lane >> 3);
    ka[j] = ((lane & 7) ^ ((r >> 1) & 7)) << 3;
    pa[j] = A + (long)min(m0 + r, M - 1) * lda + ka[j];
  }
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    kb[j] = (j * NW + wave) * LPB + lane / CPL;
    const int c = (lane % CPL) ^ swz_tr<BN>(kb[j]);
    pb[j] = B + (long)kb[j] * ldb + min(n0 + c * 8, N - 8);
  }

  f32x16 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int nk = (K + 63) / 64;
  auto issue = [&](int t) {  // tile t into its stage; every k-block before the last is whole
    if (t >= nk) return;
    bf16_t* a_s = sA + (t % ST) * (BM * 64);
    bf16_t* b_s = sB + (t % ST) * (BN * 64);
    const int k0 = t * 64;
    const bool whole = k0 + 64 <= K;
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      const void* p = pa[j] + k0;
      if (!whole && k0 + ka[j] >= K) p = &kZeroChunk;
      dma16(p, a_s + (j * NW + wave) * 512);
    }
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      const void* p = pb[j] + (long)k0 * ldb;
      if (!whole && k0 + kb[j] >= K) p = &kZeroChunk;
      dma16(p, b_s + (j * NW + wave) * 512);
    }
  };
#pragma unroll
  for (int t = 0; t < ST - 1; ++t) issue(t);
  for (int it = 0; it < nk; ++it) {
    // this wave's loads of tile `it` have landed (those of the ST-2 tiles after it may stay in flight)
    if (it + ST - 2 < nk) __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 2) * (LA + LB)));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_barrier();
    const bf16_t* a_s = sA + (it % ST) * (BM * 64);
    const bf16_t* b_s = sB + (it % ST) * (BN * 64);
    bf16x8 af[4][MT], bf[4][NT];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
      for (int i = 0; i < MT; ++i) af[kk][i] = frag_rows(a_s, wm + i * 32, kk, lane);
#pragma unroll
      for (int j = 0; j < NT; ++j) bf[kk][j] = frag_tr<BN>(b_s, wn + j * 32, kk * 16, lane);
    }
    issue(it + ST - 1);  // into the stage that step it-1 read
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk][i], bf[kk][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this stage's reads are done before the next barrier
  }

  const int lrow = lane & 31, lhi = (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int mb = m0 + wm + i * 32, nb = n0 + wn + j * 32;
      if (mb + 32 <= M && nb + 32 <= N) {
        epilogue_tile<bf16_t, MODE>(epi, mb + lhi, nb + lrow, acc[i][j]);
      } else if (nb + lrow < N) {
        epilogue_edge<MODE>(epi, mb + lhi, M, nb + lrow, acc[i][j]);
      }
    }
}

template <int BM, int BN, int NWM, int NWN, int MODE>
hipError_t run_edge(const GemmArgs& g, long lda, long ldb, hipStream_t s, int slices) {
  auto kern = gemm_edge_kernel<BM, BN, NWM, NWN, MODE>;
  constexpr size_t smem = (size_t)ST * (BM + BN) * 64 * sizeof(bf16_t);
  static_assert(smem <= 160 * 1024, "LDS budget");
  static bool attr_set = false;  // one device per process in this library
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const long tiles = (long)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  if (tiles * slices >= (1L << 31)) return hipErrorInvalidValue;
  kern<<<(unsigned)(tiles * slices), 64 * NWM * NWN, smem, s>>>((const bf16_t*)g.A, (const bf16_t*)g.B, g.M, g.N, g.K, lda,
                                                               ldb, make_epi(g), slices);
  return hipGetLastError();
}

template <int MODE> hipError_t run_edge_tile(const GemmArgs& g, long lda, long ldb, hipStream_t s, int tile, int slices) {
  return tile == 128 ? run_edge<128, 128, 2, 4, MODE>(g, lda, ldb, s, slices)
                     : run_edge<64, 64, 2, 2, MODE>(g, lda, ldb, s, slices);
}

}  // namespace

// Microseconds the kernel above is expected to take with this tile and number of K slices, the launch that adds
// the planes included (`rides`: a LayerNorm that has to run anyway does it).  Fitted to single launches: a step of 64 k
// takes 0.31 us with one 64 x 64 workgroup per CU and 0.44 with two (0.57 and 0.79 for a 128 x 128 tile on a
// nearly empty and on a full chip), 3 us go to the start, the fill of the ring and the epilogue.  Against 39 shapes from
// 1 x 64 x 72 to 6144 x 2304 x 2304, 76 unsliced points: -20 to +15 %, but for three products under 12 us (100 x 96 x 96,
// 1 x 64 x 72, 333 x 264 x 520: up to 59 % short).  218 sliced points: 43 more than 20 % short, up to 42 % (512 x 3072 x 768 in
// four slices: 7.0 against 12.1; the planes' stores are not in the step), so slices are taken a little too readily.
double edge_cost(int M, int N, int K, int tile, int slices, bool rides) {
  const long tiles = (long)((M + tile - 1) / tile) * ((N + tile - 1) / tile) * slices;
  const int steps = ((K + 63) / 64 + slices - 1) / slices;
  const long at_once = tile == 128 ? 256 : 512;
  const double full = tile == 128 ? 0.79 : 0.44, empty = tile == 128 ? 0.57 : 0.31;
  const long rounds = tiles / at_once, rest = tiles % at_once;
  double us = 3.0 + steps * full * rounds;
  if (rest) us += steps * (empty + (full - empty) * rest / at_once);
  if (slices > 1) us += split_cost(M, N, slices, rides);
  return us;
}

// Cheapest tile and number of K slices (within the workspace); 512 x 768 x 3072: 17.9 us whole, 8.3 in four slices and
// 4.6 for the launch that adds them (25.7 on the 256-column tiles).
void choose_edge(int M, int N, int K, size_t workspace_floats, bool rides, int* tile, int* slices, double* us) {
  *us = 1e30;
  const int blocks = (K + 63) / 64;
  for (int t = 64; t <= 128; t += 64)
    for (int sl = 1; sl <= 4; ++sl) {
      if (sl > 1 && (size_t)sl * M * N > workspace_floats) break;
      const int per = (blocks + sl - 1) / sl;
      if ((sl - 1) * per >= blocks) continue;  // an empty slice
      const double c = edge_cost(M, N, K, t, sl, rides);
      if (c < *us) { *us = c; *tile = t; *slices = sl; }
    }
}

// Microseconds that cutting a product into K slices adds: the planes are read back at about 4 TB/s, by a launch of
// its own unless a LayerNorm that runs anyway takes it over.
double split_cost(int M, int N, int slices, bool rides) { return (rides ? 0.0 : 4.5) + (double)slices * M * N * 1e-6; }

// forward / dgrad GEMM with the given tile (128 or 64); slices > 1: the K slices' planes only (g.outf)
hipError_t launch_gemm_edge(const GemmArgs& g, long lda, long ldb, int tile, int slices, hipStream_t s) {
  switch (g.epilogue) {
    case EPI_STORE: return run_edge_tile<EPI_STORE>(g, lda, ldb, s, tile, 1);
    case EPI_BIAS: return run_edge_tile<EPI_BIAS>(g, lda, ldb, s, tile, 1);
    case EPI_BIAS_RESID: return run_edge_tile<EPI_BIAS_RESID>(g, lda, ldb, s, tile, 1);
    case EPI_BIAS_GELU: return run_edge_tile<EPI_BIAS_GELU>(g, lda, ldb, s, tile, 1);
    case EPI_DGELU: return run_edge_tile<EPI_DGELU>(g, lda, ldb, s, tile, 1);
    case EPI_PARTIAL: return run_edge_tile<EPI_PARTIAL>(g, lda, ldb, s, tile, slices);
  }
  return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------------------
// wgrad
// ------------------------------------------------------------------------------------------------
namespace {

constexpr int WT = 128;   // tile rows and columns
constexpr int WKS = 32;   // k per step

struct EdgeWgradTable {
  int nprob, ngroup;
  int tile0[kWgradMaxProblems + 1];
  int M[kWgradMaxProblems], N[kWgradMaxProblems];
  float* outf[kWgradMaxProblems];
  const bf16_t* a[kWgradMaxPairs];
  const bf16_t* b[kWgradMaxPairs];
  int ntiles;
  int strip0[kWgradMaxProblems + 1];
  float* bias[kWgradMaxProblems];
};

// Bias gradient of one 128-column strip: 256 threads = 16 chunks of 8 columns x 16 row groups, every sum in a
// fixed order, pair by pair onto the running value (one launch of several pairs gives the bits of one each).
__device__ __forceinline__ void edge_bias_strip(const EdgeWgradTable& tb, int sid, int Kc, float* red) {
  int q = 0;
#pragma unroll
  for (int i = 1; i < kWgradMaxProblems; ++i) q += (i < tb.nprob && sid >= tb.strip0[i]) ? 1 : 0;
  sid -= tb.strip0[q];
  const int N = tb.N[q], ngroup = tb.ngroup;
  const int n0 = sid * WT;
  const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
  const bool in = n0 + c * 8 < N;
  float* __restrict__ bias = tb.bias[q];
  const int col = n0 + threadIdx.x;
  const bool own = threadIdx.x < WT && col < N;
  float run = own ? bias[col] : 0.f;
  for (int gi = 0; gi < ngroup; ++gi) {
    const bf16_t* __restrict__ b = tb.b[q * ngroup + gi] + n0 + c * 8;
    float sum[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) sum[j] = 0.f;
    if (in) {
#pragma unroll 8
      for (int r = g; r < Kc; r += 16) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(b + (long)r * N);
#pragma unroll
        for (int j = 0; j < 8; ++j) sum[j] += (float)v[j];
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[g * WT + c * 8 + j] = sum[j];
    __syncthreads();
    if (own) {
      float t = 0.f;
#pragma unroll
      for (int gg = 0; gg < 16; ++gg) t += red[gg * WT + threadIdx.x];
      run += t;
    }
    __syncthreads();
  }
  if (own) bias[col] = run;
}

__global__ __launch_bounds__(256, 2) void gemm_wgrad_edge_kernel(EdgeWgradTable tb, int Kc) {
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* sA = reinterpret_cast<bf16_t*>(smem_raw);
  bf16_t* sB = sA + ST * WT * WKS;
  const int nblk = tb.ntiles;
  if ((int)blockIdx.x >= nblk) {
    edge_bias_strip(tb, blockIdx.x - nblk, Kc, reinterpret_cast<float*>(smem_raw));
    return;
  }
  int pid = xcd_run(blockIdx.x, nblk);
  int q = 0;
#pragma unroll
  for (int i = 1; i < kWgradMaxProblems; ++i) q += (i < tb.nprob && pid >= tb.tile0[i]) ? 1 : 0;
  pid -= tb.tile0[q];
  const int M = tb.M[q], N = tb.N[q], ngroup = tb.ngroup, pair0 = q * ngroup;
  int tm, tn;
  tile_of(pid, (M + WT - 1) / WT, (N + WT - 1) / WT, 4, &tm, &tn);
  const int m0 = tm * WT, n0 = tn * WT;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const int lrow = lane & 31, lhi = (lane >> 5) * 4;
  float* __restrict__ outf = tb.outf[q];

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {  // rows and columns past the edge: some valid element, never stored
      const int n = min(n0 + wn + j * 32 + lrow, N - 1);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = min(m0 + wm + i * 32 + lhi + (v >> 2) * 8 + (v & 3), M - 1);
        acc[i][j][v] = __builtin_nontemporal_load(outf + (size_t)m * N + n);
      }
    }

  // run j of a tile: 4 k-lines of 16 chunks
  int kl[2];
  long oa[2], ob[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    kl[j] = (j * 4 + wave) * 4 + (lane >> 4);
    const int c = ((lane & 15) ^ swz_tr<WT>(kl[j])) * 8;
    oa[j] = (long)kl[j] * M + min(m0 + c, M - 8);
    ob[j] = (long)kl[j] * N + min(n0 + c, N - 8);
  }
  const int spc = (Kc + WKS - 1) / WKS, nk = ngroup * spc;
  int g_next = 0, k_next = 0;
  auto issue = [&](int t) {  // tiles are fetched in order
    if (t >= nk) return;
    const bf16_t* pa = tb.a[pair0 + g_next] + (long)k_next * M;
    const bf16_t* pb = tb.b[pair0 + g_next] + (long)k_next * N;
    bf16_t* a_s = sA + (t % ST) * (WT * WKS);
    bf16_t* b_s = sB + (t % ST) * (WT * WKS);
    const bool whole = k_next + WKS <= Kc;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bool out = !whole && k_next + kl[j] >= Kc;
      const void* p = pa + oa[j];
      const void* r = pb + ob[j];
      if (out) p = r = &kZeroChunk;
      dma16(p, a_s + (j * 4 + wave) * 512);
      dma16(r, b_s + (j * 4 + wave) * 512);
    }
    k_next += WKS;
    if (k_next >= Kc) { k_next = 0; ++g_next; }
  };
#pragma unroll
  for (int t = 0; t < ST - 1; ++t) issue(t);
  for (int it = 0; it < nk; ++it) {
    if (it + ST - 2 < nk) __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 2) * 4));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_barrier();
    const bf16_t* a_s = sA + (it % ST) * (WT * WKS);
    const bf16_t* b_s = sB + (it % ST) * (WT * WKS);
    bf16x8 af[2][2], bf[2][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[kk][i] = frag_tr<WT>(a_s, wm + i * 32, kk * 16, lane);
        bf[kk][i] = frag_tr<WT>(b_s, wn + i * 32, kk * 16, lane);
      }
    issue(it + ST - 1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk][i], bf[kk][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_waitcnt(0xC07F);
  }

#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + wn + j * 32 + lrow, mb = m0 + wm + i * 32 + lhi;
      if (n < N) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = mb + (v >> 2) * 8 + (v & 3);
          if (m < M) __builtin_nontemporal_store(acc[i][j][v], outf + (size_t)m * N + n);
        }
      }
    }
}

}  // namespace

// The gradients of one W pass whose sizes the 256-column tiles do not take; *taken stays false where a width is
// no multiple of 8 or an operand is not 16-byte aligned.
hipError_t launch_wgrad_multi_edge(const WgradMultiArgs& w, hipStream_t s, bool* taken) {
  *taken = false;
  EdgeWgradTable tb{};
  tb.nprob = w.nprob;
  tb.ngroup = w.ngroup;
  long tiles = 0;
  int strips = 0;
  for (int q = 0; q < w.nprob; ++q) {
    const int M = w.M[q], N = w.N[q];
    if (M <= 0 || N <= 0 || M % 8 != 0 || N % 8 != 0) return hipSuccess;
    tb.M[q] = M; tb.N[q] = N; tb.outf[q] = w.outf[q];
    tb.bias[q] = w.bias_done ? w.bias[q] : nullptr;
    tb.tile0[q] = (int)tiles;
    tb.strip0[q] = strips;
    tiles += (long)((M + WT - 1) / WT) * ((N + WT - 1) / WT);
    if (tiles >= (1L << 30)) return hipSuccess;
    if (tb.bias[q]) strips += (N + WT - 1) / WT;
    for (int g = 0; g < w.ngroup; ++g) {
      const void* a = w.a[q * w.ngroup + g];
      const void* b = w.b[q * w.ngroup + g];
      if (!a || !b || !aligned16(a) || !aligned16(b)) return hipSuccess;
      tb.a[q * w.ngroup + g] = (const bf16_t*)a;
      tb.b[q * w.ngroup + g] = (const bf16_t*)b;
    }
  }
  for (int q = w.nprob; q <= kWgradMaxProblems; ++q) { tb.tile0[q] = (int)tiles; tb.strip0[q] = strips; }
  tb.ntiles = (int)tiles;
  constexpr size_t smem = (size_t)ST * 2 * WT * WKS * sizeof(bf16_t);
  static_assert(smem <= 64 * 1024 && smem >= 16 * WT * sizeof(float), "no attribute needed; the strips' buffer fits");
  *taken = true;
  if (w.bias_done) *w.bias_done = true;
  gemm_wgrad_edge_kernel<<<(unsigned)(tiles + strips), 256, smem, s>>>(tb, w.K);
  return hipGetLastError();
}

}  // namespace zb
