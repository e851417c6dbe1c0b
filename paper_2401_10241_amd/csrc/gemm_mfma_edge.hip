// bf16 GEMMs on the matrix cores for what the 256-column tiles of gemm_mfma.hip do not take or do not fill the
// chip with: any M, N and K that are multiples of 8 in their contiguous direction (forward / dgrad: K and N;
// wgrad: M and N, any number of tokens), and small products.
//
//   forward / dgrad  A [m][k] K-contiguous, B [k][n] row-contiguous, 64 k per step, tiles 128 x 128 (8 waves,
//                    2 x 4) or 64 x 64 (4 waves, 2 x 2), optionally cut into K slices
//   wgrad            both operands row-contiguous ([k][m], [k][n]), 32 k per step, tile 128 x 128 (4 waves), the
//                    accumulators start from the old gradient as in gemm_mfma.hip
//
// Tiles travel global memory -> LDS directly, five stages deep.  Nothing out of range is ever read: rows and
// columns past the edge are fetched from the last valid one (their products are never stored), and 16-byte
// chunks whose k lies past the end are fetched from a chunk of zeros, so that the last step adds exact zeros
// whatever the neighbouring memory holds (infinities and NaN included).  Which chunk a lane fetches also
// implements the LDS swizzle.
//
// What bounds them: at these sizes a GEMM is a chain of K / 64 steps on a chip that is filled once or less, so
// the latency of a step (barrier, LDS -> fragments, MFMA) times the number of steps is the time, and with two 64 x 64
// workgroups on a CU what it can fetch from L2 (about 100 GB/s); smaller tiles and K slices shorten the chain or use
// more CUs (the rule is at `kTiles` in gemm_mfma.hip).  The steps overlap as `ring_steps` says.  Measured (M x N x K with a bias
// epilogue, us per launch back to back; fragments read and used in the same step, 32x32x16 MFMAs -> now): 1024 x 2304 x 2304
// 25.7 -> 18.3, 512 x 2048 x 2048 13.7 -> 10.4, 256 x 3072 x 2048 12.8 -> 10.4, 777 x 3600 x 1200 17.1 -> 14.6, 1024 x 4096 x
// 4096 (256-column tiles and the launch that adds four slices) 49.0 -> 34.4; W of h 1200, 777 tokens, two layers 143 -> 117.
// A ring of seven or nine stages: the same or slower (256 x 3072 x 1024 7.3 -> 7.9 and 8.3).
#include "gemm_epilogue.h"
#include "gemm_lds.h"

namespace zb {

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

constexpr int ST = 5;  // LDS stages

// The steps of a chain.  While a step's NM MFMAs run, the NR fragments of the next one are read from LDS and the ND loads
// of the tile ST-1 ahead are issued, singly and in this order, so that a step is one barrier and its MFMAs: read and used
// in the same step, the fragments' way out of LDS and a chain of dependent MFMAs stood in the open (0.31 us per 64-k
// step of a 64 x 64 tile where the MFMAs take 0.06).
// read(it, r, f) fetches fragment r of step it, dma(t, d, guard) issues load d of tile t (tiles in order; guard: the tile
// may be past the end or cut by it), fetched() follows the last load of a tile, mma(f, e) is MFMA e.
template <int NM, int NR, int ND, class F, class R, class D, class FE, class MM>
__device__ __forceinline__ void ring_steps(int nk, F& f0, F& f1, R&& read, D&& dma, FE&& fetched, MM&& mma) {
  auto advance = [&](int it, bool guard, const F& cur, F& nxt) {
    // this wave's loads of tile it + 1 have landed (those of the ST-3 tiles after it may stay in flight)
    if (guard && it + ST - 2 >= nk) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 3) * ND));
    __builtin_amdgcn_s_barrier();  // everybody's; and everybody is done with tile it - 1, whose stage is refilled
#pragma unroll
    for (int e = 0; e < NM; ++e) {
      mma(cur, e);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (r * NM / NR == e) read(it + 1, r, nxt);
#pragma unroll
      for (int d = 0; d < ND; ++d)
        if ((d + 1) * NM / ND - 1 == e) dma(it + ST - 1, d, guard);
      __builtin_amdgcn_sched_barrier(0);
    }
    fetched();
  };
#pragma unroll
  for (int t = 0; t < ST - 1; ++t) {
#pragma unroll
    for (int d = 0; d < ND; ++d) dma(t, d, true);
    fetched();
  }
  if (nk >= ST - 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 2) * ND));
  else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int r = 0; r < NR; ++r) read(0, r, f0);
  int it = 0;
  for (; it + 1 < nk - ST; it += 2) {  // the tiles fetched meanwhile are whole
    advance(it, false, f0, f1);
    advance(it + 1, false, f1, f0);
  }
  for (; it + 2 < nk; it += 2) {
    advance(it, true, f0, f1);
    advance(it + 1, true, f1, f0);
  }
  if (it + 1 < nk) {
    advance(it, true, f0, f1);
    f0 = f1;
  }
#pragma unroll
  for (int e = 0; e < NM; ++e) mma(f0, e);
}

// epilogue_wave for a tile that the last row or column cuts: all reads of 8 rows first (from the last row where a row does
// not exist), or every row would wait for a read of its own behind the store before it
template <int MODE, int MT, int NT>
__device__ __forceinline__ void epilogue_edge(const EpiParams& e, int m0, int M, int n0, int N, int lane,
                                              const f32x4 (&acc)[MT][NT]) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int q = 0; q < NT / 2; ++q) {
      const f32x8 c = rows8(acc[i][2 * q], acc[i][2 * q + 1]);
      const int m = m0 + i * 16 + (lane >> 5) * 8, n = n0 + q * 32 + (lane & 31);
      if (n >= N) continue;
      size_t idx[8];
      float a[8];
#pragma unroll
      for (int v = 0; v < 8; ++v) idx[v] = (size_t)min(m + v, M - 1) * e.N + n;
      if (MODE == EPI_BIAS_RESID || MODE == EPI_DGELU) {
#pragma unroll
        for (int v = 0; v < 8; ++v) a[v] = to_f32(((const bf16_t*)e.aux)[idx[v]]);
      }
      const float b = MODE == EPI_BIAS || MODE == EPI_BIAS_RESID || MODE == EPI_BIAS_GELU ? e.bias[n] : 0.f;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        if (m + v >= M) continue;
        const float f = c[v] + b;
        if (MODE == EPI_PARTIAL) {
          e.outf[idx[v]] = c[v];
        } else if (MODE == EPI_DGELU) {
          ((bf16_t*)e.out0)[idx[v]] = (bf16_t)(c[v] * gelu_grad<bf16_t>(a[v]));
        } else {
          ((bf16_t*)e.out0)[idx[v]] = (bf16_t)(MODE == EPI_BIAS_RESID ? f + a[v] : f);
          if (MODE == EPI_BIAS_GELU) ((bf16_t*)e.out1)[idx[v]] = (bf16_t)gelu<bf16_t>(f);
        }
      }
    }
}

template <int BM, int BN, int NWM, int NWN, int MODE>
__global__ __launch_bounds__(64 * NWM * NWN) void gemm_edge_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                                  int M, int N, int K, long lda, long ldb, EpiParams epi,
                                                                  int slices) {
  constexpr int NW = NWM * NWN;
  constexpr int WM = BM / NWM, WN = BN / NWN, MT = WM / 16, NT = WN / 16;
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
    const int c = (lane % CPL) ^ swz16_tr<BN>(kb[j]);
    pb[j] = B + (long)kb[j] * ldb + min(n0 + c * 8, N - 8);
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = (K + 63) / 64;
  auto dma = [&](int t, int d, bool guard) {  // every tile before the last is whole
    if (guard && t >= nk) return;
    const int k0 = t * 64;
    if (d < LA) {
      const void* p = pa[d] + k0;
      if (guard && k0 + ka[d] >= K) p = &kZeroChunk;
      dma16(p, sA + (t % ST) * (BM * 64) + (d * NW + wave) * 512);
    } else {
      const int j = d - LA;
      const void* p = pb[j] + (long)k0 * ldb;
      if (guard && k0 + kb[j] >= K) p = &kZeroChunk;
      dma16(p, sB + (t % ST) * (BN * 64) + (j * NW + wave) * 512);
    }
  };
  struct Frags {
    bf16x8 a[2][MT], b[2][NT];  // of both halves of the 64 k
  } f0, f1;
  auto read = [&](int it, int r, Frags& f) {
    const int kk = r / (MT + NT), q = r % (MT + NT);  // columns first
    if (q < NT) f.b[kk][q] = frag16_tr<BN>(sB + (it % ST) * (BN * 64), wn + q * 16, kk * 32, lane);
    else f.a[kk][q - NT] = frag16_rows(sA + (it % ST) * (BM * 64), wm + (q - NT) * 16, kk, lane);
  };
  auto mma = [&](const Frags& f, int e) {
    const int kk = e / (MT * NT), i = e % (MT * NT) / NT, j = (i & 1) ? NT - 1 - e % NT : e % NT;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[kk][i], f.b[kk][j], acc[i][j], 0, 0, 0);
  };
  ring_steps<2 * MT * NT, 2 * (MT + NT), LA + LB>(nk, f0, f1, read, dma, [] {}, mma);

  if (m0 + wm + WM <= M && n0 + wn + WN <= N) epilogue_wave<MODE, MT, NT>(epi, m0 + wm, n0 + wn, lane, acc);
  else epilogue_edge<MODE, MT, NT>(epi, m0 + wm, M, n0 + wn, N, lane, acc);
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
  const int row = m0 + wm + (lane >> 5) * 8, col = n0 + wn + (lane & 31);  // this lane's first row and column (rows8)
  float* __restrict__ outf = tb.outf[q];

  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; j += 2) {  // rows and columns past the edge: some valid element, never stored
      const int n = min(col + j * 16, N - 1);
      f32x8 c;
#pragma unroll
      for (int v = 0; v < 8; ++v) c[v] = __builtin_nontemporal_load(outf + (size_t)min(row + i * 16 + v, M - 1) * N + n);
      from_rows8(c, &acc[i][j], &acc[i][j + 1]);
    }

  // run j of a tile: 4 k-lines of 16 chunks
  int kl[2];
  long oa[2], ob[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    kl[j] = (j * 4 + wave) * 4 + (lane >> 4);
    const int c = ((lane & 15) ^ swz16_tr<WT>(kl[j])) * 8;
    oa[j] = (long)kl[j] * M + min(m0 + c, M - 8);
    ob[j] = (long)kl[j] * N + min(n0 + c, N - 8);
  }
  const int spc = (Kc + WKS - 1) / WKS, nk = ngroup * spc;
  // the next tile to fetch: its operand pair, k offset and addresses
  int g_next = 0, k_next = 0;
  const bf16_t *a_next = tb.a[pair0], *b_next = tb.b[pair0];
  auto dma = [&](int t, int d, bool guard) {
    if (guard && t >= nk) return;
    const int j = d >> 1;
    const void* p = (d & 1) ? b_next + ob[j] : a_next + oa[j];
    if (k_next + kl[j] >= Kc) p = &kZeroChunk;  // a pair's last tile may be cut anywhere in the chain
    dma16(p, ((d & 1) ? sB : sA) + (t % ST) * (WT * WKS) + (j * 4 + wave) * 512);
  };
  auto fetched = [&]() {
    a_next += (long)WKS * M;
    b_next += (long)WKS * N;
    k_next += WKS;
    if (k_next >= Kc && ++g_next < ngroup) {
      k_next = 0;
      a_next = tb.a[pair0 + g_next];
      b_next = tb.b[pair0 + g_next];
    }
  };
  struct Frags {
    bf16x8 a[4], b[4];
  } f0, f1;
  auto read = [&](int it, int r, Frags& f) {
    if (r & 1) f.a[r >> 1] = frag16_tr<WT>(sA + (it % ST) * (WT * WKS), wm + (r >> 1) * 16, 0, lane);
    else f.b[r >> 1] = frag16_tr<WT>(sB + (it % ST) * (WT * WKS), wn + (r >> 1) * 16, 0, lane);
  };
  auto mma = [&](const Frags& f, int e) {
    const int i = e >> 2, j = (i & 1) ? 3 - (e & 3) : e & 3;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
  };
  ring_steps<16, 8, 4>(nk, f0, f1, read, dma, fetched, mma);

#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      const f32x8 c = rows8(acc[i][j], acc[i][j + 1]);
      const int n = col + j * 16;
      if (n >= N) continue;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const int m = row + i * 16 + v;
        if (m < M) __builtin_nontemporal_store(c[v], outf + (size_t)m * N + n);
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
  static_assert(smem <= 80 * 1024 && smem >= 16 * WT * sizeof(float), "two workgroups per CU; the strips' buffer fits");
  static bool attr_set = false;  // one device per process in this library
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_wgrad_edge_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  *taken = true;
  if (w.bias_done) *w.bias_done = true;
  gemm_wgrad_edge_kernel<<<(unsigned)(tiles + strips), 256, smem, s>>>(tb, w.K);
  return hipGetLastError();
}

}  // namespace zb
