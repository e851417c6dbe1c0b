// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulation.
//
//   C[M,N] (epilogue)= A * B, with B always given "row-contiguous" ([k][n] in memory, n contiguous: the
//   weight W[in][out] in the forward GEMM, the transposed weight copy in the dgrad GEMM, dY in the wgrad
//   GEMM) and A either K-contiguous ([m][k]: activations in forward / dgrad) or row-contiguous ([k][m]:
//   the stashed layer input in wgrad).
//
// The wgrad GEMM (both operands row-contiguous, fp32 accumulate into C) has a kernel of its own below.
//
// One 512-thread workgroup (8 wavefronts, 2 x 4) owns a BM x 256 output tile (BM = 256 or 128) and walks K
// in steps of 32.  Tiles travel global memory -> LDS directly (global_load_lds_dwordx4: each lane's 16
// bytes land at consecutive LDS addresses, no registers in between) into rings of LDS stages, several
// steps ahead of the MFMAs.  Per step: wait until this wave's loads of the current tiles have landed
// (s_waitcnt vmcnt with the number of younger loads that may stay in flight), one barrier (all waves'
// loads landed, all waves done with the stage about to be refilled), then the step's MFMAs in two halves; between
// them, one at a time, stand the fragment reads of the half step to come and the loads for the step BS-1 ahead.
//
// What bounds the loop, and why it looks like this:
//   - Per step the matrix pipe takes 1024 cycles and the 32 load instructions 512 cycles of the load unit.  Issued in a
//     block (after the barrier or before it) the loads hold up the MFMAs behind them: in a probe of loads and MFMAs alone a
//     step took 1475 (loads first) and 1385 cycles (last), 1220 with a load after every fourth MFMA.
//   - On real operands the chip lowers its clock under the power of the matrix cores.  16x16x32 instructions, each
//     sharing an operand with the one before it, sustain 2.00-2.08 PFLOP/s on N(0,1) operands where 32x32x16 ones
//     sustain 1.79-1.82 (both 2.4 on zeros), and give the same bits.
// Before -> after on one box, N(0,1) operands: 1024 x 15360 x 5120 194 -> 175 us, 6144 x 6912 x 2304 209 -> 187, 6144 x
// 2304 x 9216 258 -> 227; W of h 5120, 1024 tokens 963 -> 896, of h 4096 in pairs 994 -> 888, of h 2304, 6144 tokens,
// three layers 2506 -> 2209.  All zeros: 1024 x 15360 x 5120 126 -> 121, 6144 x 2304 x 9216 188 -> 165.
//
// LDS layouts (no padding: the DMA writes 1 KB runs; bank conflicts are avoided by choosing WHICH global
// chunk each lane fetches).  The LDS has 64 banks of 4 bytes; 16-byte accesses go 16 lanes at a time,
// 8-byte accesses 32 lanes at a time.
//   row-contiguous source: ring of BS stages of [32 k][R]; chunk c (16 B) of k-line k sits at position
//     c ^ swz16_tr(k).  Read back with the transposing LDS load ds_read_b64_tr_b16 (frag16_tr): within 16 lanes,
//     lane a points at 4 consecutive rows (a & 3) * 4 of k-line (a >> 2) and receives, as lane r, the 4 k
//     values of row r.
//   K-contiguous source: 64 k at a time (128-byte rows, so every fetched cache line is used whole), two or
//     three stages of [BM][64]; chunk c of row r sits at position
//     c ^ ((r >> 1) & 7): 16 consecutive rows reading the same k cover all banks.
//
// Ring shape for the 256-row tile: 3 A stages (96 KB) + 4 B stages (64 KB) = the whole 160 KB; A is fetched four and
// three steps ahead (half a stage on each step, so that every step issues four loads per wave) and B three.
//
// MFMA 16x16x32 operand layout: lane l supplies row (l & 15) of its operand and the 8 consecutive k
// starting at 8 * (l >> 4); it receives column (l & 15) and rows 4 * (l >> 4) + v of the 16 x 16 result in accumulator
// element v.
#include "gemm_epilogue.h"
#include "gemm_lds.h"

namespace zb {

// gemm_mfma_edge.hip: other tiles for sizes that the 256-column tiles do not take or do not fill the chip with
hipError_t launch_gemm_edge(const GemmArgs& g, long lda, long ldb, int tile, int slices, hipStream_t s);
hipError_t launch_wgrad_multi_edge(const WgradMultiArgs& w, hipStream_t s, bool* taken);

namespace {

constexpr int KS = 32;   // k per pipeline step
constexpr int BN = 256;
constexpr int NTHREADS = 512;
constexpr int WN = 64;   // wave tile columns
constexpr int LB = BN / 128;  // DMA instructions per wave per B tile

// Direct-to-LDS loads.  Every DMA instruction of a wave writes one 1 KB run of the tile (run index
// blk = j * 8 + wave); which 16-byte global chunk a lane fetches implements the LDS swizzle.  The address
// splits into a part that is the same for the whole wave (tile origin, k offset, run) and a per-lane byte
// offset that never changes during the kernel, so the wave-uniform part is scalar arithmetic and the
// lane offset one register per operand (`wave` must be a scalar: readfirstlane'd by the caller).
//
// [32 k][R] tile of a row-contiguous operand (element (k, r) at p[k*ld + r]): run blk holds k-lines
// blk*LPB .. +LPB-1, LPB = 1024 B / (2R B).
template <int R> __device__ __forceinline__ unsigned dma_tr_lane_off(long ld, int wave, int lane) {
  constexpr int CPL = R / 8, LPB = 64 / CPL;  // chunks per k-line, k-lines per run
  const int kl = lane / CPL;
  static_assert(R == 128 || R == 256, "a wave's runs must be a multiple of 16 k-lines apart, where the swizzle repeats");
  const int c = (lane % CPL) ^ swz16_tr<R>(wave * LPB + kl);
  return (unsigned)((kl * ld + c * 8) * (long)sizeof(bf16_t));
}
// run j of the tile whose first element (k0, r0) is *p0
template <int R>
__device__ __forceinline__ void dma_tr(const bf16_t* __restrict__ p0, long ld, unsigned lane_off, bf16_t* s, int wave, int j) {
  constexpr int LPB = 64 / (R / 8);
  const int blk = j * 8 + wave;
  dma16_at(p0 + (long)(blk * LPB) * ld, lane_off, s + blk * 512);
}
// [R][64 k] tile of a K-contiguous operand (element (r, k) at p[r*ld + k]): run blk holds rows blk*8 .. +7.
__device__ __forceinline__ unsigned dma_rows_lane_off(long ld, int wave, int lane) {
  const int rl = lane >> 3;
  const int c = (lane & 7) ^ ((((wave & 1) << 2) | (lane >> 4)) & 7);  // ((r >> 1) & 7), r = blk*8 + rl
  return (unsigned)((rl * ld + c * 8) * (long)sizeof(bf16_t));
}
__device__ __forceinline__ void dma_rows(const bf16_t* __restrict__ p0, long ld, unsigned lane_off, bf16_t* s, int wave, int j) {
  const int blk = j * 8 + wave;
  dma16_at(p0 + (long)(blk * 8) * ld, lane_off, s + blk * 512);
}

// AS = LDS stages of a K-contiguous A (64 k each); with three or more a stage is refilled half on the even and half on
// the odd step, 2(AS-1) steps ahead, with two it is refilled whole on even steps.  A row-contiguous A travels with B in
// the BS-stage ring.
template <int BM, int BS, bool ATR, int AS = 2> struct Cfg {
  static constexpr bool HALVES = !ATR && AS >= 3;
  static constexpr int A_ELEMS = ATR ? KS * BM : BM * 64;      // per A stage
  static constexpr int A_STAGES = ATR ? BS : AS;
  static constexpr int B_ELEMS = KS * BN;
  static constexpr int LA = ATR ? BM / 128 : HALVES ? BM / 128 : BM / 64;  // DMA instructions per wave per refill of A
  static constexpr size_t SMEM = ((size_t)A_STAGES * A_ELEMS + (size_t)BS * B_ELEMS) * sizeof(bf16_t);
  static_assert(!HALVES || 2 * AS >= BS + 2, "the second half of an A stage must not be younger than B of the same step");
  // younger loads that may still be in flight when step `it` starts computing: the refills of the BS-2 steps since the
  // one that fetched B tile `it` (the last part of A tile it/2 is no younger)
  static constexpr int allowed(int parity) {
    if (ATR || HALVES) return (BS - 2) * (LA + LB);
    int even = 0;  // even steps among them
    for (int i = 1000 + parity - BS + 2; i <= 1000 + parity - 1; ++i) even += (i % 2 == 0);
    const int wrt_b = (BS - 2) * LB + LA * even;
    if (parity) return wrt_b;               // the A tile of this pair was checked on the even step
    const int wrt_a = 2 * (AS - 1) * LB + (AS - 2) * LA;
    return wrt_b < wrt_a ? wrt_b : wrt_a;
  }
};

// Half a step: the products of MH row fragments with NT column fragments.  After MFMA e the e-th fragment of the half
// step to come is read from LDS (NR of them), and the ND refills are spread evenly over the MFMAs.  The order is pinned:
// left to itself the compiler reads fragments right before their use and issues all refills together, and then the
// matrix pipe waits for the LDS and for the load unit (which takes 16 cycles per 1 KB instruction, 512 for the 32 of a
// step).  Each MFMA shares an operand with the one before it.
template <int NR, int ND, int MH, int NT, class R, class D>
__device__ __forceinline__ void half_step(f32x4 (*acc)[NT], const bf16x8 (&fa)[MH], const bf16x8 (&fb)[NT], R&& read,
                                          D&& dma) {
  constexpr int H = MH * NT;
  static_assert(NR <= H && ND <= H, "one read and one refill at most after an MFMA");
#pragma unroll
  for (int e = 0; e < H; ++e) {
    const int i = e / NT, j = (i & 1) ? NT - 1 - e % NT : e % NT;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);  // a wait for this MFMA's operands must not take in the read that follows
    if (e < NR) read(e);
#pragma unroll
    for (int d = 0; d < ND; ++d)
      if ((d + 1) * H / (ND > 0 ? ND : 1) - 1 == e) dma(d);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// What one wave's steps share.  it counts steps of 32 k; L holds the first MH row fragments of a step, H the others.
// read_a(it, i) and read_b(it, j) fetch fragments, dma(it, d, guard) issues refill d < ND of step it, wait(it, guard)
// waits for the tiles of step it (and meets the other waves), fetched() follows the last refill of a step.
// guard: near the end, where tiles past the end are not fetched and fewer loads are in flight than allowed() assumes.
template <int MH, int NT, int ND, class RA, class RB, class DM, class WA, class FE>
__device__ __forceinline__ void pipelined_steps(f32x4 (*acc)[NT], int nk, int safe, RA&& read_a, RB&& read_b, DM&& dma,
                                                WA&& wait, FE&& fetched) {
  constexpr int N0 = ND / 2, N1 = ND - N0;  // refills of a step issued before / after the MFMAs of its first half
  bf16x8 aL[MH], aH[MH], b0[NT], b1[NT];
  // order of the fragments of a step's start: b0 a0, the other columns, the other rows
  auto read_start = [&](int it, int r, bf16x8 (&b)[NT]) {
    if (r == 0) b[0] = read_b(it, 0);
    else if (r == 1) aL[0] = read_a(it, 0);
    else if (r <= NT) b[r - 1] = read_b(it, r - 1);
    else aL[r - NT] = read_a(it, r - NT);
  };
  // From step it to step it + 1: the MFMAs of the first half of step it run while the row fragments of its second half
  // are read; then the next step's tiles are waited for, and the second half's MFMAs run while the first fragments of
  // the next step are read.  A wave so reaches the barrier with matrix work queued and holds the fragments of half a step.
  auto advance = [&](int it, bool guard, const bf16x8 (&b)[NT], bf16x8 (&bn)[NT]) {
    half_step<MH, N1>(acc, aL, b, [&](int r) { aH[r] = read_a(it, MH + r); }, [&](int d) { dma(it, N0 + d, guard); });
    fetched();
    // these LDS reads must have completed before the barrier lets another wave refill the stage
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) only
    wait(it + 1, guard);
    half_step<MH + NT, N0>(acc + MH, aH, b, [&](int r) { read_start(it + 1, r, bn); },
                           [&](int d) { dma(it + 1, d, guard); });
  };
  wait(0, true);
#pragma unroll
  for (int r = 0; r < MH + NT; ++r) read_start(0, r, b0);
#pragma unroll
  for (int d = 0; d < N0; ++d) dma(0, d, true);
  int it = 0;
  for (; it < safe; it += 2) {  // every refill of steps it .. it + 2 exists
    advance(it, false, b0, b1);
    advance(it + 1, false, b1, b0);
  }
  for (; it + 2 < nk; it += 2) {
    advance(it, true, b0, b1);
    advance(it + 1, true, b1, b0);
  }
  advance(it, true, b0, b1);
  half_step<MH, 0>(acc, aL, b1, [&](int r) { aH[r] = read_a(nk - 1, MH + r); }, [](int) {});
  half_step<0, 0>(acc + MH, aH, b1, [](int) {}, [](int) {});
}

// The steps with two workgroups per CU (three-stage ring, half the registers): the other workgroup fills the gaps.
template <int MH, int NT, int ND, class RA, class RB, class DM, class WA, class FE>
__device__ __forceinline__ void plain_steps(f32x4 (*acc)[NT], int nk, RA&& read_a, RB&& read_b, DM&& dma, WA&& wait,
                                            FE&& fetched) {
  for (int it = 0; it < nk; ++it) {
    wait(it, true);
#pragma unroll
    for (int d = 0; d < ND; ++d) dma(it, d, true);
    fetched();
    bf16x8 a[MH], b[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) b[j] = read_b(it, j);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < MH; ++i) a[i] = read_a(it, h * MH + i);
#pragma unroll
      for (int i = 0; i < MH; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[h * MH + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[h * MH + i][j], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the reads are done before the next barrier
  }
}

template <int BM, int BS, int MODE, int AS>
__global__ __launch_bounds__(NTHREADS, (BM == 128 && BS == 3) ? 4 : 2) void gemm_mfma_kernel(const bf16_t* __restrict__ A,
                                                            const bf16_t* __restrict__ B, int M, int N, int K,
                                                            long lda, long ldb, EpiParams epi, int ksplit) {
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  typedef Cfg<BM, BS, false, AS> C;
  bf16_t* sA = reinterpret_cast<bf16_t*>(smem_raw);
  bf16_t* sB = sA + C::A_STAGES * C::A_ELEMS;
  constexpr int WM = BM / 2;
  constexpr int MT = WM / 16, NT = WN / 16;

  // Consecutive workgroup ids go to different XCDs (8, each with its own L2): renumber so that every
  // XCD gets a contiguous run of tiles, M fastest, and tiles that share a weight block share an L2.
  const int tiles_m = M / BM;
  const int nblk = gridDim.x;
  int pid = blockIdx.x;
  if ((nblk & 7) == 0) pid = (pid & 7) * (nblk >> 3) + (pid >> 3);
  if constexpr (MODE == EPI_PARTIAL) {
    // split-K: the K range is cut into ksplit slices of whole 64-k blocks; slice s of every tile writes its
    // fp32 partial product to plane s of the workspace (a fix-up kernel adds the planes in order)
    const int tiles = nblk / ksplit;
    const int slice = pid / tiles;
    pid -= slice * tiles;
    const int blocks64 = K / 64, per = (blocks64 + ksplit - 1) / ksplit;
    const int kb0 = slice * per, kb1 = min(blocks64, kb0 + per);
    A += (long)kb0 * 64;          // K-contiguous A
    B += (long)kb0 * 64 * ldb;    // row-contiguous B
    K = (kb1 - kb0) * 64;
    epi.outf += (size_t)slice * M * N;
  }
  // Tiles are walked in bands of GROUP_M tile rows, M fastest within a band: the 64 or so workgroups that
  // an XCD runs at one time then cover a block of about GROUP_M x 8 tiles and share, through its L2, both
  // the A panels (8 ways) and the B panels (GROUP_M ways) instead of streaming all of A once per column.
  constexpr int GROUP_M = 8;
  const int tiles_n = N / BN;
  const int band = pid / (GROUP_M * tiles_n);
  const int band_rows = min(tiles_m - band * GROUP_M, GROUP_M);
  const int in_band = pid - band * GROUP_M * tiles_n;
  const int m0 = (band * GROUP_M + in_band % band_rows) * BM;
  const int n0 = (in_band / band_rows) * BN;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = (wave >> 2) * WM, wn = (wave & 3) * WN;
  const unsigned a_off = dma_rows_lane_off(lda, wave, lane), b_off = dma_tr_lane_off<BN>(ldb, wave, lane);
  const bf16_t* a_tile = A + (long)m0 * lda;  // + k
  const bf16_t* b_tile = B + n0;              // + k * ldb

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = K / KS;  // even

  // Refills of step `it` (also used, with negative it, for the pipeline fill so that the order of loads is the same from
  // the first step on), as single DMA instructions: 0 .. LA-1 of A, then LB of B.  A tile j covers steps 2j, 2j+1.
  auto refill_a = [&](int it, int d, bool guard) {
    const int j = (it >> 1) + AS - 1;
    if (!C::HALVES && (it & 1)) return;
    if (guard && !(j >= 0 && 2 * j < nk)) return;
    dma_rows(a_tile + j * 64, lda, a_off, sA + (j % AS) * C::A_ELEMS, wave, C::HALVES ? (it & 1) * C::LA + d : d);
  };
  auto refill_b = [&](int it, int d, bool guard) {
    const int nt = it + BS - 1;
    if (guard && !(nt >= 0 && nt < nk)) return;
    dma_tr<BN>(b_tile + (long)(nt * KS) * ldb, ldb, b_off, sB + (nt % BS) * C::B_ELEMS, wave, d);
  };
  auto read_a = [&](int it, int i) { return frag16_rows(sA + ((it >> 1) % AS) * C::A_ELEMS, wm + i * 16, it & 1, lane); };
  auto read_b = [&](int it, int j) { return frag16_tr<BN>(sB + (it % BS) * C::B_ELEMS, wn + j * 16, 0, lane); };
  constexpr int AHEAD = (BS - 2) > (2 * AS - 3) ? (BS - 2) : (2 * AS - 3);  // last step whose refills all exist
  auto dma = [&](int it, int d, bool guard) {
    if (d < C::LA) refill_a(it, d, guard);
    else refill_b(it, d - C::LA, guard);
  };
  auto wait = [&](int it, bool guard) {
    if (guard && it + AHEAD >= nk) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    else if (it & 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::allowed(1)));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::allowed(0)));
    __builtin_amdgcn_s_barrier();
  };
  // pipeline fill: the same sequence of refills as in the loop, from the first step that issues anything
  constexpr int FILL0 = (1 - BS) < -2 * (AS - 1) ? (1 - BS) : -2 * (AS - 1);
#pragma unroll
  for (int it = FILL0; it < 0; ++it) {
#pragma unroll
    for (int d = 0; d < C::LA + LB; ++d) dma(it, d, true);
  }
  if constexpr (BS > 3) pipelined_steps<MT / 2, NT, C::LA + LB>(acc, nk, nk - AHEAD - 3, read_a, read_b, dma, wait, [] {});
  else plain_steps<MT / 2, NT, C::LA + LB>(acc, nk, read_a, read_b, dma, wait, [] {});

  epilogue_wave<MODE, MT, NT>(epi, m0 + wm, n0 + wn, lane, acc);
}

// ldo: row stride of the outputs when the GEMM covers a column range of a wider matrix (0: g.N)
template <int BM, int BS, int MODE, int AS = 2>
hipError_t run_cfg(const GemmArgs& g, long lda, long ldb, hipStream_t s, int ksplit = 1, int ldo = 0) {
  auto kern = gemm_mfma_kernel<BM, BS, MODE, AS>;
  constexpr size_t smem = Cfg<BM, BS, false, AS>::SMEM;
  static_assert(smem <= 160 * 1024, "LDS budget");
  static bool attr_set = false;  // one device per process in this library
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int grid = (g.M / BM) * (g.N / BN) * ksplit;
  EpiParams epi = make_epi(g);
  if (ldo) epi.N = ldo;
  kern<<<grid, NTHREADS, smem, s>>>((const bf16_t*)g.A, (const bf16_t*)g.B, g.M, g.N, g.K, lda, ldb, epi, ksplit);
  return hipGetLastError();
}

// Split-K fix-up: out = epilogue(sum of the K-slice planes, added in slice order), 4 columns per thread.
// The planes are [M, N] dense; the outputs (and aux) have row stride epi.N >= N.
template <int MODE>
__global__ __launch_bounds__(256) void gemm_splitk_fixup_kernel(const float* __restrict__ ws, int slices, size_t plane,
                                                                int N, EpiParams epi) {
  const size_t p4 = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (p4 >= plane) return;
  f32x4 acc = *reinterpret_cast<const f32x4*>(ws + p4);
  for (int sl = 1; sl < slices; ++sl) acc += *reinterpret_cast<const f32x4*>(ws + (size_t)sl * plane + p4);
  const int n = (int)(p4 % (size_t)N);
  const size_t i4 = (p4 / (size_t)N) * (size_t)epi.N + n;
  bf16x4 o0, o1;
  if (MODE == EPI_STORE) {
#pragma unroll
    for (int e = 0; e < 4; ++e) o0[e] = (bf16_t)acc[e];
  } else if (MODE == EPI_DGELU) {
    const bf16x4 a = *reinterpret_cast<const bf16x4*>((const bf16_t*)epi.aux + i4);
#pragma unroll
    for (int e = 0; e < 4; ++e) o0[e] = (bf16_t)(acc[e] * gelu_grad<bf16_t>((float)a[e]));
  } else {
    const f32x4 b = *reinterpret_cast<const f32x4*>(epi.bias + n);
    if (MODE == EPI_BIAS_RESID) {
      const bf16x4 a = *reinterpret_cast<const bf16x4*>((const bf16_t*)epi.aux + i4);
#pragma unroll
      for (int e = 0; e < 4; ++e) o0[e] = (bf16_t)(acc[e] + b[e] + (float)a[e]);
    } else if (MODE == EPI_BIAS_GELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float f = acc[e] + b[e];
        o0[e] = (bf16_t)f;
        o1[e] = (bf16_t)gelu<bf16_t>(f);
      }
      *reinterpret_cast<bf16x4*>((bf16_t*)epi.out1 + i4) = o1;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) o0[e] = (bf16_t)(acc[e] + b[e]);
    }
  }
  *reinterpret_cast<bf16x4*>((bf16_t*)epi.out0 + i4) = o0;
}

// wgrad: C += A_0^T B_0 + A_1^T B_1 + ... for `ngroup` >= 1 operand pairs of one shape (the W passes of one
// or of several consecutive microbatches), both operands row-contiguous ([k][m], [k][n]).  The accumulators
// START from the old C (requested before anything else, so the read travels while the ring of LDS stages
// fills) and every MFMA adds into them, pair after pair, in k order; the new C is written once at the end
// and nothing is read back there.  An element's value is therefore the same chain of fp32 MFMA additions
// whatever the tile shape, ring depth or grouping: `ngroup` pairs in one launch give exactly the bits of
// `ngroup` launches of one pair.  The ring runs on across the pairs without draining.
// One launch covers up to kWgradMaxProblems gradients (the weight matrices of one W pass: tiles of equal
// duration, so the partly filled last round of workgroups is paid once per pass instead of once per
// matrix) with `ngroup` operand pairs each.
struct WgradTable {
  int nprob, ngroup;
  int tile0[kWgradMaxProblems + 1];  // first tile of each problem in the launch
  int M[kWgradMaxProblems], N[kWgradMaxProblems];
  float* outf[kWgradMaxProblems];
  const bf16_t* a[kWgradMaxPairs];   // pair g of problem q at [q * ngroup + g]
  const bf16_t* b[kWgradMaxPairs];
  int ntiles;                        // workgroups [0, ntiles) are GEMM tiles, the rest column-sum strips
  int strip0[kWgradMaxProblems + 1]; // first strip (256 columns) of each problem; equal entries: no bias
  float* bias[kWgradMaxProblems];
};

// Bias gradient of one 256-column strip of one problem: bias[n] += sum over the Kc rows of every operand pair's
// b (the output gradient), pair by pair.  512 threads = 32 chunks of 8 columns x 16 row groups; a thread adds
// its rows in ascending order, the 16 row groups are added in ascending order, then the pair's sum goes onto
// the running value: the same chain of additions whether the pairs come in one launch or one launch each.
__device__ __forceinline__ void wgrad_bias_strip(const WgradTable& tb, int sid, int Kc, float* red) {
  int q = 0;
#pragma unroll
  for (int i = 1; i < kWgradMaxProblems; ++i) q += (i < tb.nprob && sid >= tb.strip0[i]) ? 1 : 0;
  sid -= tb.strip0[q];
  const int N = tb.N[q], ngroup = tb.ngroup;
  const int n0 = sid * BN;
  const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
  float* __restrict__ bias = tb.bias[q];
  float run = 0.f;
  if (threadIdx.x < BN) run = bias[n0 + threadIdx.x];
  for (int gi = 0; gi < ngroup; ++gi) {
    const bf16_t* __restrict__ b = tb.b[q * ngroup + gi] + n0 + c * 8;
    float sum[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) sum[j] = 0.f;
#pragma unroll 8
    for (int r = g; r < Kc; r += 16) {
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(b + (long)r * N);
#pragma unroll
      for (int j = 0; j < 8; ++j) sum[j] += (float)v[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[g * BN + c * 8 + j] = sum[j];
    __syncthreads();
    if (threadIdx.x < BN) {
      float t = 0.f;
#pragma unroll
      for (int gg = 0; gg < 16; ++gg) t += red[gg * BN + threadIdx.x];
      run += t;
    }
    __syncthreads();
  }
  if (threadIdx.x < BN) bias[n0 + threadIdx.x] = run;
}

template <int BM, int BS>
__global__ __launch_bounds__(512, (BM == 128 && BS == 3) ? 4 : 2) void gemm_wgrad_kernel(WgradTable tb, int Kc) {
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  typedef Cfg<BM, BS, true> C;
  bf16_t* sA = reinterpret_cast<bf16_t*>(smem_raw);
  bf16_t* sB = sA + C::A_STAGES * C::A_ELEMS;
  constexpr int WM = BM / 2;
  constexpr int MT = WM / 16, NT = WN / 16;

  const int nblk = tb.ntiles;
  int pid = blockIdx.x;
  if (pid >= nblk) {  // the launch's last workgroups: bias gradients (they fill the CUs the last round of tiles leaves idle)
    wgrad_bias_strip(tb, pid - nblk, Kc, reinterpret_cast<float*>(smem_raw));
    return;
  }
  if ((nblk & 7) == 0) pid = (pid & 7) * (nblk >> 3) + (pid >> 3);
  int q = 0;  // which problem this tile belongs to
#pragma unroll
  for (int i = 1; i < kWgradMaxProblems; ++i) q += (i < tb.nprob && pid >= tb.tile0[i]) ? 1 : 0;
  pid -= tb.tile0[q];
  const int M = tb.M[q], N = tb.N[q], ngroup = tb.ngroup;
  const long lda = M, ldb = N;
  float* __restrict__ outf = tb.outf[q];
  const int pair0 = q * ngroup;
  const int tiles_m = M / BM, tiles_n = N / BN;
  // Bands of 4 tile rows: an XCD runs 32 of these tiles at a time (one per CU), a block of 4 x 8.  Its four
  // A panels (K x 256 bf16, 512 KB each at K = 1024) then stay in the 4 MB L2 for the whole walk along the
  // band while B panels and the gradient tiles (non-temporal) stream past; at 8 rows the A panels alone fill
  // the L2 and are fetched again for every block (measured on the 14.6B stage: 785 -> 841 TFLOP/s; 2 rows
  // the same as 4, 1 row 818).
  constexpr int GROUP_M = 4;
  const int band = pid / (GROUP_M * tiles_n);
  const int band_rows = min(tiles_m - band * GROUP_M, GROUP_M);
  const int in_band = pid - band * GROUP_M * tiles_n;
  const int m0 = (band * GROUP_M + in_band % band_rows) * BM;
  const int n0 = (in_band / band_rows) * BN;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = (wave >> 2) * WM, wn = (wave & 3) * WN;
  const unsigned c_off = rows8_lane_off(N, lane);
  const unsigned a_off = dma_tr_lane_off<BM>(lda, wave, lane), b_off = dma_tr_lane_off<BN>(ldb, wave, lane);

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; j += 2) {
      const float* p0 = outf + (size_t)(m0 + wm + i * 16) * N + n0 + wn + j * 16;
      f32x8 c;
#pragma unroll
      for (int v = 0; v < 8; ++v) c[v] = __builtin_nontemporal_load(at_lane(p0 + (size_t)v * N, c_off));
      from_rows8(c, &acc[i][j], &acc[i][j + 1]);
    }

  const int spc = Kc / KS;        // steps per operand pair
  const int nk = ngroup * spc;
  // the next tile to fetch (tiles are fetched in order): its operand pair, k offset and addresses
  int g_next = 0, k_next = 0;
  const bf16_t* a_next = tb.a[pair0] + m0;
  const bf16_t* b_next = tb.b[pair0] + n0;
  auto dma = [&](int it, int d, bool guard) {
    const int nt = it + BS - 1;
    if (guard && nt >= nk) return;
    if (d < C::LA) dma_tr<BM>(a_next, lda, a_off, sA + (nt % BS) * C::A_ELEMS, wave, d);
    else dma_tr<BN>(b_next, ldb, b_off, sB + (nt % BS) * C::B_ELEMS, wave, d - C::LA);
  };
  auto next_tile = [&]() {
    a_next += (long)KS * lda;
    b_next += (long)KS * ldb;
    k_next += KS;
    if (k_next == Kc && ++g_next < ngroup) {
      k_next = 0;
      a_next = tb.a[pair0 + g_next] + m0;
      b_next = tb.b[pair0 + g_next] + n0;
    }
  };
  auto read_a = [&](int it, int i) { return frag16_tr<BM>(sA + (it % BS) * C::A_ELEMS, wm + i * 16, 0, lane); };
  auto read_b = [&](int it, int j) { return frag16_tr<BN>(sB + (it % BS) * C::B_ELEMS, wn + j * 16, 0, lane); };
  auto wait = [&](int it, bool guard) {
    if (guard && it + BS - 2 >= nk) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::allowed(0)));
    __builtin_amdgcn_s_barrier();
  };
#pragma unroll
  for (int it = 1 - BS; it < 0; ++it) {
#pragma unroll
    for (int d = 0; d < C::LA + LB; ++d) dma(it, d, true);
    next_tile();
  }
  if constexpr (BS > 3) pipelined_steps<MT / 2, NT, C::LA + LB>(acc, nk, nk - BS - 1, read_a, read_b, dma, wait, next_tile);
  else plain_steps<MT / 2, NT, C::LA + LB>(acc, nk, read_a, read_b, dma, wait, next_tile);

  // the store addresses are worked out again here (from a copy of the tile origin the compiler cannot
  // connect with the one used for the loads), or they would stay in registers across the loop
  int m0s = m0, n0s = n0;
  asm volatile("" : "+s"(m0s), "+s"(n0s));
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; j += 2) {
      float* p0 = outf + (size_t)(m0s + wm + i * 16) * N + n0s + wn + j * 16;
      const f32x8 c = rows8(acc[i][j], acc[i][j + 1]);
#pragma unroll
      for (int v = 0; v < 8; ++v) __builtin_nontemporal_store(c[v], at_lane(p0 + (size_t)v * N, c_off));
    }
}

// The K slices' planes are in the workspace: add them and apply the epilogue.
template <int MODE>
void finish_split_k(const GemmArgs& g, int slices, size_t plane, hipStream_t s, hipError_t* err) {
  // The last step owns whole rows: a LayerNorm on those rows rides along instead of running as a kernel of
  // its own on the stored result.
  const bool ln_shape = g.ln_done && g.N <= 8192;
  if (MODE == EPI_BIAS_RESID && g.ln_mode == 1 && ln_shape) {
    *err = launch_splitk_layernorm_fwd<bf16_t>(g.workspace, slices, plane, g.bias, (const bf16_t*)g.aux,
                                               (bf16_t*)g.out0, g.ln_gamma, g.ln_beta, (bf16_t*)g.ln_out, g.ln_stats,
                                               g.M, g.N, g.ln_eps, s);
    *g.ln_done = *err == hipSuccess;
    return;
  }
  if (MODE == EPI_STORE && g.ln_mode == 2 && ln_shape) {
    *err = launch_splitk_layernorm_bwd<bf16_t>(g.workspace, slices, plane, (bf16_t*)g.out0, (const bf16_t*)g.ln_x, g.ln_stats,
                                               g.ln_gamma, (const bf16_t*)g.ln_resid, (bf16_t*)g.ln_out, g.ln_dgamma,
                                               g.ln_dbeta, g.ln_partials, g.M, g.N, s);
    *g.ln_done = *err == hipSuccess;
    return;
  }
  const size_t threads = plane / 4;
  gemm_splitk_fixup_kernel<MODE><<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(g.workspace, slices, plane, g.N,
                                                                                 make_epi(g));
  *err = hipGetLastError();
}

// A little more than a whole number of rounds of 256 x 256 tiles over the 256 CUs (N = ffn with 1024
// tokens: 320 tiles): the full rounds run as they are and the tile columns left over are cut along K so
// that they, too, fill every CU once instead of occupying a quarter of the chip for a whole round.
struct Tail {
  int cols = 0, slices = 0;  // tile columns past the last full round (0: none worth it), the slices they are cut into
};
inline Tail tail_of(const GemmArgs& g) {
  if (g.M % 256 != 0 || g.K < 2048 || !g.workspace) return {};
  const int tm = g.M / 256, tn = g.N / BN;
  if ((long)tm * tn <= 256 || tm > 256 || 256 % tm != 0) return {};
  const int cols = tn % (256 / tm);
  if (cols == 0 || cols * tm > 128) return {};
  const int slices = 256 / (cols * tm) < 4 ? 256 / (cols * tm) : 4;
  return (size_t)slices * g.M * cols * BN > g.workspace_floats ? Tail{} : Tail{cols, slices};
}
template <int MODE>
hipError_t run_tail_split(const GemmArgs& g, long lda, long ldb, hipStream_t s, Tail tail) {
  const int slices = tail.slices;
  const int n_tail = tail.cols * BN, n_main = g.N - n_tail;
  const size_t plane = (size_t)g.M * n_tail;
  GemmArgs a = g;
  a.N = n_main;
  hipError_t e = run_cfg<256, 4, MODE, 3>(a, lda, ldb, s, 1, g.N);
  if (e != hipSuccess) return e;
  GemmArgs t = g;  // the same GEMM on columns n_main .. N-1
  t.N = n_tail;
  t.B = (const bf16_t*)g.B + n_main;
  if (t.out0) t.out0 = (bf16_t*)g.out0 + n_main;
  if (t.out1) t.out1 = (bf16_t*)g.out1 + n_main;
  if (t.aux) t.aux = (const bf16_t*)g.aux + n_main;
  if (t.bias) t.bias = g.bias + n_main;
  GemmArgs p = t;
  p.epilogue = EPI_PARTIAL;
  p.outf = g.workspace;
  e = run_cfg<256, 4, EPI_PARTIAL, 3>(p, lda, ldb, s, slices);
  if (e != hipSuccess) return e;
  EpiParams epi = make_epi(t);
  epi.N = g.N;
  const size_t threads = plane / 4;
  gemm_splitk_fixup_kernel<MODE><<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(g.workspace, slices, plane, n_tail,
                                                                                 epi);
  return hipGetLastError();
}

// The tiles that a product may be cut into, and the microseconds a launch of each takes: `start` for the launch and the
// fill of its ring, then for every round of the workgroups that the chip holds at once the steps of a workgroup (`few`
// with one on the chip, `all` with one on every CU; `over` with one more than that, `twice` with two on every CU; linear
// between) and an epilogue (2.9 times as long where a second matrix is read or written; none where K slices leave planes), but
// no less than the weights take to come from memory (us per 10^6 of them).  K slices add a launch that adds the planes (3.8 us,
// or 2.6 if it takes a LayerNorm over that runs anyway) and 1.7 us per 10^6 floats of planes, written and read.
//
// Fitted to 22 000 timings, back to back: every tile with up to four slices for the products of stages of hidden 96 to 6144,
// 128 to 6144 tokens (2447 products, 757 of them with a LayerNorm behind).  The figures tell the time of a launch within 9 %
// on average, and which is the shortest: what they choose takes 0.4 % longer than the shortest on average.  But a launch
// that is a little shorter on much more of the chip costs the launches beside it (777 x 4808 x 1200 alone 22.3 us on 64 x 64
// tiles, 27.3 on 128 x 128 ones; three stages at once, an iteration of hidden 1200 2370 and 2254 us), so half of what a
// launch takes of the chip is added: 0.8 % longer than the shortest on average, 6.7 % in one of 20 products, 23 % at most,
// and 4 % less of the chip.  A rule that took 256-column tiles wherever they fill half the chip and asked for the cost of the
// others alone took 2.3 % longer, 13 % in one of 20.
constexpr double kBusy = 0.5;
struct Tile {
  int rows, cols, k, at_once;
  double start, few, all, over, twice, epilogue, weights;
};
enum { kTile64, kTile128, kTile256, kTile128x256, kTile128x256Two, kTileTail };
constexpr Tile kTiles[] = {
    {64, 64, 64, 512, 1.6, 0.20, 0.29, 0.42, 0.48, 0.8, 0.63},   // gemm_mfma_edge.hip, any size
    {128, 128, 64, 256, 2.7, 0.41, 0.53, 0, 0, 1.2, 0.21},       // likewise
    {256, 256, 32, 256, 3.2, 0.53, 0.62, 0, 0, 4.1, 0.21},       // whole tiles, as the two below
    {128, 256, 32, 256, 1.5, 0.36, 0.46, 0, 0, 2.2, 0.21},
    {128, 256, 32, 512, 9.1, 0.45, 0.58, 0.82, 0.88, 0, 0.21},   // two workgroups per CU: one's loop hides the other's epilogue
};
double rounds_us(const Tile& t, long tiles, int steps, double epilogue) {
  auto round = [&](long r) {  // with r workgroups on the chip
    const double step = r <= 256 ? t.few + (t.all - t.few) * r / 256 : t.over + (t.twice - t.over) * (r - 256) / 256;
    return steps * step + epilogue * t.epilogue;
  };
  return (tiles / t.at_once) * round(t.at_once) + (tiles % t.at_once ? round(tiles % t.at_once) : 0.0);
}
// What the launch takes of the chip: the time it would have it busy alone if its workgroups were packed without gaps.
double busy_us(const Tile& t, long tiles, int steps) { return tiles * steps * (t.at_once > 256 ? t.twice : t.all) / t.at_once; }
double planes_us(double floats, bool rides) { return (rides ? 2.6 : 3.8) + 1.7e-6 * floats; }

struct Plan {
  int tile = -1, slices = 1;  // tile -1: no tile takes the shape
  Tail tail;                  // kTileTail: 256 x 256 tiles with the last columns in slices
};
// rides: a LayerNorm on the output's rows, which the launch that adds K slices takes over (finish_split_k)
Plan choose_tile(const GemmArgs& g, int mode, bool rides) {
  Plan best;
  double us = 1e30;
  auto take = [&](double c, int tile, int slices, Tail tail) {
    if (c < us) { us = c; best.tile = tile; best.slices = slices; best.tail = tail; }
  };
  const bool whole = g.K % 64 == 0 && g.M % 128 == 0 && g.N % BN == 0;
  const double epilogue = mode == EPI_STORE || mode == EPI_BIAS ? 1.0 : 2.9;
  const size_t plane = (size_t)g.M * g.N, room = g.workspace ? g.workspace_floats : 0;
  const int blocks = (g.K + 63) / 64;
  for (int i = kTile64; i <= kTile128x256Two; ++i) {
    const Tile& t = kTiles[i];
    if (i <= kTile128 ? g.N % 8 != 0 : !whole || g.M % t.rows != 0) continue;
    const long tiles = (long)((g.M + t.rows - 1) / t.rows) * ((g.N + t.cols - 1) / t.cols);
    for (int sl = 1; sl <= (i <= kTile256 ? 4 : 1); ++sl) {
      const int per = (blocks + sl - 1) / sl;
      if (sl > 1 && (sl * plane > room || (sl - 1) * per >= blocks)) continue;  // no room; an empty slice
      const double c = rounds_us(t, tiles * sl, per * (64 / t.k), sl > 1 ? 0.0 : epilogue);
      const double mem = t.weights * 1e-6 * g.N * g.K;
      take(t.start + (c > mem ? c : mem) + (sl > 1 ? planes_us((double)sl * plane, rides) : 0.0) +
               kBusy * busy_us(t, tiles * sl, per * (64 / t.k)),
           i, sl, {});
    }
  }
  const Tail tail = whole ? tail_of(g) : Tail{};
  if (tail.cols) {
    const Tile& t = kTiles[kTile256];
    const long main = (long)(g.M / 256) * (g.N / BN - tail.cols), rest = (long)(g.M / 256) * tail.cols * tail.slices;
    const int steps = blocks * 2, rest_steps = (blocks + tail.slices - 1) / tail.slices * 2;
    take(2 * t.start + rounds_us(t, main, steps, epilogue) + rounds_us(t, rest, rest_steps, 0.0) +
             planes_us((double)tail.slices * g.M * tail.cols * BN, false) +
             kBusy * (busy_us(t, main, steps) + busy_us(t, rest, rest_steps)),
         kTileTail, tail.slices, tail);
  }
  return best;
}

template <int MODE>
hipError_t run_shape(const GemmArgs& g, long lda, long ldb, hipStream_t s, bool* taken) {
  const bool rides = g.ln_done && g.N <= 8192 && (MODE == EPI_BIAS_RESID ? g.ln_mode == 1 : MODE == EPI_STORE && g.ln_mode == 2);
  const Plan plan = choose_tile(g, MODE, rides);
  *taken = plan.tile >= 0;
  if (!*taken) return hipSuccess;
  const int edge = plan.tile == kTile64 ? 64 : 128;
  if (plan.tile == kTileTail) return run_tail_split<MODE>(g, lda, ldb, s, plan.tail);
  if (plan.slices > 1) {
    GemmArgs p = g;
    p.epilogue = EPI_PARTIAL;
    p.outf = g.workspace;
    hipError_t e = plan.tile == kTile256 ? run_cfg<256, 4, EPI_PARTIAL, 3>(p, lda, ldb, s, plan.slices)
                                         : launch_gemm_edge(p, lda, ldb, edge, plan.slices, s);
    if (e == hipSuccess) finish_split_k<MODE>(g, plan.slices, (size_t)g.M * g.N, s, &e);
    return e;
  }
  if (plan.tile == kTile256) return run_cfg<256, 4, MODE, 3>(g, lda, ldb, s);
  if (plan.tile == kTile128x256) return run_cfg<128, 5, MODE>(g, lda, ldb, s);
  if (plan.tile == kTile128x256Two) return run_cfg<128, 3, MODE>(g, lda, ldb, s);
  return launch_gemm_edge(g, lda, ldb, edge, 1, s);
}

template <int BM, int BS>
hipError_t run_wgrad(WgradTable& tb, int K, hipStream_t s) {
  auto kern = gemm_wgrad_kernel<BM, BS>;
  constexpr size_t smem = Cfg<BM, BS, true>::SMEM;
  static_assert(smem <= 160 * 1024, "LDS budget");
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  int tiles = 0;
  for (int q = 0; q < tb.nprob; ++q) {
    tb.tile0[q] = tiles;
    tiles += (tb.M[q] / BM) * (tb.N[q] / BN);
  }
  for (int q = tb.nprob; q <= kWgradMaxProblems; ++q) tb.tile0[q] = tiles;
  tb.ntiles = tiles;
  int strips = 0;
  for (int q = 0; q < tb.nprob; ++q) {
    tb.strip0[q] = strips;
    if (tb.bias[q]) strips += tb.N[q] / BN;
  }
  for (int q = tb.nprob; q <= kWgradMaxProblems; ++q) tb.strip0[q] = strips;
  static_assert(smem >= 16 * BN * sizeof(float), "the strips' reduction buffer");
  kern<<<tiles + strips, NTHREADS, smem, s>>>(tb, K);
  return hipGetLastError();
}

}  // namespace

template <typename T> hipError_t launch_gemm_mfma(const GemmArgs& g, hipStream_t s, bool* taken);  // fp32: gemm_f32.hip

// wgrad launch for the gradients of one W pass; *taken stays false if a shape is not one for the MFMA kernel
template <typename T> hipError_t launch_wgrad_multi_mfma(const WgradMultiArgs& w, hipStream_t s, bool* taken);
template <> hipError_t launch_wgrad_multi_mfma<bf16_t>(const WgradMultiArgs& w, hipStream_t s, bool* taken) {
  *taken = false;
  if (w.nprob < 1 || w.nprob > kWgradMaxProblems || w.ngroup < 1 || w.ngroup > kGemmGroupMax ||
      w.nprob * w.ngroup > kWgradMaxPairs || w.K <= 0)
    return hipSuccess;
  if (w.K % 64 != 0) return launch_wgrad_multi_edge(w, s, taken);
  WgradTable tb{};
  tb.nprob = w.nprob;
  tb.ngroup = w.ngroup;
  bool all256 = true;
  long t256 = 0, t128 = 0;
  for (int q = 0; q < w.nprob; ++q) {
    const int M = w.M[q], N = w.N[q];
    if (M <= 0 || N <= 0 || M % 128 != 0 || N % BN != 0 || !aligned16(w.outf[q]))
      return launch_wgrad_multi_edge(w, s, taken);
    tb.M[q] = M; tb.N[q] = N; tb.outf[q] = w.outf[q];
    tb.bias[q] = w.bias_done ? w.bias[q] : nullptr;
    all256 = all256 && M % 256 == 0;
    t256 += (long)(M / 256) * (N / BN);
    t128 += (long)(M / 128) * (N / BN);
    for (int g = 0; g < w.ngroup; ++g) {
      const void* a = w.a[q * w.ngroup + g];
      const void* b = w.b[q * w.ngroup + g];
      if (!a || !b || !aligned16(a) || !aligned16(b)) return hipSuccess;
      tb.a[q * w.ngroup + g] = (const bf16_t*)a;
      tb.b[q * w.ngroup + g] = (const bf16_t*)b;
    }
  }
  if (t128 >= (1L << 30)) return hipSuccess;
  *taken = true;
  if (w.bias_done) *w.bias_done = true;
  // 256-row tiles (one workgroup per CU, four-stage ring) when they fill most of the chip and the chain is long; else 128-row
  // tiles, two workgroups per CU with a three-stage ring if there are more tiles than CUs, one with a
  // five-stage ring otherwise.  With a short chain the gradient's way in and out is most of the time, and a second
  // workgroup's loop hides it: 256 tokens of h 1024, two layers 50.7 us on 256-row tiles, 42.1 on 128-row ones, 2 x 192 of
  // h 1280 51.4 and 45.7, 2 x 128 of h 2048 95.8 and 88.8, 512 of h 768, four layers 66.1 both, 1024 of h 4096 554 and 559,
  // 6144 of h 2304 2018 and 2407.  But with up to four steps the second workgroup has too little to hide behind where 256-row
  // tiles make one round or all but fill two: 128 of h 1024 (192 tiles) 20.3 and 23.3, 192 of it 21.7 and 22.2, 128 of h
  // 1536 (432) 45.5 and 47.6, of two layers of h 1024 (384) 45.4 and 37.3.  The choice does not change the result (see the kernel).
  const long chain = (long)w.K * w.ngroup;
  const bool full_rounds = t256 <= 256 || (t256 > 400 && t256 <= 512);
  if (all256 && t256 >= 192 && (chain >= 512 || (chain <= 128 && full_rounds))) return run_wgrad<256, 4>(tb, w.K, s);
  if (t128 > 256) return run_wgrad<128, 3>(tb, w.K, s);
  return run_wgrad<128, 5>(tb, w.K, s);
}

namespace {

// one accumulate GEMM (one pair, or g.group pairs) through the same kernel
hipError_t launch_wgrad(const GemmArgs& g, hipStream_t s, bool* taken) {
  const int ngroup = g.group >= 2 ? g.group : 1;
  if (g.epilogue != EPI_ACCUM_F32 || ngroup > kGemmGroupMax) return hipSuccess;
  if (!(g.a_sm == 1 && g.b_sn == 1) || g.a_sk != g.M || g.b_sk != g.N) return hipSuccess;
  WgradMultiArgs w{};
  w.nprob = 1; w.ngroup = ngroup; w.K = g.K;
  w.M[0] = g.M; w.N[0] = g.N; w.outf[0] = g.outf;
  for (int i = 0; i < ngroup; ++i) {
    w.a[i] = g.group >= 2 ? g.group_a[i] : g.A;
    w.b[i] = g.group >= 2 ? g.group_b[i] : g.B;
  }
  return launch_wgrad_multi_mfma<bf16_t>(w, s, taken);
}

}  // namespace

template <> hipError_t launch_gemm_mfma<bf16_t>(const GemmArgs& g, hipStream_t s, bool* taken) {
  *taken = false;
  if (g.epilogue == EPI_ACCUM_F32) return launch_wgrad(g, s, taken);
  // forward X[M,K] * W[K,N]; dgrad dY[M,K'] * Wt[K',N']: A K-contiguous, B row-contiguous
  if (g.a_sk != 1 || !(g.b_sn == 1 && g.b_sk != 1)) return hipSuccess;
  const long lda = g.a_sm, ldb = g.b_sk;
  if (g.K % 8 != 0 || lda % 8 != 0 || ldb % 8 != 0 || !aligned16(g.A) || !aligned16(g.B)) return hipSuccess;
  if (g.epilogue == EPI_BIAS) return run_shape<EPI_BIAS>(g, lda, ldb, s, taken);
  if (g.epilogue == EPI_BIAS_RESID) return run_shape<EPI_BIAS_RESID>(g, lda, ldb, s, taken);
  if (g.epilogue == EPI_BIAS_GELU) return run_shape<EPI_BIAS_GELU>(g, lda, ldb, s, taken);
  if (g.epilogue == EPI_STORE) return run_shape<EPI_STORE>(g, lda, ldb, s, taken);
  if (g.epilogue == EPI_DGELU) return run_shape<EPI_DGELU>(g, lda, ldb, s, taken);
  return hipSuccess;
}

}  // namespace zb
