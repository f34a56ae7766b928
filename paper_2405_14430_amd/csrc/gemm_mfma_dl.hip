// bf16 MFMA GEMMs with direct global->LDS loads (gfx950): C = epilogue(A W^T + bias), A [M,K], W [N,K], both
// contiguous along K, K a multiple of 64.
//
// Tiles are brought in with global_load_lds_dwordx4: one instruction moves 64 x 16 B = 1 KB = eight 128-byte tile
// rows (64 bf16 of K each), lane l filling row l/8, 16-byte slot l%8.  The LDS side of such a load is lane-linear (no
// padding possible), so bank conflicts are avoided with an XOR swizzle: chunk c (8 bf16) of tile row r is kept in slot
// c ^ ((r >> 1) & 7); the loading lane picks its global chunk accordingly and the MFMA fragment reads undo it.  Rows
// beyond M (or N) are clamped to the last valid row: they only feed accumulators that the epilogue never stores.
//
// Two kernels share that machinery:
//  * gemm_tile_kernel<BM,BN,NSTAGE>: WGM x WGN wavefronts share one BM x BN tile.  For GEMMs with enough tiles to fill the
//    chip.  K loops: rings of whole K tiles here, operand rings in gemm_ring.h, half tiles in gemm_half_tiles.h.
//  * gemm_wavek_kernel<BM,BN>: for skinny GEMMs (n = 512 patch rows: a few hundred tiles at most).  The four
//    wavefronts of a workgroup split K between them: each streams its own K tiles through a private two-stage LDS
//    ring with no workgroup barrier in the loop, which quadruples the loads in flight per CU and divides the serial
//    chain of K iterations by four; the four partial tiles are then summed through LDS.
// Both finish through LDS: the fp32 tile is laid out row-major and every thread applies the epilogue to runs of 8
// consecutive columns (16-byte bf16 stores, 32-byte fp32 stores).
#include <algorithm>

#include "gemm_half_tiles.h"
#include "gemm_ring.h"
#include "gemm_tile.h"

namespace pf {

namespace {

constexpr int BK = 64;
constexpr int ROW_BYTES = BK * 2;  // 128

// ------------------------------------------------------------------------------------------------------------------
// WGM x WGN wavefronts on one shared tile
// ------------------------------------------------------------------------------------------------------------------

// K loops of gemm_tile_kernel.  256x256: half tiles refilled one by one (gemm_half_tiles.h).  The other tiles 256
// rows high: a ring for either operand, NSTAGE K tiles of A and loop_depth_w of W deep, as LDS allows (gemm_ring.h).  Below, one
// ring of whole K tiles (this file).  us with this file's loop -> with the other:
//    2048x9216x3072   256x192 132 -> 113     2048x12288x3072 GELU   256x192 154 -> 136
//    2560x3072x15360 residual   256x128 241 -> 204                          16896x9216x3072   256x256 847 -> 737
// and where the ring is not used (two builds in one run): 2048x9216x3072, 128x192 two stages 109, ring of two 108, but 125 and 134
// inside the Flux-scale stage, whose weights are cold (two K tiles deep, the ring asks for W a quarter of a K tile later);
// 2048x3072x15360 residual, 128x192 three stages 185, ring of four 188; 4096x1152x4608 residual, 128x128 59, ring 64; 1024x4608x1152
// GELU, 128x64 21.4, ring 24.4; 512x4608x1536 GELU, 64x128 18.2, ring 18.6.
constexpr bool loop_half_tiles(int BM, int BN) { return BM == 256 && BN == 256; }
constexpr int loop_depth_w(int BM, int BN, bool SPREAD) {
  return SPREAD || loop_half_tiles(BM, BN) || BM < 256 ? 0 : 4;
}

template <int NP, int EM, int BM, int BN, int NSTAGE, int WGM = 2, int WGN = 2, bool SPREAD_LOADS = false>
__global__ __launch_bounds__(64 * WGM * WGN, NSTAGE * (BM + BN) * ROW_BYTES <= 80 * 1024 ? WGM * WGN / 2 : WGM * WGN / 4) void gemm_tile_kernel(GemmLaunch<bf16_t, NP> L) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  constexpr int DW = loop_depth_w(BM, BN, SPREAD_LOADS);
  if constexpr (loop_half_tiles(BM, BN)) {
    gemm_half_tiles_body<NP, EM>(L, smem);
  } else if constexpr (DW > 0) {
    gemm_ring_body<NP, EM, BM, BN, WGM, WGN, NSTAGE, DW>(L, smem);
  } else {
  const bool second = NP == 2 && blockIdx.x >= L.grid0;
  const GemmProblem<bf16_t> &prob = L.p[second ? 1 : 0];
  const bf16_t *__restrict__ A = prob.A, *__restrict__ W = prob.W;
  const int64_t lda = prob.lda, ldw = prob.ldw;
  const int M = prob.M, N = L.N, K = L.K;
  const Epilogue<bf16_t> &epi = prob.epi;
  const int vec_ok = prob.vec_ok;
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int MI = WM / 32, NI = WN / 32;
  constexpr int RPI = 1024 / ROW_BYTES, CPR = BK / 8;    // rows per load instruction, 16-byte chunks per row
  constexpr int LA = BM / RPI / NW, LW = BN / RPI / NW;  // load instructions per wave per stage
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile rows must split evenly over the waves' load instructions");
  constexpr int LPS = LA + LW;
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES;
  auto key = [](int r) { return (r >> 1) & 7; };
  constexpr int TLD = BN + 4;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  int tm, tn;
  if (!tile_of_id((int)(blockIdx.x - (second ? L.grid0 : 0)), (M + BM - 1) / BM, (N + BN - 1) / BN, prob.xcd_gx, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;

  // per-lane byte offsets of this wave's load instructions inside the tile's rows (rows past the matrix repeat its last row)
  const TileSource srcA(A + (size_t)m0 * lda), srcW(W + (size_t)n0 * ldw);
  unsigned pa[LA], pw[LW];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    int r = (i * NW + wave) * RPI + lane / CPR;
    int c = (lane % CPR) ^ key(r);
    pa[i] = (unsigned)(((size_t)min(r, M - 1 - m0) * lda + c * 8) * 2);
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    int r = (i * NW + wave) * RPI + lane / CPR;
    int c = (lane % CPR) ^ key(r);
    pw[i] = (unsigned)(((size_t)min(r, N - 1 - n0) * ldw + c * 8) * 2);
  }
  const int nk = K / BK;
  auto issue = [&](int stage, int kt) {
    unsigned char *sa = smem + stage * STAGE_BYTES;
    unsigned char *sw = sa + BM * ROW_BYTES;
    const unsigned koff = (unsigned)kt * (BK * 2);
#pragma unroll
    for (int i = 0; i < LA; ++i) srcA.load16(pa[i], koff, sa + (i * NW + wave) * 1024);
#pragma unroll
    for (int i = 0; i < LW; ++i) srcW.load16(pw[i], koff, sw + (i * NW + wave) * 1024);
  };
  // load instruction `idx` (A instructions first, then W) of this wave for K tile kt
  auto issue_one = [&](auto idx_c, int stage, int kt) __attribute__((always_inline)) {
    constexpr int idx = decltype(idx_c)::value;
    unsigned char *sa = smem + stage * STAGE_BYTES;
    const unsigned koff = (unsigned)kt * (BK * 2);
    if constexpr (idx < LA) srcA.load16(pa[idx], koff, sa + (idx * NW + wave) * 1024);
    else srcW.load16(pw[idx - LA], koff, sa + BM * ROW_BYTES + ((idx - LA) * NW + wave) * 1024);
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
  for (int s = 0; s < NSTAGE - 1; ++s)
    if (s < nk) issue(s, s);

  // the epilogue's operands (residual and gate of small tiles) behind the first tiles, whose latency covers the address arithmetic
  constexpr bool EPRE = EM == EM_RESIDUAL && BM * BN / 8 / (64 * NW) <= 2;
  EpiOperands<BM, BN, 64 * NW> eops;
  if constexpr (EPRE) eops.fetch(m0, n0, M, N, epi, vec_ok != 0);

  // The bias behind the loop where the ring is deeper than two: the loop's waits count tile loads, so with the bias in flight the
  // first one would wait for a part of the next tile too.  us with the bias in front of the loop -> behind it: 576x2048x2048 13.5 -> 12.7
  // and 22x2304x768 6.4 -> 6.0 (64x64, four stages), 1024x3456x1152 15.5 -> 15.0 (64x128), 1038x4608x1152 GELU 22.0 -> 21.7 (128x192,
  // three).  A ring of two waits for all loads anyway: 4096x1152x1152 residual, 128x128, 22.1 in front and 22.5 behind; 2000x2304x1152,
  // 128x64, 21.4 and 21.8; 1024x4608x1152 GELU, 64x64, 26.5 and 26.9.
  constexpr bool BIAS_FIRST = NSTAGE == 2;
  ColumnBias<NI, 32, bf16_t> column_bias;
  if constexpr (BIAS_FIRST) column_bias.fetch(epi, n0 + wn * WN + (lane & 31), N);

  const int l32 = lane & 31, hi = lane >> 5;
  int arow[MI], akey[MI], wrow[NI], wkey[NI];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    int r = wm * WM + i * 32 + l32;
    arow[i] = r * ROW_BYTES;
    akey[i] = key(r);
  }
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    int r = wn * WN + j * 32 + l32;
    wrow[j] = BM * ROW_BYTES + r * ROW_BYTES;
    wkey[j] = key(r);
  }

  // SPREAD: the loads of the tile that is prefetched during K tile kt are not issued in one burst after the barrier but
  // one at a time between the MFMA groups of the tile (the burst fills the memory pipeline's queue and every wave
  // then stalls at its own load instructions before it can start on its MFMAs).  Every iteration issues the same LPS
  // loads - past the last K tile it repeats the last tile into the stage that has just been freed - so the loop body has
  // no branch around a load and the wait in front of tile kt is the same for every kt.
  constexpr int KS = BK / 16;
  constexpr bool SPREAD = SPREAD_LOADS && MI * NI * KS >= 2 * LPS;
  const int prologue_tiles = min(NSTAGE - 1, nk);
  if constexpr (EPRE && NP == 2) wait_scalar_loads();
  for (int kt = 0; kt < nk; ++kt) {
    // tiles still in flight behind tile kt: min(NSTAGE-2, nk-1-kt); wait until only their loads are outstanding
    const int behind = SPREAD ? prologue_tiles - 1 : min(NSTAGE - 2, nk - 1 - kt);
    wait_tiles_behind<LPS, NSTAGE - 2>(behind);
    // plain s_barrier: __syncthreads() would also drain every global load in flight (vmcnt(0)), i.e. the prefetches
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int ld_stage = (kt + NSTAGE - 1) % NSTAGE, ld_kt = min(kt + NSTAGE - 1, nk - 1);
    if constexpr (!SPREAD) {
      if (kt + NSTAGE - 1 < nk) issue(ld_stage, kt + NSTAGE - 1);
    }
    const unsigned char *st = smem + (kt % NSTAGE) * STAGE_BYTES;
    // Fragments are read from LDS PRE k-steps ahead of the MFMAs that use them: with one accumulator per wave
    // (64x64 tile) a k-step is a single MFMA, far shorter than an LDS read, so the whole tile is preloaded.
    constexpr int PRE = (MI * NI <= 2) ? KS : 2;
    bf16x8 af[PRE][MI], wf[PRE][NI];
    auto lread = [&](int buf, int ks) {
      const int c = ks * 2 + hi;
#pragma unroll
      for (int i = 0; i < MI; ++i) af[buf][i] = *reinterpret_cast<const bf16x8 *>(st + arow[i] + ((c ^ akey[i]) << 4));
#pragma unroll
      for (int j = 0; j < NI; ++j) wf[buf][j] = *reinterpret_cast<const bf16x8 *>(st + wrow[j] + ((c ^ wkey[j]) << 4));
    };
#pragma unroll
    for (int ks = 0; ks < PRE - 1; ++ks) lread(ks, ks);
    unrolled<KS>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      if (ks + PRE - 1 < KS) lread((ks + PRE - 1) % PRE, ks + PRE - 1);
      // keep the LDS reads of the next k-step ahead of this k-step's MFMAs (the scheduler would otherwise sink them
      // to reuse the fragment registers, exposing the LDS latency at every k-step)
      __builtin_amdgcn_sched_barrier(0);
      unrolled<MI * NI>([&](auto m_c) __attribute__((always_inline)) {
        constexpr int m = decltype(m_c)::value, i = m / NI, j = m % NI;
        if constexpr (SPREAD) {
          // MFMA number g of the tile's G = MI * NI * KS; load l goes in front of MFMA (2 l + 1) G / (2 LPS)
          constexpr int g = ks * MI * NI + m, G = MI * NI * KS;
          constexpr int l = g * LPS / G;
          if constexpr (l < LPS && g == ((2 * l + 1) * G) / (2 * LPS)) {
            issue_one(std::integral_constant<int, l>{}, ld_stage, ld_kt);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks % PRE][i], wf[ks % PRE][j], acc[i][j], 0, 0, 0);
      });
    });
  }

  if constexpr (!BIAS_FIRST) column_bias.fetch(epi, n0 + wn * WN + (lane & 31), N);
  float bias[NI];
  column_bias.widen(bias);
  // accumulators -> row-major fp32 tile in LDS (lane -> column l32, register r -> row 8*(r/4) + 4*hi + r%4), in
  // passes of RB rows when the whole tile does not fit in the stage memory
  constexpr int RING = NSTAGE * STAGE_BYTES;
  constexpr int RB = (BM * TLD * 4 <= RING) ? BM : ((BM / 2) * TLD * 4 <= RING ? BM / 2 : BM / 4);
  static_assert(RB * TLD * 4 <= RING || RB == BM, "epilogue pass does not fit");
  static_assert(RB % WM == 0 || WM % RB == 0, "pass rows and wave rows must nest");
  float *tile = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int pass = 0; pass < BM / RB; ++pass) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int rbase = wm * WM + i * 32;          // first tile row of this 32-row block
      if (rbase / RB != pass) continue;
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          tile[(rbase - pass * RB + 8 * (r >> 2) + 4 * hi + (r & 3)) * TLD + wn * WN + j * 32 + l32] = acc[i][j][r] + bias[j];
    }
    __syncthreads();
    if constexpr (EPRE && RB == BM) tile_epilogue<EM, BM, BN, TLD, 64 * NW, true>(tile, m0, n0, M, N, epi, vec_ok != 0, &eops);
    else tile_epilogue<EM, RB, BN, TLD, 64 * NW>(tile, m0 + pass * RB, n0, M, N, epi, vec_ok != 0);
  }
  }
}

// ------------------------------------------------------------------------------------------------------------------
// four wavefronts split K; each owns a private two-stage ring for its own BM x BN x 64 tiles
// ------------------------------------------------------------------------------------------------------------------

// Workgroups behind the tiles of a launch that leaves CUs idle: they read the rows of their XCD's block of the tile grid (see
// tile_of_id) ahead of the workgroups that multiply, K tile by K tile, two words of every 128-byte row piece, so that the tile loads
// find them in the XCD's L2.  The weights of a stage's GEMMs come from the memory-side cache or HBM, and a CU that waits for
// them takes in 60 bytes a ns, half of what it gets from its L2.  A reader asks for READ_AHEAD_LOADS words a thread at a time and
// takes 1 - 1.2 us for a K tile of 576 rows (one word at a time: 2 us).  us of a launch without readers, with, weights from HBM:
//   512x1152x4608 residual (11 per XCD)   20.5, 16.1      512x1152x1152 (11)   9.1, 8.2      375x1536x6144 (11)   26.6, 19.8
//   512x1536x6144 (8)   26.6, 23.7      64x3072x15360 (11)   66.7, 43.7
// PixArt-scale call (144 tiles) 410 -> 400, SD3-scale (192 tiles) 326 -> 320.
// The launch lasts until the readers are through, so how many there are is bounded (gemm_read_ahead_workgroups).  Launches of two
// problems lose by them (SD3-scale with 77 text rows 245 -> 267 us: every XCD has blocks of two matrices to read) and do without.
// Readers hold a CU each, which a launch on another stream does not get meanwhile: a call each of two PixArt-scale stages on two
// streams takes 636 us with them and 656 without, of two SD3-scale stages 703 and 740, sixteen PixArt-scale calls beside a Flux-scale
// one 12220 and 12260.
constexpr int READ_AHEAD_LOADS = 6;

template <int BM, int BN>
__device__ void read_ahead(const GemmLaunch<bf16_t, 1> &L) {
  const GemmProblem<bf16_t> &p = L.p[0];
  const int x = blockIdx.x & 7, first = (int)((blockIdx.x - L.grid) >> 3), step = (int)((gridDim.x - L.grid) >> 3);
  const int gx = p.xcd_gx & 255, tiles_m = (p.M + BM - 1) / BM, tiles_n = (L.N + BN - 1) / BN;
  const int bm = (tiles_m + gx - 1) / gx, bn = (tiles_n + 8 / gx - 1) / (8 / gx);
  const int w0 = min(L.N, (x / gx) * bn * BN), w_rows = min(L.N, (x / gx + 1) * bn * BN) - w0;
  const int a0 = min(p.M, (x % gx) * bm * BM), a_rows = min(p.M, (x % gx + 1) * bm * BM) - a0;
  const int words = 2 * (w_rows + a_rows);
  unsigned keep = 0;
  for (int kt = first; kt < L.K / BK; kt += step) {
#pragma unroll 1
    for (int from = threadIdx.x; from < words; from += READ_AHEAD_LOADS * 256) {
      unsigned v[READ_AHEAD_LOADS];
#pragma unroll
      for (int i = 0; i < READ_AHEAD_LOADS; ++i) {   // (past the last word: that one again)
        const int u = min(from + i * 256, words - 1), r = u >> 1;
        const bf16_t *row = r < w_rows ? p.W + (size_t)(w0 + r) * p.ldw : p.A + (size_t)(a0 + r - w_rows) * p.lda;
        v[i] = *reinterpret_cast<const unsigned *>(row + kt * BK + (u & 1) * (BK / 2));
      }
#pragma unroll
      for (int i = 0; i < READ_AHEAD_LOADS; ++i) keep ^= v[i];
    }
  }
  asm volatile("" ::"v"(keep));
}

template <int NP, int EM, int BM, int BN>
__global__ __launch_bounds__(256) void gemm_wavek_kernel(GemmLaunch<bf16_t, NP> L) {
  if constexpr (NP == 1) {
    if (blockIdx.x >= L.grid) {
      read_ahead<BM, BN>(L);
      return;
    }
  }
  const bool second = NP == 2 && blockIdx.x >= L.grid0;
  const GemmProblem<bf16_t> &prob = L.p[second ? 1 : 0];
  const bf16_t *__restrict__ A = prob.A, *__restrict__ W = prob.W;
  const int64_t lda = prob.lda, ldw = prob.ldw;
  const int M = prob.M, N = L.N, K = L.K;
  const Epilogue<bf16_t> &epi = prob.epi;
  const int vec_ok = prob.vec_ok;
  constexpr int MI = BM / 32, NI = BN / 32;
  constexpr int LA = BM / 8, LW = BN / 8;   // load instructions per wave per stage (a wave loads whole tiles)
  constexpr int LPS = LA + LW;
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES;
  constexpr int WAVE_BYTES = 2 * STAGE_BYTES;
  constexpr int TLD = BN + 4;
  static_assert(LPS <= 31, "two stages of loads must fit the vmcnt counter");
  static_assert(WAVE_BYTES >= BM * TLD * 4, "a wave's partial tile must fit in its own ring");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  if (!tile_of_id((int)(blockIdx.x - (second ? L.grid0 : 0)), (M + BM - 1) / BM, (N + BN - 1) / BN, prob.xcd_gx, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  unsigned char *ring = smem + wave * WAVE_BYTES;

  // K tiles of this wave: wave, wave + 4, ...
  const int nk = K / BK;
  const int my_nk = (nk - wave + 3) / 4;

  const int lr = lane >> 3, lc = lane & 7;
  const TileSource srcA(A + (size_t)m0 * lda), srcW(W + (size_t)n0 * ldw);
  unsigned pa[LA], pw[LW];   // per-lane byte offsets inside the tile's rows; instruction i covers tile rows 8i .. 8i+7
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    int r = i * 8 + lr;
    int c = lc ^ ((r >> 1) & 7);
    pa[i] = (unsigned)(((size_t)min(r, M - 1 - m0) * lda + c * 8) * 2);
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    int r = i * 8 + lr;
    int c = lc ^ ((r >> 1) & 7);
    pw[i] = (unsigned)(((size_t)min(r, N - 1 - n0) * ldw + c * 8) * 2);
  }
  auto issue = [&](int stage, int t) {   // t-th tile of this wave
    unsigned char *sa = ring + stage * STAGE_BYTES;
    unsigned char *sw = sa + BM * ROW_BYTES;
    const unsigned koff = (unsigned)(wave + 4 * t) * (BK * 2);
#pragma unroll
    for (int i = 0; i < LA; ++i) srcA.load16(pa[i], koff, sa + i * 1024);
#pragma unroll
    for (int i = 0; i < LW; ++i) srcW.load16(pw[i], koff, sw + i * 1024);
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  constexpr bool EPRE = EM == EM_RESIDUAL && BM * BN / 8 / 256 <= 2 && BM * BN / 8 >= 256;
  EpiOperands<BM, BN, 256> eops;
  if (my_nk > 0) issue(0, 0);
  if (my_nk > 1) issue(1, 1);
  // the epilogue's operands behind the first tiles, whose latency covers the address arithmetic (row / gate_seg)
  if constexpr (EPRE) eops.fetch(m0, n0, M, N, epi, vec_ok != 0);

  const int l32 = lane & 31, hi = lane >> 5;
  if constexpr (EPRE && NP == 2) wait_scalar_loads();
  for (int t = 0; t < my_nk; ++t) {
    if (t + 1 < my_nk) wait_vmcnt<LPS>(); else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    const unsigned char *st = ring + (t & 1) * STAGE_BYTES;
    bf16x8 af[2][MI], wf[2][NI];
    auto lread = [&](int buf, int ks) {
      const int c = ks * 2 + hi;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        int r = i * 32 + l32;
        af[buf][i] = *reinterpret_cast<const bf16x8 *>(st + r * ROW_BYTES + ((c ^ ((r >> 1) & 7)) << 4));
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        int r = j * 32 + l32;
        wf[buf][j] = *reinterpret_cast<const bf16x8 *>(st + (BM + r) * ROW_BYTES + ((c ^ ((r >> 1) & 7)) << 4));
      }
    };
    lread(0, 0);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      if (ks + 1 < BK / 16) lread((ks + 1) & 1, ks + 1);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks & 1][i], wf[ks & 1][j], acc[i][j], 0, 0, 0);
    }
    // this wave's LDS reads of the stage are complete (the MFMAs above consumed them): refill it
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (t + 2 < my_nk) issue(t & 1, t + 2);
  }

  // (in front of the loop, whose waits count tile loads, the bias costs: 704x1152x1152 7.6 us against 7.2, 1x12288x3072 GELU 16.8
  // against 16.1)
  ColumnBias<4, 1, bf16_t> column_bias;   // of the columns this thread sums
  column_bias.fetch(epi, n0 + (tid % (BN / 4)) * 4, N, vec_ok != 0);
  float bias[4];
  column_bias.widen(bias);
  // partial tiles -> LDS (each wave into its own ring), then sum of the four and epilogue
  float *part = reinterpret_cast<float *>(ring);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part[(i * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)) * TLD + j * 32 + l32] = acc[i][j][r];
  __syncthreads();
  float *p0 = reinterpret_cast<float *>(smem);
  constexpr int WSTRIDE = WAVE_BYTES / 4;
  static_assert(256 % (BN / 4) == 0, "a thread sums the same columns of every row");
  for (int e = tid; e < BM * BN / 4; e += 256) {
    int r = e / (BN / 4), c = (e % (BN / 4)) * 4;
    float4 s0 = *reinterpret_cast<const float4 *>(p0 + r * TLD + c);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      float4 s1 = *reinterpret_cast<const float4 *>(p0 + w * WSTRIDE + r * TLD + c);
      s0.x += s1.x; s0.y += s1.y; s0.z += s1.z; s0.w += s1.w;
    }
    s0.x += bias[0]; s0.y += bias[1]; s0.z += bias[2]; s0.w += bias[3];
    *reinterpret_cast<float4 *>(p0 + r * TLD + c) = s0;
  }
  __syncthreads();
  if constexpr (EPRE) tile_epilogue<EM, BM, BN, TLD, 256, true>(p0, m0, n0, M, N, epi, vec_ok != 0, &eops);
  else tile_epilogue<EM, BM, BN, TLD>(p0, m0, n0, M, N, epi, vec_ok != 0);
}

}  // namespace

// Host view of the workgroup -> tile map of a launch with BM x BN tiles (what workgroup `id` of the kernel computes):
// the grid size in *grid, and whether `id` has a tile (then in *tm, *tn).  For the unit test of the map.
bool gemm_tile_map(int M, int N, int BM, int BN, unsigned id, unsigned *grid, int *tm, int *tn) {
  GemmArgs a{};
  a.M = M; a.N = N;
  const int gx = xcd_cut(a, BM, BN, grid);
  if (id >= *grid) return false;
  return tile_of_id((int)id, (M + BM - 1) / BM, (N + BN - 1) / BN, gx, *tm, *tn);
}

// Readers behind the 64x64 tiles of a wave-split-K launch of one problem (see read_ahead), as many per XCD as it has idle CUs, up to
// 11, or up to 20 where the XCD's block of both operands, all of K, stays in its L2 (4 MB, the rest for what else the launch touches).
// Every one reads 1 / readers of the K tiles, whatever K is, so too few of them, or too many rows for each, end long after the
// multiplication would; too many run so far ahead that the L2 drops what they read.  us without and with readers:
//   at least five per XCD   5: 704x1152x4608 residual 20.8, 20.0   4: 256x3584x14336 60.7, 59.6, 448x2048x8192 32.2, 32.3   2: 320x3072x15360 63, 131
//   at most eleven          64x3072x15360, weights from HBM 66.7, 43.7 (8: 49.9, 26: 57.9), from the memory-side cache 45.1, 44.9 (8: 38.7, 26: 52.5);
//                           256x1152x4608 (3.9 MB), HBM 21.2, 14.4 (8: 16.1, 22: 14.9), 320x1536x6144, memory-side cache 21.7, 18.9 (8: 20.0, 17: 21.4)
//   at most twenty          64x6144x2048 (3.25 MB), HBM 13.0, 10.8 (11: 11.9, 14: 11.3), memory-side cache 9.2, 9.9 (11: 9.8);
//                           128x1152x4608 (3.4 MB) 22.5, 14.2 (11: 14.7) and 15.8, 13.9 (11: 13.6); 64x3072x3072 18.0, 11.6 (11: 12.1) and 12.4, 11.1 (11: 10.8)
//   a K tile of the block in two rounds of loads (24 tiles wide and high)   1x20 tiles: 64x10240x2560 19.8, 18.5   1x24: 64x12288x3072 22.4, 23.9
unsigned gemm_read_ahead_workgroups(int M, int N, int K) {
  constexpr int CUS = 256, TILE = 64, L2_KEEPS = 3584 * 1024;
  GemmArgs a{};
  a.M = M; a.N = N;
  unsigned grid = 0;
  const int gx = xcd_cut(a, TILE, TILE, &grid) & 255, gy = 8 / gx;
  if (grid >= CUS) return 0;
  const int bm = ((M + TILE - 1) / TILE + gx - 1) / gx, bn = ((N + TILE - 1) / TILE + gy - 1) / gy;
  const int most = (int64_t)(bm + bn) * TILE * K * 2 <= L2_KEEPS ? 20 : 11;
  const int readers = std::min((CUS - (int)grid) / 8, most);
  const bool two_rounds = 2 * (bm + bn) * TILE <= 2 * READ_AHEAD_LOADS * 256;
  return readers >= 5 && two_rounds ? 8 * readers : 0;
}

namespace {

// the rings, or the fp32 tile (row stride BN + 4) that replaces them for the epilogue, whichever is larger
constexpr int tile_lds_bytes(int BM, int BN, int NSTAGE, bool SPREAD) {
  const int ring = NSTAGE * (BM + BN) * ROW_BYTES, tile = BM * (BN + 4) * 4, dw = loop_depth_w(BM, BN, SPREAD);
  if (loop_half_tiles(BM, BN)) return HalfTiles256::SMEM;
  if (dw) return (NSTAGE * BM + dw * BN) * ROW_BYTES;
  return (tile > ring && tile <= 96 * 1024) ? tile : ring;   // larger tiles finish in row passes
}

// PINNED: a configuration that only pf_op_gemm_tile asks for (one problem, no K/V route); ROUTE: the rule takes it for K/V routes too
template <int BM, int BN, int NSTAGE, int WGM = 2, int WGN = 2, bool SPREAD = false, bool PINNED = false, bool ROUTE = !PINNED>
hipError_t launch_tile(const GemmArgs &a, const GemmArgs *b, hipStream_t s) {
  constexpr int smem = tile_lds_bytes(BM, BN, NSTAGE, SPREAD);
  auto go = [&](auto np, auto em) -> hipError_t {
    constexpr int NP = decltype(np)::value, EM = decltype(em)::value;
    if constexpr ((PINNED && NP == 2) || (!ROUTE && EM == EM_KV_ROUTE)) {
      return hipErrorInvalidValue;
    } else {
      constexpr auto kernel = &gemm_tile_kernel<NP, EM, BM, BN, NSTAGE, WGM, WGN, SPREAD>;
      if (hipError_t e = allow_dynamic_lds<kernel, smem>(); e != hipSuccess) return e;
      GemmLaunch<bf16_t, NP> L;
      const unsigned grid = make_launch(a, b, BM, BN, &L);
      kernel<<<grid, 64 * WGM * WGN, smem, s>>>(L);
      return hipGetLastError();
    }
  };
  return for_launch_form(a, b, go);
}

template <int BM, int BN>
hipError_t launch_wavek(const GemmArgs &a, const GemmArgs *b, hipStream_t s) {
  constexpr int smem = 4 * 2 * (BM + BN) * ROW_BYTES;
  auto go = [&](auto np, auto em) -> hipError_t {
    constexpr int NP = decltype(np)::value, EM = decltype(em)::value;
    constexpr auto kernel = &gemm_wavek_kernel<NP, EM, BM, BN>;
    if (hipError_t e = allow_dynamic_lds<kernel, smem>(); e != hipSuccess) return e;
    GemmLaunch<bf16_t, NP> L;
    const unsigned grid = make_launch(a, b, BM, BN, &L);
    static_assert(BM == 64 && BN == 64, "gemm_read_ahead_workgroups");
    const unsigned ahead = NP == 1 ? gemm_read_ahead_workgroups(a.M, a.N, a.K) : 0;
    kernel<<<grid + ahead, 256, smem, s>>>(L);
    return hipGetLastError();
  };
  return for_launch_form(a, b, go);
}

}  // namespace

bool gemm_kv_route_supported(const GemmArgs &a) {
  const bool kernel = a.dt == DT_BF16 ? a.path != PATH_SIMT && a.K % BK == 0 && a.K >= BK : gemm_mfma_f32_supported(a);
  // per-head norm: bf16 tiles come in widths of 64 and 128 columns (pick_variant sees to it); the lanes of a head exchange
  // their sums, so its groups of eight channels have to be a power of two; the scales are read sixteen bytes at a time
  const int groups = a.kvr.dh / 8;
  if (a.kvr.q_norm && (a.dt != DT_BF16 || groups > 16 || (groups & (groups - 1)) || (((uintptr_t)a.kvr.q_norm | (uintptr_t)a.kvr.k_norm) & 15)))
    return false;
  return kernel && a.epilogue == 0 && a.N % 8 == 0 && vec_epilogue_ok(a) && a.kvr.dh % 8 == 0 && a.kvr.d % 8 == 0 && a.N == 3 * a.kvr.d;
}

// (the tile loads address a tile's rows with 32-bit byte offsets inside a 2 GB window: 256 rows of either operand must fit)
bool gemm_mfma_dl_supported(const GemmArgs &a) {
  const int64_t ld = a.lda > a.ldw ? a.lda : a.ldw;
  return a.K % BK == 0 && a.K >= BK && a.M >= 1 && a.N >= 1 && (256 * ld + a.K) * 2 < 0x7ffffff0LL;
}

// Tile choice.
//
// Launches with enough tiles to fill the chip (512 of 128x64, or long K and 128 of 256x128): the candidate with the least
//   rounds x (us x (K tiles + fill) + epilogue)
// rounds = padded grid / 256 CUs.  The grid counts, not the tiles: an XCD's block of the tile grid is padded to whole rows and
// columns, and 52 x 9 tiles of 64x128 cut into blocks of 13 x 5 take one more round than fits on every XCD (3306x1152x4608: 85 us
// against 65).  us, fill (the start-up, in K tiles) and the epilogues' us are fitted (least squares of the relative error) to
// isolated GEMMs whose weights no cache holds, each shape with every tile: those of 256x256, 256x192 and 256x128 to 330 shapes of
// 259 .. 16896 rows at widths of 384 .. 3072, the others to 290 such shapes of an earlier run, whose mean they still meet within 5 %
// (64x128, 6 % low on plain stores, has fill and us raised until 431x9216x3072 goes to the three-stage tile, 37 us against 42).  us1
// and fill1 hold where one workgroup has a CU to itself; an epilogue weighs most where no second one runs beside it.  The K/V
// route's us are what 30 QKV launches inside stages (812 .. 16896 rows; with and without per-head norm and RoPE) take beyond that, the
// median per round; 256x128 is no candidate for it: at 640, 1562 and 1664 x 9216 x 3072, where that price chose it, the call took 2, 8 and
// 9 us a layer longer than with 128x128, and it was the fastest at none of 50 launches.
// Over 450 shapes (120 of them not of the fit) the choice is 0.9 % off the fastest tile on average, 24 % at most (128x64 in two rounds
// of long K: 1956x2048x8192 residual 97 us, 64x128 80); over 50 calls with each QKV tile 0.1 % of the call, 1.6 % at most.  Measured (us; * =
// chosen), the table and the figures of the list below in one run (pairs of figures elsewhere are of runs of their own; boxes differ by 3 %):
//                                     256x256  256x192  256x128  128x192  3-stage  128x128   128x64   64x128
//     2048 x   9216 x   3072 store         129      112      118     110*      116      129      147      166
//     2048 x  12288 x   3072 GELU          146     133*      142      154      171      152      200      214
//     2048 x   3072 x  15360 residual      277      246      189      242     179*      223      254      290
//     2560 x   9216 x   3072 store         132     120*      131      138      150      139      193      206
//     2560 x  12288 x   3072 GELU         156*      185      180      185      208      189      245      262
//     2560 x   3072 x  15360 residual      281      249     201*      297      319      225      376      328
//    16896 x   9216 x   3072 store        726*      799      852      826      924      893     1135     1183
//    16896 x  12288 x   3072 GELU        1017*     1111     1193     1152     1355     1241     1509     1610
//    16896 x   3072 x  15360 residual    1362*     1513     1528     1555     1667     1694     2056     2203
//     4096 x   3456 x   1152 store       33.5*     47.2     40.4     45.1     50.5     39.8     49.3     53.0
//     4096 x   4608 x   1152 GELU         67.0     59.5     63.1    57.0*     65.9     63.4     61.7     72.7
//     4096 x   1152 x   4608 residual     90.6     80.6     62.3     78.6    58.8*     68.3     70.3     85.1
//     4096 x   1152 x   1152 residual     34.5     29.8     23.5     26.0     23.1     22.3    23.9*     28.6
//     2882 x   2048 x  10240 residual      171      160     118*      196      195      141      161      194
// The three-stage 128x192 tile issues its prefetch loads one at a time between the MFMAs (instead of in a burst behind the
// barrier): 2048x3072x15360 204 -> 183 us, 4096x1152x4608 65 -> 55 us; every other tile loses by it or keeps nothing of the
// gain inside a stage.
//
// Fewer tiles (patches of a few hundred rows), by counts of 64x64 tiles:
//  * the wave-split-K kernel, one workgroup per CU (128 KB of LDS): up to one tile per CU, from K = 1024 on.  512x1152x1152
//    residual 7.7 us (four-stage 64x64: 8.4), 512x1152x4608 15.7 (24.0), 512x1536x6144 22.0 (31.9), with their read-ahead (without:
//    8.6, 20.2, 26.0), 512x1152x768 6.9 (6.9); with more tiles than CUs it loses: 1024x1152x4608 34.4 (29.0) - until the second
//    round of its workgroups is nearly full too and K is long: 633x3072x15360 107 (120; 432 tiles: 108 against 93), 1275x1536x6144
//    44.8 (50.2), 633x3072x3072 27.4 (28.7), 1275x1536x1536 17.4 (16.4).
//  * 64x64 with four stages while every workgroup of the padded grid is resident at once (two per CU), 375x4608x1536 13.7 us
//    (two stages 19.5); 1339x1536x6144, 21 x 24 tiles in a grid of 528, 63 us (64x128 51);
//  * beyond, 64x128 with three stages under the same condition, where its rounds (of 256 tiles) are no more work than those
//    of 64x64 tiles or K is long enough to pay for it: 1024x3456x1152 15.3 us, 512x6144x1536 with GELU 19.7, 512x4608x1536 17.4, against
//    19.4, 22.1 and 20.0 with two-stage 64x64 tiles, which take what is left (512x4608x1152 with GELU inside a stage, whose K is not
//    long: 16.1 us, with 64x128 17.4, though alone 16.8 and 14.3; 512x4608x1536 with a residual and an unaligned bias 28 us, with 64x128 32).
// 64x64 with three stages is there for pf_op_gemm_tile only: the rule never takes it.
enum { V_256x256 = 0, V_64x128_S3, V_256x128_S3, V_128x128, V_128x64, V_WAVEK, V_64x64_S4, V_64x64_S3, V_64x64_S2,
       V_128x192_S2, V_256x192_S2, V_128x192_S3, V_COUNT };

static int pick_variant(const GemmArgs &a, const GemmArgs *b = nullptr) {
  auto tiles = [&](int bm, int bn) { return launch_tiles(a, b, bm, bn); };
  auto grid = [&](int bm, int bn) -> int64_t {
    unsigned ga = 0, gb = 0;
    xcd_cut(a, bm, bn, &ga);
    if (b) xcd_cut(*b, bm, bn, &gb);
    return (int64_t)ga + gb;
  };
  // per-head norm in the epilogue: heads of 128 channels need tiles of 128 or 256 columns
  const bool wide_heads = a.kvr.q_norm && a.kvr.dh > 64;
  // operands that are not aligned for vectors have an element-wise epilogue (`odd` us per round, with a residual 2.6 times that)
  const bool odd = !vec_epilogue_ok(a) || (b && !vec_epilogue_ok(*b));
  if (tiles(128, 64) >= 512 || (a.K >= 4096 && tiles(256, 128) >= 128)) {
    struct Candidate { int v, bm, bn; double us1, fill1, us, fill, gelu, residual, route, odd; };   // us1, fill1: one round
    static constexpr Candidate cand[] = {
        {V_256x256, 256, 256, 1.07, 9.3, 1.34, 5.2, 5.3, 7.8, 16.0, 31.0}, {V_256x192_S2, 256, 192, 0.95, 9.5, 1.13, 5.6, 4.3, 6.7, 15.0, 27.0},
        {V_256x128_S3, 256, 128, 0.71, 10.5, 0.79, 6.8, 2.6, 5.4, 0.0, 16.0}, {V_128x192_S2, 128, 192, 0.90, 8, 0.65, 5, 2.5, 5.0, 8.5, 16.0},
        {V_128x192_S3, 128, 192, 0.64, 11, 0.65, 9, 5.0, 7.5, 11.5, 22.0}, {V_128x128, 128, 128, 0.80, 6, 0.45, 6, 1.5, 3.5, 5.5, 10.0},
        {V_128x64, 128, 64, 0.76, 0, 0.31, 4, 0.4, 1.7, 2.0, 2.7},       {V_64x128_S3, 64, 128, 0.46, 9, 0.34, 8, 0.7, 2.0, 2.0, 4.6}};
    const int form = gemm_epilogue_form(a);
    int best = V_128x128;
    double best_cost = 1e300;
    for (const Candidate &c : cand) {
      if ((wide_heads && c.bn % 128) || (form == EM_KV_ROUTE && c.v == V_256x128_S3)) continue;
      const int64_t rounds = (grid(c.bm, c.bn) + 255) / 256;
      const double epilogue = odd ? c.odd * (form == EM_RESIDUAL ? 2.6 : 1.0)
                                  : form == EM_KV_ROUTE ? c.route : form == EM_RESIDUAL ? c.residual : a.gelu_from < a.N ? c.gelu : 0.0;
      const double cost = rounds * ((rounds == 1 ? c.us1 * (a.K / BK + c.fill1) : c.us * (a.K / BK + c.fill)) + epilogue);
      if (cost < best_cost) { best_cost = cost; best = c.v; }
    }
    return best;
  }
  if (wide_heads) return V_64x128_S3;
  const int64_t t64 = tiles(64, 64);
  if (t64 <= g_wavek_max_tiles && a.K >= g_wavek_min_k) return V_WAVEK;
  if (grid(64, 64) <= 512) return t64 >= 472 && a.K >= 2560 ? V_WAVEK : V_64x64_S4;
  const bool even = (tiles(64, 128) + 255) / 256 * 2 <= (t64 + 255) / 256;
  return grid(64, 128) <= 512 && (even || a.K >= 1536) && !odd ? V_64x128_S3 : V_64x64_S2;
}

static hipError_t launch_variant(int v, const GemmArgs &a, const GemmArgs *b, hipStream_t s) {
  switch (v) {
    case V_256x256: return launch_tile<256, 256, 2, 4, 2>(a, b, s);
    case V_64x128_S3: return launch_tile<64, 128, 3>(a, b, s);
    case V_256x128_S3: return launch_tile<256, 128, 3, 4, 2, false, false, false>(a, b, s);
    case V_128x128: return launch_tile<128, 128, 2>(a, b, s);
    case V_128x64: return launch_tile<128, 64, 2>(a, b, s);
    case V_WAVEK: return launch_wavek<64, 64>(a, b, s);
    case V_64x64_S4: return launch_tile<64, 64, 4>(a, b, s);
    case V_64x64_S3: return launch_tile<64, 64, 3, 2, 2, false, true>(a, b, s);
    case V_128x192_S2: return launch_tile<128, 192, 2>(a, b, s);
    case V_256x192_S2: return launch_tile<256, 192, 2, 4, 2>(a, b, s);
    case V_128x192_S3: return launch_tile<128, 192, 3, 2, 2, true>(a, b, s);
    default: return launch_tile<64, 64, 2>(a, b, s);
  }
}

// configurations a caller can pin
int gemm_mfma_dl_tile_count() { return V_COUNT; }

hipError_t launch_gemm_mfma_dl(const GemmArgs &a, hipStream_t s, const GemmArgs *b) {
#ifdef PF_TUNING
  // tile configurations outside the heuristic's set, for sweeps
  switch (g_gemm_tile_override) {
    case 1: return launch_tile<256, 128, 3>(a, b, s);
    case 2: return launch_tile<128, 128, 3>(a, b, s);
    case 3: return launch_tile<128, 128, 2>(a, b, s);
    case 4: return launch_tile<128, 64, 4>(a, b, s);
    case 5: return launch_tile<64, 64, 4>(a, b, s);
    case 6: return launch_tile<256, 128, 2>(a, b, s);
    case 7: return launch_tile<128, 64, 2>(a, b, s);
    case 8: return launch_tile<64, 64, 2>(a, b, s);
    case 10: return launch_wavek<64, 64>(a, b, s);
    case 14: return launch_tile<256, 128, 3, 4, 2>(a, b, s);
    case 15: return launch_tile<256, 256, 2, 4, 2>(a, b, s);
    case 16: return launch_tile<128, 256, 3, 2, 4>(a, b, s);
    case 17: return launch_tile<256, 128, 2, 4, 2>(a, b, s);
    case 27: return launch_tile<128, 64, 3>(a, b, s);
    case 28: return launch_tile<128, 192, 2>(a, b, s);
    case 29: return launch_tile<256, 192, 2, 4, 2>(a, b, s);
    case 30: return launch_tile<128, 192, 3>(a, b, s);
    case 31: return launch_tile<64, 128, 3>(a, b, s);
    case 40: return launch_tile<128, 192, 2, 2, 2, true>(a, b, s);
    case 41: return launch_tile<256, 192, 2, 4, 2, true>(a, b, s);
    case 42: return launch_tile<128, 192, 3, 2, 2, true>(a, b, s);
    case 43: return launch_tile<256, 256, 2, 4, 2, true>(a, b, s);
    case 44: return launch_tile<256, 128, 3, 4, 2, true>(a, b, s);
    case 45: return launch_tile<128, 128, 2, 2, 2, true>(a, b, s);
    case 46: return launch_tile<128, 192, 4, 2, 2, true>(a, b, s);
    case 47: return launch_tile<128, 128, 3, 2, 2, true>(a, b, s);
    case 48: return launch_tile<128, 128, 4, 2, 2, true>(a, b, s);
    case 49: return launch_tile<128, 64, 4, 2, 2, true>(a, b, s);
    case 50: return launch_tile<64, 64, 4, 2, 2, true>(a, b, s);
    case 51: return launch_tile<128, 256, 3, 2, 2, true>(a, b, s);
    case 52: return launch_tile<128, 192, 3, 2, 2, false>(a, b, s);
    default: break;
  }
#endif
  if (a.tile >= 1 && a.tile <= gemm_mfma_dl_tile_count()) return launch_variant(a.tile - 1, a, b, s);
  return launch_variant(pick_variant(a, b), a, b, s);
}

const char *gemm_mfma_dl_variant_name(const GemmArgs &a) {
  static const char *names[V_COUNT] = {"gemm_tile_kernel<256,256,2,4,2,false>", "gemm_tile_kernel<64,128,3,2,2,false>",
                                       "gemm_tile_kernel<256,128,3,4,2,false>", "gemm_tile_kernel<128,128,2,2,2,false>",
                                       "gemm_tile_kernel<128,64,2,2,2,false>", "gemm_wavek_kernel<64,64>",
                                       "gemm_tile_kernel<64,64,4,2,2,false>", "gemm_tile_kernel<64,64,3,2,2,false>",
                                       "gemm_tile_kernel<64,64,2,2,2,false>", "gemm_tile_kernel<128,192,2,2,2,false>",
                                       "gemm_tile_kernel<256,192,2,4,2,false>", "gemm_tile_kernel<128,192,3,2,2,true>"};
  return names[(a.tile >= 1 && a.tile <= gemm_mfma_dl_tile_count()) ? a.tile - 1 : pick_variant(a)];
}

}  // namespace pf
