// fp32 MFMA GEMMs with direct global->LDS loads (gfx950): C = epilogue(A W^T + bias), A [M,K], W [N,K] fp32, both
// contiguous along K, K a multiple of 32.
//
// Bound by the fp32 matrix rate (157 TFLOP/s; the vector unit without packed arithmetic reaches half of that).  A K tile is
// 32 floats = 128 bytes of a row, so the LDS rows, the tile loads and the XOR swizzle are byte for byte those of the bf16
// kernels (gemm_mfma_dl.hip).  A fragment is one 16-byte LDS read per lane: lanes 0..31 get k = 8s .. 8s+3 of their row,
// lanes 32..63 k = 8s+4 .. 8s+7, and four v_mfma_f32_32x32x2_f32 take one float of each half at a time; A and W are
// permuted along k alike, so the sum is the plain one in another order.  An MFMA takes 64 cycles, a fragment read feeds at
// least four of them, and neither LDS nor the barriers show.
//
//  * gemm_f32_tile_kernel: WGM x WGN wavefronts on one tile, NSTAGE-deep ring, one barrier per K tile.
//  * gemm_f32_wavek_kernel: NW wavefronts split K, each with a private two-stage ring and no barrier in the loop; partial
//    tiles are summed through LDS.  For launches with too few tiles to fill the chip.
#include "gemm_tile.h"

namespace pf {

namespace {

constexpr int KB = 32;                // K elements per tile
constexpr int ROW_BYTES = KB * 4;     // 128
constexpr int KSTEPS = KB / 8;        // fragment reads per K tile

template <int N>
__device__ __forceinline__ void mma8(const f32x4 (&a)[N], const f32x4 &w, f32x16 (&acc)[N]) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], w[e], acc[i], 0, 0, 0);
}

template <int NP, int EM, int BM, int BN, int NSTAGE, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_f32_tile_kernel(GemmLaunch<float, NP> L) {
  const bool second = NP == 2 && blockIdx.x >= L.grid0;
  const GemmProblem<float> &prob = L.p[second ? 1 : 0];
  const float *__restrict__ A = prob.A, *__restrict__ W = prob.W;
  const int64_t lda = prob.lda, ldw = prob.ldw;
  const int M = prob.M, N = L.N, K = L.K;
  const Epilogue<float> &epi = prob.epi;
  const int vec_ok = prob.vec_ok;
  constexpr int NW = WGM * WGN, WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NI = WN / 32;
  constexpr int LA = BM / 8 / NW, LW = BN / 8 / NW, LPS = LA + LW;   // load instructions (8 rows each) per wave and K tile
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile rows must split evenly over the waves' load instructions");
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES, TLD = BN + 4;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  int tm, tn;
  if (!tile_of_id((int)(blockIdx.x - (second ? L.grid0 : 0)), (M + BM - 1) / BM, (N + BN - 1) / BN, prob.xcd_gx, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;

  const TileSource srcA(A + (size_t)m0 * lda), srcW(W + (size_t)n0 * ldw);
  unsigned pa[LA], pw[LW];   // per-lane byte offsets (rows past the matrix repeat its last row)
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (i * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    pa[i] = (unsigned)(((size_t)min(r, M - 1 - m0) * lda + c * 4) * 4);
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int r = (i * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    pw[i] = (unsigned)(((size_t)min(r, N - 1 - n0) * ldw + c * 4) * 4);
  }
  auto issue = [&](int stage, int kt) {
    unsigned char *sa = smem + stage * STAGE_BYTES, *sw = sa + BM * ROW_BYTES;
    const unsigned koff = (unsigned)kt * ROW_BYTES;
#pragma unroll
    for (int i = 0; i < LA; ++i) srcA.load16(pa[i], koff, sa + (i * NW + wave) * 1024);
#pragma unroll
    for (int i = 0; i < LW; ++i) srcW.load16(pw[i], koff, sw + (i * NW + wave) * 1024);
  };

  f32x16 acc[NI][MI];
#pragma unroll
  for (int j = 0; j < NI; ++j)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  const int nk = K / KB;
#pragma unroll
  for (int s = 0; s < NSTAGE - 1; ++s)
    if (s < nk) issue(s, s);

  const int l32 = lane & 31, hi = lane >> 5;
  for (int kt = 0; kt < nk; ++kt) {
    wait_tiles_behind<LPS, NSTAGE - 2>(min(NSTAGE - 2, nk - 1 - kt));
    __builtin_amdgcn_s_barrier();   // (not __syncthreads, which would drain the prefetches)
    asm volatile("" ::: "memory");
    if (kt + NSTAGE - 1 < nk) issue((kt + NSTAGE - 1) % NSTAGE, kt + NSTAGE - 1);
    const unsigned char *st = smem + (kt % NSTAGE) * STAGE_BYTES;
    f32x4 af[2][MI], wf[2][NI];
    auto lread = [&](int buf, int ks) {
      const int c = ks * 2 + hi;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r = wm * WM + i * 32 + l32;
        af[buf][i] = *reinterpret_cast<const f32x4 *>(st + r * ROW_BYTES + ((c ^ ((r >> 1) & 7)) << 4));
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int r = wn * WN + j * 32 + l32;
        wf[buf][j] = *reinterpret_cast<const f32x4 *>(st + (BM + r) * ROW_BYTES + ((c ^ ((r >> 1) & 7)) << 4));
      }
    };
    lread(0, 0);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      if (ks + 1 < KSTEPS) lread((ks + 1) & 1, ks + 1);
#pragma unroll
      for (int j = 0; j < NI; ++j) mma8<MI>(af[ks & 1], wf[ks & 1][j], acc[j]);
    }
  }

  // (in front of the loop, whose waits count tile loads, the bias costs: 2423x2048x2048 197 us against 166, 512x3456x1152 42.5 against
  // 40.8, 2944x1152x4608 residual 313 against 296)
  ColumnBias<NI, 32, float> column_bias;
  column_bias.fetch(epi, n0 + wn * WN + (lane & 31), N);
  float bias[NI];
  column_bias.widen(bias);
  // accumulators -> row-major tile in LDS (lane -> column l32, register r -> row 8*(r/4) + 4*hi + r%4)
  float *tile = reinterpret_cast<float *>(smem);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        tile[(wm * WM + i * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)) * TLD + wn * WN + j * 32 + l32] = acc[j][i][r] + bias[j];
  __syncthreads();
  tile_epilogue<EM, BM, BN, TLD, 64 * NW>(tile, m0, n0, M, N, epi, vec_ok != 0);
}

template <int NP, int EM, int BM, int BN, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_f32_wavek_kernel(GemmLaunch<float, NP> L) {
  const bool second = NP == 2 && blockIdx.x >= L.grid0;
  const GemmProblem<float> &prob = L.p[second ? 1 : 0];
  const float *__restrict__ A = prob.A, *__restrict__ W = prob.W;
  const int64_t lda = prob.lda, ldw = prob.ldw;
  const int M = prob.M, N = L.N, K = L.K;
  const Epilogue<float> &epi = prob.epi;
  const int vec_ok = prob.vec_ok;
  constexpr int MI = BM / 32, NI = BN / 32, LA = BM / 8, LW = BN / 8, LPS = LA + LW;   // a wave loads whole tiles
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES, WAVE_BYTES = 2 * STAGE_BYTES, TLD = BN + 4, NT = 64 * NW;
  static_assert(WAVE_BYTES >= BM * TLD * 4, "a wave's partial tile must fit in its own ring");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  if (!tile_of_id((int)(blockIdx.x - (second ? L.grid0 : 0)), (M + BM - 1) / BM, (N + BN - 1) / BN, prob.xcd_gx, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  unsigned char *ring = smem + wave * WAVE_BYTES;
  const int nk = K / KB, my_nk = (nk - wave + NW - 1) / NW;   // K tiles wave, wave + NW, ...

  const TileSource srcA(A + (size_t)m0 * lda), srcW(W + (size_t)n0 * ldw);
  unsigned pa[LA], pw[LW];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = i * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    pa[i] = (unsigned)(((size_t)min(r, M - 1 - m0) * lda + c * 4) * 4);
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int r = i * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    pw[i] = (unsigned)(((size_t)min(r, N - 1 - n0) * ldw + c * 4) * 4);
  }
  auto issue = [&](int stage, int t) {   // t-th tile of this wave
    unsigned char *sa = ring + stage * STAGE_BYTES, *sw = sa + BM * ROW_BYTES;
    const unsigned koff = (unsigned)(wave + NW * t) * ROW_BYTES;
#pragma unroll
    for (int i = 0; i < LA; ++i) srcA.load16(pa[i], koff, sa + i * 1024);
#pragma unroll
    for (int i = 0; i < LW; ++i) srcW.load16(pw[i], koff, sw + i * 1024);
  };

  f32x16 acc[NI][MI];
#pragma unroll
  for (int j = 0; j < NI; ++j)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  if (my_nk > 0) issue(0, 0);
  if (my_nk > 1) issue(1, 1);
  const int l32 = lane & 31, hi = lane >> 5;
  for (int t = 0; t < my_nk; ++t) {
    if (t + 1 < my_nk) wait_vmcnt<LPS>(); else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    const unsigned char *st = ring + (t & 1) * STAGE_BYTES;
    f32x4 af[KSTEPS][MI], wf[KSTEPS][NI];   // the whole tile: its stage can be refilled while the MFMAs run
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      const int c = ks * 2 + hi;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r = i * 32 + l32;
        af[ks][i] = *reinterpret_cast<const f32x4 *>(st + r * ROW_BYTES + ((c ^ ((r >> 1) & 7)) << 4));
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int r = j * 32 + l32;
        wf[ks][j] = *reinterpret_cast<const f32x4 *>(st + (BM + r) * ROW_BYTES + ((c ^ ((r >> 1) & 7)) << 4));
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // every fragment is in registers
    if (t + 2 < my_nk) issue(t & 1, t + 2);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks)
#pragma unroll
      for (int j = 0; j < NI; ++j) mma8<MI>(af[ks], wf[ks][j], acc[j]);
  }

  // the epilogue's operands: their latency runs under the exchange through LDS.  Residual and gate only with eight waves, that is
  // with tiles for few of the CUs (tiny stage 43.9 -> 43.6 us a call); four waves have a neighbour on their CU to hide it
  // (PixArt-scale fp32 call 396 -> 403 us with them, 412 with them in front of the K loop).
  constexpr bool EPRE = EM == EM_RESIDUAL && NW == 8;
  EpiOperands<BM, BN, NT> eops;
  if constexpr (EPRE) eops.fetch(m0, n0, M, N, epi, vec_ok != 0);
  ColumnBias<4, 1, float> column_bias;   // of the columns this thread sums
  column_bias.fetch(epi, n0 + (tid % (BN / 4)) * 4, N, vec_ok != 0);

  // partial tiles -> LDS (each wave into its own ring), sum in wave order, epilogue
  float *part = reinterpret_cast<float *>(ring);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part[(i * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)) * TLD + j * 32 + l32] = acc[j][i][r];
  __syncthreads();
  float bias[4];
  column_bias.widen(bias);
  float *p0 = reinterpret_cast<float *>(smem);
  constexpr int WSTRIDE = WAVE_BYTES / 4;
  static_assert(NT % (BN / 4) == 0, "a thread sums the same columns of every row");
  for (int e = tid; e < BM * BN / 4; e += NT) {
    const int r = e / (BN / 4), c = (e % (BN / 4)) * 4;
    float4 s0 = *reinterpret_cast<const float4 *>(p0 + r * TLD + c);
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const float4 s1 = *reinterpret_cast<const float4 *>(p0 + w * WSTRIDE + r * TLD + c);
      s0.x += s1.x; s0.y += s1.y; s0.z += s1.z; s0.w += s1.w;
    }
    s0.x += bias[0]; s0.y += bias[1]; s0.z += bias[2]; s0.w += bias[3];
    *reinterpret_cast<float4 *>(p0 + r * TLD + c) = s0;
  }
  __syncthreads();
  if constexpr (EPRE) tile_epilogue<EM, BM, BN, TLD, NT, true>(p0, m0, n0, M, N, epi, vec_ok != 0, &eops);
  else tile_epilogue<EM, BM, BN, TLD, NT>(p0, m0, n0, M, N, epi, vec_ok != 0);
}

template <int BM, int BN, int NSTAGE, int WGM, int WGN>
hipError_t launch_tile(const GemmArgs &a, const GemmArgs *b, hipStream_t s) {
  constexpr int ring = NSTAGE * (BM + BN) * ROW_BYTES, tile = BM * (BN + 4) * 4, smem = tile > ring ? tile : ring;
  auto go = [&](auto np, auto em) -> hipError_t {
    constexpr int NP = decltype(np)::value, EM = decltype(em)::value;
    constexpr auto kernel = &gemm_f32_tile_kernel<NP, EM, BM, BN, NSTAGE, WGM, WGN>;
    if (hipError_t e = allow_dynamic_lds<kernel, smem>(); e != hipSuccess) return e;
    GemmLaunch<float, NP> L;
    const unsigned grid = make_launch(a, b, BM, BN, &L);
    kernel<<<grid, 64 * WGM * WGN, smem, s>>>(L);
    return hipGetLastError();
  };
  return for_launch_form(a, b, go);
}

template <int BM, int BN, int NW>
hipError_t launch_wavek(const GemmArgs &a, const GemmArgs *b, hipStream_t s) {
  constexpr int smem = NW * 2 * (BM + BN) * ROW_BYTES;
  auto go = [&](auto np, auto em) -> hipError_t {
    constexpr int NP = decltype(np)::value, EM = decltype(em)::value;
    constexpr auto kernel = &gemm_f32_wavek_kernel<NP, EM, BM, BN, NW>;
    if (hipError_t e = allow_dynamic_lds<kernel, smem>(); e != hipSuccess) return e;
    GemmLaunch<float, NP> L;
    const unsigned grid = make_launch(a, b, BM, BN, &L);
    kernel<<<grid, 64 * NW, smem, s>>>(L);
    return hipGetLastError();
  };
  return for_launch_form(a, b, go);
}

enum { F_64x64 = 0, F_WAVEK4, F_WAVEK8, F_COUNT };

// Tile rule, from isolated launches (us; 64x64 | 32x32 with K over 4 waves | over 8):
//  * 64x64 from 384 tiles on: 512x3456x1152 45 | 50 | 53, 2048x3072x3072 304 | 339 | 379, 2048x9216x3072 886 | 1028 | 1138
//    (131 TFLOP/s).  128x128 tiles never beat it (2048x9216x3072 925).
//  * below, 32x32 tiles with K over four waves: 512x1152x1152 27 | 21 | 23, 512x1152x4608 97 | 67 | 68, 375x1536x1536
//    34 | 25 | 27, 77x4608x1536 34 | 17 | 19;
//  * over eight waves for at most one tile per CU and for very long K, where the serial chain is the bound:
//    256x3072x15360 313 | 252 | 207, 375x1536x6144 129 | 88.5 | 86.
// The plain kernel (gemm_simt.hip) took 85 us for 512x3456x1152 and 129 us on average for the four 512-row GEMMs into 1152
// columns of a PixArt-scale block.
int pick_variant(const GemmArgs &a, const GemmArgs *b = nullptr) {
  auto tiles = [&](int bm, int bn) { return launch_tiles(a, b, bm, bn); };
  if (tiles(64, 64) >= 384) return F_64x64;
  return tiles(32, 32) > 256 && a.K < 6144 ? F_WAVEK4 : F_WAVEK8;
}

}  // namespace

// K a multiple of the K tile, operand rows 16-byte aligned for the tile loads, and 256 rows of either operand inside the
// 2 GB window of 32-bit byte offsets; every other fp32 GEMM stays with the plain kernel.
bool gemm_mfma_f32_supported(const GemmArgs &a) {
  const int64_t ld = a.lda > a.ldw ? a.lda : a.ldw;
  return a.dt == DT_F32 && a.path != PATH_SIMT && a.K % KB == 0 && a.K >= KB && a.M >= 1 && a.N >= 1 && a.lda % 4 == 0 &&
         a.ldw % 4 == 0 && (((uintptr_t)a.A | (uintptr_t)a.W) & 15) == 0 && (256 * ld + a.K) * 4 < 0x7ffffff0LL;
}

const char *gemm_mfma_f32_variant_name(const GemmArgs &a) {
  static const char *names[F_COUNT] = {"gemm_f32_tile_kernel<64,64,3,2,2>", "gemm_f32_wavek_kernel<32,32,4>",
                                       "gemm_f32_wavek_kernel<32,32,8>"};
  return names[pick_variant(a)];
}

hipError_t launch_gemm_mfma_f32(const GemmArgs &a, hipStream_t s, const GemmArgs *b) {
  switch (pick_variant(a, b)) {
    case F_64x64: return launch_tile<64, 64, 3, 2, 2>(a, b, s);
    case F_WAVEK4: return launch_wavek<32, 32, 4>(a, b, s);
    default: return launch_wavek<32, 32, 8>(a, b, s);
  }
}

}  // namespace pf
