// bf16 MFMA GEMM body of the 256x192 and 256x128 tiles: C = epilogue(A W^T + bias), K a multiple of 64.
//
// WGM x WGN wavefronts on one tile; a ring of DA K tiles (64 wide) of A and one of DW of W in LDS, the deeper one for W because
// its rows come from farther away (nothing has read a layer's weights since the last call).  A K tile is four slices of 16:
// the MFMAs of a slice run on fragments read during the slice before, and the reads and the loads go between the MFMAs.
// One barrier a K tile, in front of its last slice: by then every wave has read all of the tile, whose place is loaded again from
// there on, and the next tile has landed for every wave, whose first slice is read next.
//
// What bounds it: power and, for the smaller tiles, the path from the L2s into the CUs (gemm_mfma_dl.hip has the figures of the
// loop it replaces).  2048x12288x3072 GELU, 256x192: 154 -> 136 us; 2048x9216x3072, 256x192 132 -> 113;
// 2560x3072x15360 residual, 256x128: 241 -> 204 us.  Four waves with a quarter of a 256x256 tile each (128 KB of fragment
// reads a K tile instead of 192) multiply 2 - 5 % faster but finish a tile 10 us later: one wave per SIMD has nothing beside
// its epilogue's latencies (16896x12288x3072 GELU 1132 us against 1033).
#pragma once
#include "gemm_tile.h"

namespace pf {

namespace {

template <int BM, int BN, int DA, int DW>
struct RingShape {
  static constexpr int A_BYTES = BM * 128, W_BYTES = BN * 128;   // a K tile of either operand
  static constexpr int RING = DA * A_BYTES + DW * W_BYTES;
  static constexpr int TLD = BN + 4;
  static constexpr int RB = BM * TLD * 4 <= RING ? BM : BM / 2;      // rows of an epilogue pass
  static constexpr int SMEM = RING;
  static_assert(SMEM <= 160 * 1024 && RB * TLD * 4 <= RING && DA >= 2 && DW >= DA, "rings");
};

template <int NP, int EM, int BM, int BN, int WGM, int WGN, int DA, int DW>
__device__ __forceinline__ void gemm_ring_body(const GemmLaunch<bf16_t, NP> &L, unsigned char *smem) {
  using S = RingShape<BM, BN, DA, DW>;
  constexpr int NW = WGM * WGN, BK = 64, ROW_BYTES = BK * 2, NT = 64 * NW, TLD = S::TLD, RB = S::RB;
  constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NI = WN / 32, G = MI * NI;
  constexpr int LA = BM / 8 / NW, LW = BN / 8 / NW;     // load instructions per wave and K tile
  const bool second = NP == 2 && blockIdx.x >= L.grid0;
  const GemmProblem<bf16_t> &prob = L.p[second ? 1 : 0];
  const int64_t lda = prob.lda, ldw = prob.ldw;
  const int M = prob.M, N = L.N;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  int tm, tn;
  if (!tile_of_id((int)(blockIdx.x - (second ? L.grid0 : 0)), (M + BM - 1) / BM, (N + BN - 1) / BN, prob.xcd_gx, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  auto key = [](int r) { return (r >> 1) & 7; };

  // per-lane byte offsets of this wave's load instructions (rows past the matrix repeat its last row)
  const TileSource srcA(prob.A + (size_t)m0 * lda), srcW(prob.W + (size_t)n0 * ldw);
  unsigned pa[LA], pw[LW];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (i * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ key(r);
    pa[i] = (unsigned)(((size_t)min(r, M - 1 - m0) * lda + c * 8) * 2);
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int r = (i * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ key(r);
    pw[i] = (unsigned)(((size_t)min(r, N - 1 - n0) * ldw + c * 8) * 2);
  }
  const int nk = L.K / BK;
  unsigned char *const ringA = smem, *const ringW = smem + DA * S::A_BYTES;
  auto load_a = [&](int i, int slot, int kt) __attribute__((always_inline)) {
    srcA.load16(pa[i], (unsigned)kt * (BK * 2), ringA + slot * S::A_BYTES + (i * NW + wave) * 1024);
  };
  auto load_w = [&](int i, int slot, int kt) __attribute__((always_inline)) {
    srcW.load16(pw[i], (unsigned)kt * (BK * 2), ringW + slot * S::W_BYTES + (i * NW + wave) * 1024);
  };

  const int l32 = lane & 31, hi = lane >> 5;
  unsigned la[4], lw[4];   // the lane's 16 bytes of K slice ks in its row of either operand (rows of a lane differ by multiples of 32)
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    la[ks] = (unsigned)((wm * WM + l32) * ROW_BYTES + (((ks * 2 + hi) ^ key(l32)) << 4));
    lw[ks] = (unsigned)((wn * WN + l32) * ROW_BYTES + (((ks * 2 + hi) ^ key(l32)) << 4));
  }
  bf16x8 fa[2][MI], fw[2][NI];
  auto read = [&](auto o_c, int buf, int ks, int slotA, int slotW) __attribute__((always_inline)) {
    constexpr int o = decltype(o_c)::value;
    if constexpr (o < MI) fa[buf][o] = *reinterpret_cast<const bf16x8 *>(ringA + slotA * S::A_BYTES + la[ks] + o * 32 * ROW_BYTES);
    else fw[buf][o - MI] = *reinterpret_cast<const bf16x8 *>(ringW + slotW * S::W_BYTES + lw[ks] + (o - MI) * 32 * ROW_BYTES);
  };

  ColumnBias<NI, 32, bf16_t> column_bias;
  column_bias.fetch(prob.epi, n0 + wn * WN + l32, N);

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // the rings, in the order of the loop: A of K tile s + DA, W of K tile s + DW for s = -DW .. -1 (the last W in K tile 0)
#pragma unroll
  for (int s = -DW; s < 0; ++s) {
    if (s + DA >= 0 && s + DA < nk) {
#pragma unroll
      for (int i = 0; i < LA; ++i) load_a(i, s + DA, s + DA);
    }
    if (s + 1 < 0 && s + DW < nk) {
#pragma unroll
      for (int i = 0; i < LW; ++i) load_w(i, s + DW, s + DW);
    }
  }
  if (nk >= DW) wait_vmcnt<(DA - 1) * (LA + LW) + (DW > DA ? LW : 0) - LW>();
  else wait_vmcnt<0>();
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  unrolled<MI + NI>([&](auto o) __attribute__((always_inline)) { read(o, 0, 0, 0, 0); });

  int slotA = 0, slotW = 0;
  auto next = [](int slot, int depth) { return slot + 1 == depth ? 0 : slot + 1; };
  // K tile t.  FULL: W of t - 1 + DW and A of t + DA exist
  auto step = [&](auto full_c, int t) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full_c)::value;
    const int nextA = next(slotA, DA), nextW = next(slotW, DW), prevW = slotW == 0 ? DW - 1 : slotW - 1;
    unrolled<4>([&](auto s_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(s_c)::value;
      if constexpr (ks == 3) {
        if constexpr (FULL) wait_vmcnt<(DA - 2) * (LA + LW) + (DW > DA ? LW : 0)>();
        else wait_vmcnt<0>();
        wait_lgkmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (!FULL) {
        if constexpr (ks == 0) {
          if (t - 1 + DW < nk)
#pragma unroll
            for (int i = 0; i < LW; ++i) load_w(i, prevW, t - 1 + DW);
        }
        if constexpr (ks == 3) {
          if (t + DA < nk)
#pragma unroll
            for (int i = 0; i < LA; ++i) load_a(i, slotA, t + DA);
        }
      }
      // the next slice's fragments behind the MFMAs of the slice's first half, its loads behind all of them
      constexpr int LOADS = !FULL ? 0 : ks == 0 ? LW : ks == 3 ? LA : 0, READS = MI + NI;
      unrolled<G>([&](auto m_c) __attribute__((always_inline)) {
        constexpr int m = decltype(m_c)::value, i = m / NI, j = i & 1 ? NI - 1 - m % NI : m % NI;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks & 1][i], fw[ks & 1][j], acc[i][j], 0, 0, 0);
        unrolled<READS>([&](auto o_c) __attribute__((always_inline)) {
          constexpr int o = decltype(o_c)::value;
          if constexpr (o * G / (2 * READS) == m) read(o_c, (ks + 1) & 1, (ks + 1) & 3, ks == 3 ? nextA : slotA, ks == 3 ? nextW : slotW);
        });
        unrolled<LOADS>([&](auto o_c) __attribute__((always_inline)) {
          constexpr int o = decltype(o_c)::value;
          if constexpr ((2 * o + 1) * G / (2 * LOADS) == m) {
            if constexpr (ks == 0) load_w(o, prevW, t - 1 + DW);
            else load_a(o, slotA, t + DA);
          }
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    slotA = nextA;
    slotW = nextW;
  };
  int t = 0;
#pragma unroll 1
  for (; t + DW < nk; ++t) step(std::true_type{}, t);
#pragma unroll 1
  for (; t < nk; ++t) step(std::false_type{}, t);

  float bias[NI];
  column_bias.widen(bias);
  // accumulators -> row-major fp32 rows in LDS (lane -> column l32, register r -> row 8 * (r / 4) + 4 * hi + r % 4)
  float *tile = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int pass = 0; pass < BM / RB; ++pass) {
    __syncthreads();
    if (RB == BM || wm * WM / RB == pass) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            tile[(wm * WM - pass * RB + i * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)) * TLD + wn * WN + j * 32 + l32] = acc[i][j][r] + bias[j];
    }
    __syncthreads();
    tile_epilogue<EM, RB, BN, TLD, NT>(tile, m0 + pass * RB, n0, M, N, prob.epi, prob.vec_ok != 0);
  }
}

}  // namespace

}  // namespace pf
