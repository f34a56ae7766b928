// bf16 MFMA GEMM body of the 256x256 tile: C = epilogue(A W^T + bias), K a multiple of 64.
//
// Eight wavefronts, 2 along M x 4 along N, one workgroup per CU.  A K tile is 64 wide and lives in LDS as four half tiles
// (A0 A1 W0 W1: 128 rows x 128 bytes each), two K tiles deep (128 KB).  A wave owns 64 rows of either A half (two blocks of 32)
// and 32 rows of either W half, so a K tile is four phases of eight MFMAs, one block of A rows with both W halves each:
//
//   phase   multiplies    reads from LDS (for the next phase, for the next K tile)    loads
//     0     block 0       block 1 (A0),  W0(t+1)                                      A1(t+1)
//     1     block 1       block 2 (A1)                                                W1(t+2)
//     2     block 2       block 3 (A1),  W1(t+1)                                      A0(t+2)
//     3     block 3       block 0 of t+1 (A0)                                         W0(t+3)
//
// A half tile is loaded again as soon as its last rows have been read, one and a half to two K tiles before they are needed, and
// every fragment is read a phase before its MFMAs: nothing in a phase waits for what was asked for in it.  Reads and loads are
// issued between the MFMAs.  Two barriers a K tile, behind phases 1 and 3: what the next two phases read has landed
// (three half tiles, six of the wave's load instructions, may still be in flight), and what they overwrite has been read (the four
// reads behind the barrier's phase may still be on their way; they are of the half that is loaded a barrier later).
// LDS rows are swizzled as in gemm_mfma_dl.hip.
//
// What bounds it is power: 81 % of the cycles have the matrix unit busy (8192x8192x8192), at the clock the card then holds, 1.6 GHz.
// One K tile at a time behind one barrier (43 - 49 % busy) -> this: 8192x8192x8192 866 -> 758 us (1.45 PFLOP/s, the vendor
// library 683), 16896x9216x3072 847 -> 737 (724), 16896x12288x3072 with GELU 1157 -> 1031, 16896x3072x15360 with a
// residual 1574 -> 1369.  Waves 4-7 half a phase behind waves 0-3, one multiplying while the other reads (eight barriers a K tile):
// 1 % slower; reads in the phase that uses them: 4 % slower.
#pragma once
#include "gemm_tile.h"

namespace pf {

namespace {

struct HalfTiles256 {
  static constexpr int BM = 256, BN = 256, NT = 512;
  static constexpr int HALF_BYTES = 128 * 128;            // 16 KB
  static constexpr int W_BASE = 4 * HALF_BYTES;           // A: [stage][half] at 0, W: the same behind it
  static constexpr int TLD = BN + 4, RB = BM / 2;         // the epilogue's row passes: fp32 rows of the tile in LDS
  static constexpr int SMEM = RB * TLD * 4 > 8 * HALF_BYTES ? RB * TLD * 4 : 8 * HALF_BYTES;
};

__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

template <int NP, int EM>
__device__ __forceinline__ void gemm_half_tiles_body(const GemmLaunch<bf16_t, NP> &L, unsigned char *smem) {
  constexpr int BK = 64, ROW_BYTES = BK * 2;
  constexpr int BM = HalfTiles256::BM, BN = HalfTiles256::BN, NT = HalfTiles256::NT, TLD = HalfTiles256::TLD, RB = HalfTiles256::RB;
  constexpr int HALF_BYTES = HalfTiles256::HALF_BYTES, W_BASE = HalfTiles256::W_BASE;
  const bool second = NP == 2 && blockIdx.x >= L.grid0;
  const GemmProblem<bf16_t> &prob = L.p[second ? 1 : 0];
  const int64_t lda = prob.lda, ldw = prob.ldw;
  const int M = prob.M, N = L.N;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  int tm, tn;
  if (!tile_of_id((int)(blockIdx.x - (second ? L.grid0 : 0)), (M + BM - 1) / BM, (N + BN - 1) / BN, prob.xcd_gx, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  auto key = [](int r) { return (r >> 1) & 7; };

  // per-lane byte offsets of this wave's two load instructions of each half tile (rows past the matrix repeat its last row)
  const TileSource srcA(prob.A + (size_t)m0 * lda), srcW(prob.W + (size_t)n0 * ldw);
  unsigned pa[2][2], pw[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (i * 8 + wave) * 8 + (lane >> 3), c = (lane & 7) ^ key(r), row = h * 128 + r;
      pa[h][i] = (unsigned)(((size_t)min(row, M - 1 - m0) * lda + c * 8) * 2);
      pw[h][i] = (unsigned)(((size_t)min(row, N - 1 - n0) * ldw + c * 8) * 2);
    }
  const int nk = L.K / BK;
  // load instruction i of half tile number Q (0 B0, 1 A0, 2 B1, 3 A1) of K tile kt
  auto load1 = [&](auto q_c, int i, int stage, int kt) __attribute__((always_inline)) {
    constexpr int Q = decltype(q_c)::value, h = Q >> 1;
    const unsigned koff = (unsigned)kt * (BK * 2);
    unsigned char *dst = smem + (Q & 1 ? 0 : W_BASE) + (stage * 2 + h) * HALF_BYTES + wave * 1024;
    if constexpr (Q & 1) srcA.load16(pa[h][i], koff, dst + i * 8192);
    else srcW.load16(pw[h][i], koff, dst + i * 8192);
  };
  auto load = [&](auto q_c, int stage, int kt) __attribute__((always_inline)) {
    load1(q_c, 0, stage, kt);
    load1(q_c, 1, stage, kt);
  };

  const int l32 = lane & 31, hi = lane >> 5;
  const unsigned char *fa = smem + (wm * 64 + l32) * ROW_BYTES, *fw = smem + W_BASE + (wn * 32 + l32) * ROW_BYTES;
  unsigned slot[4];   // byte offset of the lane's 16 bytes of K slice ks in a row (the rows of a lane differ by multiples of 32)
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) slot[ks] = (unsigned)(((ks * 2 + hi) ^ key(l32)) << 4);
  bf16x8 fragA[2][4], fragB[2][2][4];   // [phase & 1][K slice], [K tile & 1][W half][K slice]
  auto read_a1 = [&](int buf, int blk, int stage, int ks) __attribute__((always_inline)) {
    fragA[buf][ks] = *reinterpret_cast<const bf16x8 *>(fa + (stage * 2 + (blk >> 1)) * HALF_BYTES + (blk & 1) * 32 * ROW_BYTES + slot[ks]);
  };
  auto read_b1 = [&](int stage, int h, int ks) __attribute__((always_inline)) {
    fragB[stage][h][ks] = *reinterpret_cast<const bf16x8 *>(fw + (stage * 2 + h) * HALF_BYTES + slot[ks]);
  };

  ColumnBias<2, 128, bf16_t> column_bias;
  column_bias.fetch(prob.epi, n0 + wn * 32 + l32, N);

  f32x16 acc[4][2];   // [32-row block][W half]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][g][r] = 0.f;

  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  constexpr std::integral_constant<int, 2> c2{};
  constexpr std::integral_constant<int, 3> c3{};
  const int last = nk - 1;
  load(c0, 0, 0);
  load(c2, 0, 0);
  load(c1, 0, 0);
  load(c0, 1, min(1, last));
  load(c3, 0, 0);
  load(c2, 1, min(1, last));
  load(c1, 1, min(1, last));
  wait_vmcnt<8>();
  phase_barrier();
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) read_b1(0, 0, ks), read_b1(0, 1, ks), read_a1(0, 0, 0, ks);
  wait_lgkmcnt<0>();
  phase_barrier();
  load(c0, 0, min(2, last));
  wait_vmcnt<6>();
  phase_barrier();

  // K tile t in stage S (t & 1); LEFT: K tiles behind it (2 stands for two or more)
  auto step = [&](auto s_c, auto left_c, int t) __attribute__((always_inline)) {
    constexpr int S = decltype(s_c)::value, LEFT = decltype(left_c)::value;
    unrolled<4>([&](auto p_c) __attribute__((always_inline)) {
      constexpr int P = decltype(p_c)::value;
      unrolled<8>([&](auto m_c) __attribute__((always_inline)) {
        constexpr int m = decltype(m_c)::value, ks = m >> 1, g = m & 1;
        acc[P][g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fragA[P & 1][ks], fragB[S][g][ks], acc[P][g], 0, 0, 0);
        if constexpr ((m & 1) == 0) {
          if constexpr (LEFT > 0 || P < 3) {
            if constexpr (P < 3) read_a1((P + 1) & 1, P + 1, S, ks);
            else read_a1(0, 0, S ^ 1, ks);
          }
        } else if constexpr ((P & 1) == 0 && LEFT > 0) {
          read_b1(S ^ 1, P >> 1, ks);
        }
        if constexpr (m == 2 || m == 5) {
          constexpr int i = m == 5;
          if constexpr (P == 0 && LEFT > 0) load1(c3, i, S ^ 1, min(t + 1, last));
          if constexpr (P == 1 && LEFT > 1) load1(c2, i, S, min(t + 2, last));
          if constexpr (P == 2 && LEFT > 1) load1(c1, i, S, min(t + 2, last));
          if constexpr (P == 3 && LEFT > 1) load1(c0, i, S ^ 1, min(t + 3, last));
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr ((P & 1) && LEFT > 0) {
        wait_vmcnt<(LEFT > 1 ? 6 : P == 1 ? 4 : 0)>();
        wait_lgkmcnt<4>();
        phase_barrier();
      }
    });
  };
  int t = 0;
#pragma unroll 1
  for (; t + 2 < nk; t += 2) {
    step(c0, c2, t);
    step(c1, c2, t + 1);
  }
  step(c0, c1, t);
  if (!(nk & 1)) step(c1, c0, t + 1);

  float bias[2];
  column_bias.widen(bias);
  // accumulators -> row-major fp32 rows in LDS (lane -> column l32, register r -> row 8 * (r / 4) + 4 * hi + r % 4), one A half
  // at a time: every wave holds 64 rows of either
  float *tile = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          tile[(wm * 64 + i * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)) * TLD + g * 128 + wn * 32 + l32] = acc[h * 2 + i][g][r] + bias[g];
    __syncthreads();
    tile_epilogue<EM, RB, BN, TLD, NT>(tile, m0 + h * RB, n0, M, N, prob.epi, prob.vec_ok != 0);
  }
}

}  // namespace

}  // namespace pf
