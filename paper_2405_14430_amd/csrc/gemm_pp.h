// bf16 MFMA GEMM of 256x256 tiles for launches with many of them (gfx950): C = epilogue(A W^T + bias), K a multiple of 64.
//
// Eight wavefronts, 2 along M x 4 along N, one workgroup per CU; waves 0-3 sit one to a SIMD, and so do 4-7.  A K tile is
// 64 wide and lives in LDS as four half tiles (A0 A1 B0 B1: 128 rows x 128 bytes each), two K tiles deep (128 KB).  A wave owns
// 64 rows of either A half and 32 rows of either W half, so a K tile is four phases of eight MFMAs:
//
//   phase   reads from LDS        loads                  multiplies
//     0     A0(t)   8 reads       B0(t+2)                A0 B0
//     1     B1(t)   4             A0(t+2)                A0 B1
//     2     A1(t)   8             B1(t+2)                A1 B1
//     3     B0(t+1) 4             A1(t+2)                A1 B0
//
// Every phase is a memory part (reads, two load instructions per wave, waits), a barrier, the MFMAs, a barrier; waves 4-7 run
// one barrier behind waves 0-3, so on every SIMD one wave feeds the matrix unit while the other fetches its operands.
// The half tiles are numbered in the order B0 A0 B1 A1 of each K tile: number j is read in phase j - 1, so its place is free
// for number j + 8 from phase j on, where that is loaded.  A load has seven phases to arrive (six half tiles, 96 KB per CU, are in
// flight at any time), and the waits never drain the queue: in phase k a wave waits for its part of number k + 2, twelve of
// its load instructions behind it.  Both waves of a SIMD pass that wait before the first of them reads number k + 2.
// LDS rows are swizzled as in gemm_mfma_dl.hip.
#pragma once
#include "gemm_tile.h"

namespace pf {

namespace {

struct PingPong256 {
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

template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}

template <int NP, int EM>
__device__ __forceinline__ void gemm_pp256_body(const GemmLaunch<bf16_t, NP> &L, unsigned char *smem) {
  constexpr int BK = 64, ROW_BYTES = BK * 2;
  constexpr int BM = PingPong256::BM, BN = PingPong256::BN, NT = PingPong256::NT, TLD = PingPong256::TLD, RB = PingPong256::RB;
  constexpr int HALF_BYTES = PingPong256::HALF_BYTES, W_BASE = PingPong256::W_BASE;
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
          tile[(wm * 64 + i * 32 + 8 * (r >> 2) + 4 * hi + (r & 3)) * TLD + g * 128 + wn * 32 + l32] = acc[h * 2 + i][g][r];
    __syncthreads();
    tile_epilogue<EM, RB, BN, TLD, NT>(tile, m0 + h * RB, n0, M, N, prob.epi, prob.vec_ok != 0);
  }
}

}  // namespace

}  // namespace pf
