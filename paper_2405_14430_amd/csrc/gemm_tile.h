// What the direct-to-LDS MFMA GEMM kernels share (bf16: gemm_mfma_dl.hip, fp32: gemm_mfma_f32.hip): tile loads, the
// workgroup -> tile map, and the vectorised epilogue over a finished fp32 tile in LDS.
#pragma once
#include <type_traits>

#include "common.h"
#include "epilogue.h"
#include "ops.h"

namespace pf {

namespace {

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}

// In front of a K loop: the compiler asks for the epilogue's arguments up there, and while scalar loads may be in flight it waits for
// all LDS reads in front of a K tile's first MFMA instead of for those that it needs.  (The builtin, not inline assembly: the compiler
// counts it.)  For the residual GEMMs of two problems, whose operands' addresses take the most arguments: 304x3072x15360 with 64x64 tiles
// 84 us, 91 without.  The other kernels gain and lose about 2 % by it (512x4608x1152 GELU, 64x64, 12.1 -> 12.4) and go without.
__device__ __forceinline__ void wait_scalar_loads() {
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0), the other counters as they are
}

// s_waitcnt vmcnt(behind * LPS) for a wave-uniform run-time `behind` in [0, MAXB] (the count is an immediate)
template <int LPS, int MAXB>
__device__ __forceinline__ void wait_tiles_behind(int behind) {
  static_assert(MAXB * LPS <= 63, "vmcnt is a 6-bit counter");
  if constexpr (MAXB <= 0) {
    wait_vmcnt<0>();
  } else {
    if (behind >= MAXB) wait_vmcnt<MAXB * LPS>();
    else wait_tiles_behind<LPS, MAXB - 1>(behind);
  }
}

// Tile loads are raw-buffer loads into LDS: a wave-uniform resource over the rows of the operand that the tile starts
// at, a wave-uniform byte offset (the K position) and one 32-bit per-lane byte offset.  Against global loads with a
// 64-bit address per lane that saves the 64-bit address arithmetic and half the address registers of every load
// (same-box A/B inside the stages: Flux-scale QKV 141 -> 136 us, MLP-up 173 -> 165 us, long-sequence PixArt QKV 60 ->
// 53 us).  The resource spans 2 GB from its base and the offsets are built from row indices that are clamped to the
// matrix, so no load leaves the operand (gemm_mfma_dl_supported keeps the leading dimensions small enough).
// The type only exists in device code; the host pass sees a stand-in with the same interface.
#if defined(__HIP_DEVICE_COMPILE__)
struct TileSource {
  __amdgpu_buffer_rsrc_t rs;
  __device__ __forceinline__ explicit TileSource(const void *base)
      : rs(__builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0x7ffffff0, 0x00020000)) {}
  // 16 bytes per lane from base + lane_bytes + uniform_bytes to lds_wave_uniform + 16 * lane
  __device__ __forceinline__ void load16(unsigned lane_bytes, unsigned uniform_bytes, unsigned char *lds_wave_uniform) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)lds_wave_uniform, 16, lane_bytes,
                                             uniform_bytes, 0, 0);
  }
};
#else
struct TileSource {
  __device__ explicit TileSource(const void *) {}
  __device__ void load16(unsigned, unsigned, unsigned char *) const {}
};
#endif

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<N, I + 1>(f);
  }
}

// What a launch computes: one GEMM, or two that share N and K (the text and the image stream of a two-stream block: own
// operands and own rows).  Workgroups [0, grid0) belong to the first, the rest to the second; grid0 is a multiple of 8, so
// the second one's ids fall on the XCDs like the first one's.  154 text rows alone are 72 - 288 workgroups of 64x64 tiles:
// as launches of their own they took 8 - 19 us each, four a layer, of an SD3-scale call (637 -> 530 us with shared launches).
// The kernels are compiled for either count: one problem read through the two-problem form costs a 10 us launch 0.3 us
// (twice the kernel arguments, addressed at run time).
template <typename T>
struct GemmProblem {
  const T *A; int64_t lda;
  const T *W; int64_t ldw;
  int M;
  int vec_ok, xcd_gx;
  Epilogue<T> epi;
};
template <typename T, int NP>
struct GemmLaunch {
  GemmProblem<T> p[NP];
  int N, K;
  unsigned grid0, grid;   // workgroups of the first problem, of all
};

// Workgroup id -> output tile.  Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2, so XCD x runs
// the ids x, x + 8, ...  Every XCD gets one rectangular block of the tile grid - the grid is cut gx times along M and
// 8 / gx times along N - because what an XCD fetches from memory is the A rows of its block plus the W rows of its
// block: a contiguous run of tiles (a block one tile-column wide and all of M high) makes every XCD fetch all of A
// (Flux-scale MLP-down: 623 MB fetched per launch for 157 MB of operands).  Inside the block
// the tiles are walked in bands of G tile rows (G = cut >> 8), column by column: the workgroups that an XCD runs at a time
// should cover a near-square patch of the output, because per K step they fetch the A rows and the W rows of that patch, and
// what all XCDs together fetch has to stay below the 7 TB/s at which the memory side fills the L2s (row by row, 32 tiles of
// 256x256 ask for 33 operand panels per K step, in bands of four for 12).  Returns false for the surplus ids of the padded
// grid.
__host__ __device__ __forceinline__ bool tile_of_id(int id, int tiles_m, int tiles_n, int cut, int &tm, int &tn) {
  const int gx = cut & 255, G = cut >> 8, gy = 8 / gx;
  const int bm = (tiles_m + gx - 1) / gx, bn = (tiles_n + gy - 1) / gy;
  const int x = id & 7, j = id >> 3;
  if (j >= bm * bn) return false;
  const int band = j / (G * bn), jj = j - band * (G * bn);
  const int rows = G < bm - band * G ? G : bm - band * G;   // (the last band may be lower)
  const int ln = jj / rows, lm = band * G + (jj - ln * rows);
  tm = (x % gx) * bm + lm;
  tn = (x / gx) * bn + ln;
  return tm < tiles_m && tn < tiles_n;
}

// Residual and gate operands of a mode-1 epilogue, fetched by the thread that will use them before the K loop starts, so
// that their memory latency runs under the loop instead of after it (the residual rows were written by an earlier
// kernel and are in no cache).  Only for tiles small enough that a thread owns at most IT 8-column groups.  A tile is
// read and written by its own workgroup only, so reading R early is safe when the GEMM updates it in place.
template <int BM, int BN, int NT>
struct EpiOperands {
  static constexpr int GROUPS = BM * BN / 8, IT = (GROUPS + NT - 1) / NT;
  float4 r[IT][2], g[IT][2];
  bool on;
  template <typename T>
  __device__ __forceinline__ void fetch(int m0, int n0, int M, int N, const Epilogue<T> &epi, bool vec_ok) {
    on = vec_ok;
    if (!on) return;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int grp = threadIdx.x + it * NT;
      const int row = m0 + grp / (BN / 8), col = n0 + (grp % (BN / 8)) * 8;
      if ((GROUPS % NT != 0 && grp >= GROUPS) || row >= M || col + 8 > N) continue;
      const float *rp = epi.R + (size_t)row * epi.ldr + col;
      r[it][0] = *reinterpret_cast<const float4 *>(rp); r[it][1] = *reinterpret_cast<const float4 *>(rp + 4);
      if (epi.gate) {
        const float *gp = epi.gate_of(row) + col;
        g[it][0] = *reinterpret_cast<const float4 *>(gp); g[it][1] = *reinterpret_cast<const float4 *>(gp + 4);
      }
    }
  }
};

// eight consecutive elements (16-byte aligned) to and from fp32
__device__ __forceinline__ void load8(const bf16_t *p, float *o) { Vec16<bf16_t>::load(p, o); }
__device__ __forceinline__ void load8(const float *p, float *o) { Vec16<float>::load(p, o); Vec16<float>::load(p + 4, o + 4); }
__device__ __forceinline__ void store8(bf16_t *p, const float *o) { Vec16<bf16_t>::store(p, o); }
__device__ __forceinline__ void store8(float *p, const float *o) { Vec16<float>::store(p, o); Vec16<float>::store(p + 4, o + 4); }

// Bias of columns col, col + STEP, ..., for the kernels' accumulator layouts: fetched once, in front of the K loop or behind it, because
// an epilogue that asked for it group by group waited for a load from L2 in every one, and kept as stored until it is used: a conversion
// that the compiler moved up to the load would wait for it in front of the loop (0.3 us of a 10 us launch).  Columns past
// the matrix repeat its last one.
template <int N, int STEP, typename T>
struct ColumnBias {
  unsigned raw[N];
  bool pairs = false;   // raw[0] and raw[2] hold two columns each
  // vec: four consecutive columns from a multiple of four, of an operand that is aligned for vectors
  __device__ __forceinline__ void fetch(const Epilogue<T> &epi, int col, int cols, bool vec = false) {
#pragma unroll
    for (int j = 0; j < N; ++j) raw[j] = 0;
    if (!epi.bias) return;
    if constexpr (N == 4 && STEP == 1) {
      if (vec && cols % 4 == 0) {
        const T *p = epi.bias + min(col, cols - 4);
        if constexpr (sizeof(T) == 2) {
          const uint2 u = *reinterpret_cast<const uint2 *>(p);
          raw[0] = u.x, raw[2] = u.y, pairs = true;
        } else {
          const uint4 u = *reinterpret_cast<const uint4 *>(p);
          raw[0] = u.x, raw[1] = u.y, raw[2] = u.z, raw[3] = u.w;
        }
        return;
      }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const T *p = epi.bias + min(col + j * STEP, cols - 1);
      if constexpr (sizeof(T) == 2) raw[j] = *reinterpret_cast<const unsigned short *>(p);
      else raw[j] = *reinterpret_cast<const unsigned *>(p);
    }
  }
  // what the epilogue adds; once, behind the loop
  __device__ __forceinline__ void widen(float (&b)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      asm volatile("" : "+v"(raw[j]));
      if (N == 4 && STEP == 1 && sizeof(T) == 2 && pairs) b[j] = __builtin_bit_cast(float, j & 1 ? raw[j & ~1] & 0xffff0000u : raw[j] << 16);
      else b[j] = __builtin_bit_cast(float, sizeof(T) == 2 ? raw[j] << 16 : raw[j]);
    }
  }
};

// Epilogue over a finished fp32 tile held row-major in LDS (row stride TLD floats), its bias added.  PRE: residual / gate
// operands come from `ops` (fetched earlier) when ops->on.
template <int EM, int BM, int BN, int TLD, int NT = 256, bool PRE = false, typename T>
__device__ __forceinline__ void tile_epilogue(const float *tile, int m0, int n0, int M, int N, const Epilogue<T> &epi, bool vec_ok, const EpiOperands<BM, BN, NT> *ops = nullptr) {
  constexpr int GROUPS = BM * BN / 8;
  constexpr int IT = (GROUPS + NT - 1) / NT;
  if constexpr (EM != EM_KV_ROUTE) {
    // Operands that are not aligned for vectors, and the columns behind the last whole group of eight: one element per thread,
    // consecutive threads along a row (eight elements of a row per thread, as in the vector passes: 512x1152x1152, unaligned
    // bias, residual 14.5 us against 12.4; 1156 columns in rows of 1160, 4000x1156x512, 14.5 against 12.6).
    const int c_from = vec_ok ? (N & ~7) - n0 : 0, width = vec_ok ? 8 : BN;
    if (c_from < BN && n0 + c_from < N) {
      const int dr = NT / width, dc = NT % width;
      int r = threadIdx.x / width, c = c_from + threadIdx.x % width;
#pragma unroll 1
      while (r < BM) {
        if (m0 + r < M && c < BN && n0 + c < N) epi.put(m0 + r, n0 + c, tile[r * TLD + c]);
        r += dr;
        c += dc;
        if (c >= c_from + width) c -= width, ++r;
      }
    }
    if (!vec_ok) return;
  }
  // Groups of eight columns, UB of a thread at a time: what they need from memory is asked for together, since the compiler may
  // not move a load over the store of the group before it.
  constexpr int UB = PRE ? IT : IT < 4 ? IT : 4;
  constexpr bool LOADS = EM == EM_RESIDUAL || EM == EM_KV_ROUTE;
#pragma unroll 1
  for (int it0 = 0; it0 < IT; it0 += UB) {
    float4 q0[LOADS ? UB : 1], q1[LOADS ? UB : 1], g0[LOADS ? UB : 1], g1[LOADS ? UB : 1];   // residual and gate, or RoPE table (q0, q1) and norm scales (g0)
    auto place = [&](int u, int &r, int &c0) {   // group `it0 + u` of the thread; false: nothing to do
      const int g = threadIdx.x + (it0 + u) * NT;
      r = g / (BN / 8), c0 = (g % (BN / 8)) * 8;
      return (GROUPS % (NT * UB) == 0 || g < GROUPS) && m0 + r < M && n0 + c0 + 8 <= N;   // (columns behind the last whole group: above)
    };
    if constexpr (LOADS) {
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        int r, c0;
        if (!place(u, r, c0)) continue;
        const int row = m0 + r, col = n0 + c0;
        if constexpr (EM == EM_RESIDUAL) {
          if constexpr (PRE) {
            if (ops->on) { q0[u] = ops->r[u][0]; q1[u] = ops->r[u][1]; g0[u] = ops->g[u][0]; g1[u] = ops->g[u][1]; continue; }
          }
          const float *rp = epi.R + (size_t)row * epi.ldr + col;
          q0[u] = *reinterpret_cast<const float4 *>(rp); q1[u] = *reinterpret_cast<const float4 *>(rp + 4);
          if (epi.gate) {
            const float *gp = epi.gate_of(row) + col;
            g0[u] = *reinterpret_cast<const float4 *>(gp); g1[u] = *reinterpret_cast<const float4 *>(gp + 4);
          }
        } else {
          const KvRoute &kv = epi.kv;
          if (kv.rope && col < 2 * kv.d) {
            const int lrow = row - (kv.seg > 0 ? row / kv.seg * kv.seg : 0);
            const float2 *tab = kv.rope + (size_t)lrow * (kv.dh >> 1) + (col % kv.dh >> 1);   // (d is a whole number of heads)
            const float2 t0 = tab[0], t1 = tab[1], t2 = tab[2], t3 = tab[3];
            q0[u] = make_float4(t0.x, t0.y, t1.x, t1.y); q1[u] = make_float4(t2.x, t2.y, t3.x, t3.y);
          }
          if constexpr (sizeof(T) == 2) {   // scales of the per-head norm, as stored
            if (kv.q_norm && col < 2 * kv.d)
              g0[u] = *reinterpret_cast<const float4 *>(reinterpret_cast<const T *>(col < kv.d ? kv.q_norm : kv.k_norm) + col % kv.dh);
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      int r, c0;
      if (!place(u, r, c0)) continue;
      const int row = m0 + r, col = n0 + c0;
      const float *src = tile + r * TLD + c0;
      float4 lo = *reinterpret_cast<const float4 *>(src), hi4 = *reinterpret_cast<const float4 *>(src + 4);
      float v[8] = {lo.x, lo.y, lo.z, lo.w, hi4.x, hi4.y, hi4.z, hi4.w};
      if constexpr (EM == EM_KV_ROUTE) {
        // QKV projection routed into the K / V^T buffers (an 8-column group never straddles q|k|v or two heads)
        const KvRoute &kv = epi.kv;
        const int part = col / kv.d, cc = col - part * kv.d;
        const int hh = cc / kv.dh, ch = cc - hh * kv.dh;
        const int img = kv.seg > 0 ? row / kv.seg : 0;
        const int lrow = row - img * kv.seg;           // row inside its image
        if constexpr (sizeof(T) == 2) {   // (gemm_kv_route_supported: the norm is of bf16 stages)
          if (kv.q_norm && part < 2) {
            // a head's dh / 8 groups of the row are consecutive, aligned lanes (the tile is a whole number of heads wide)
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) ss = fmaf(v[e], v[e], ss);
            for (int m = 1; m < kv.dh >> 3; m <<= 1) ss += __shfl_xor(ss, m, kWave);
            const float rinv = rsqrtf(ss / (float)kv.dh + kv.norm_eps);
            const bf16x8 w = __builtin_bit_cast(bf16x8, g0[u]);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = v[e] * rinv * (float)w[e];
          }
        }
        if (kv.rope && part < 2) {
          const float2 cs[4] = {{q0[u].x, q0[u].y}, {q0[u].z, q0[u].w}, {q1[u].x, q1[u].y}, {q1[u].z, q1[u].w}};
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            float a0 = v[e], b0 = v[e + 1];
            v[e] = a0 * cs[e >> 1].x - b0 * cs[e >> 1].y;
            v[e + 1] = a0 * cs[e >> 1].y + b0 * cs[e >> 1].x;
          }
        }
        if (part == 0 && kv.q_scale != 0.f) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] *= kv.q_scale;
        }
        if (part == 0) {
          store8(reinterpret_cast<T *>(epi.C) + (size_t)row * epi.ldc + col, v);
        } else if (part == 1) {
          const int brow = lrow < kv.split ? kv.row0a + lrow : kv.row0b + (lrow - kv.split);
          store8(reinterpret_cast<T *>(kv.kbuf) + (size_t)img * kv.img_stride + ((size_t)hh * kv.Lp + brow) * kv.dh + ch, v);
        }
        // part 2 (v) is written by the transposed pass below
      } else if constexpr (EM == EM_STORE || EM == EM_STORE_ERF) {
        if (col + 8 > epi.gelu_from) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (col + e >= epi.gelu_from) v[e] = gelu_f(v[e], EM != EM_STORE_ERF);
        }
        store8(reinterpret_cast<T *>(epi.C) + (size_t)row * epi.ldc + col, v);
      } else {
        float x[8] = {q0[u].x, q0[u].y, q0[u].z, q0[u].w, q1[u].x, q1[u].y, q1[u].z, q1[u].w};
        if (epi.gate) {
          float gg[8] = {g0[u].x, g0[u].y, g0[u].z, g0[u].w, g1[u].x, g1[u].y, g1[u].z, g1[u].w};
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] += gg[e] * v[e];
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] += v[e];
        }
        float *xp = reinterpret_cast<float *>(epi.C) + (size_t)row * epi.ldc + col;
        *reinterpret_cast<float4 *>(xp) = make_float4(x[0], x[1], x[2], x[3]);
        *reinterpret_cast<float4 *>(xp + 4) = make_float4(x[4], x[5], x[6], x[7]);
        if (epi.C2) store8(epi.C2 + (size_t)row * epi.ldc2 + col, x);
      }
    }
  }
  // v columns of a routed QKV projection: V^T[h][c][buffer row].  The tile is walked column-wise, eight consecutive
  // rows per thread and consecutive threads along the rows, so that the stores run along V^T's contiguous axis.  The groups of
  // eight start where the first row's buffer row reaches a multiple of eight (text of 77 or 154 rows in front of the image puts
  // it anywhere), so that they are 16-byte stores; the eight rows left at the two ends of the tile go one element per thread.
  // Against one element at a time wherever the first row was off: three QKV launches of 512 rows behind 154 of text, SD3-scale,
  // 82.8 -> 72.9 us; two of 2048 rows behind 77, Flux-scale, 346 -> 290 us.
  if constexpr (EM != EM_KV_ROUTE) return;
  if (n0 + BN > 2 * epi.kv.d) {
    const KvRoute &kv = epi.kv;
    constexpr int RG = BM / 8;
    auto buffer_row = [&](int lrow) { return lrow < kv.split ? kv.row0a + lrow : kv.row0b + (lrow - kv.split); };
    auto put = [&](int r, int cl) {   // one element: tile row r, column cl
      const int row = m0 + r, img = kv.seg > 0 ? row / kv.seg : 0;
      reinterpret_cast<T *>(kv.vtbuf)[(size_t)img * kv.img_stride + (size_t)(n0 + cl - 2 * kv.d) * kv.Lp + buffer_row(row - img * kv.seg)] =
          (T)tile[r * TLD + cl];
    };
    const int lrow0 = m0 - (kv.seg > 0 ? m0 / kv.seg * kv.seg : 0);
    const int first = -buffer_row(lrow0) & 7;   // tile row of the first group
    if (first == 0 && m0 + BM <= M && (kv.seg <= 0 || lrow0 + BM <= kv.seg) && (lrow0 >= kv.split || lrow0 + BM <= kv.split)) {
      // the tile's rows lie in one image and one range and start on a multiple of eight: vector stores alone
      T *vt = reinterpret_cast<T *>(kv.vtbuf) + (size_t)(kv.seg > 0 ? m0 / kv.seg : 0) * kv.img_stride + buffer_row(lrow0);
      for (int u = threadIdx.x; u < RG * BN; u += NT) {
        const int r = u % RG * 8, cl = u / RG, col = n0 + cl;
        if (col >= N || col < 2 * kv.d) continue;
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = tile[(r + e) * TLD + cl];
        store8(vt + (size_t)(col - 2 * kv.d) * kv.Lp + r, o);
      }
      return;
    }
    for (int u = threadIdx.x; u < RG * BN; u += NT) {
      const int r = u % RG * 8 + first, cl = u / RG;
      const int col = n0 + cl, row = m0 + r;
      if (col >= N || col < 2 * kv.d || row >= M || r + 8 > BM) continue;
      const int img = kv.seg > 0 ? row / kv.seg : 0;
      const int lrow = row - img * kv.seg, brow = buffer_row(lrow);
      const bool whole = row + 8 <= M && (kv.seg <= 0 || lrow + 8 <= kv.seg) && (lrow >= kv.split || lrow + 8 <= kv.split);
      if (whole && (brow & 7) == 0) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = tile[(r + e) * TLD + cl];
        store8(reinterpret_cast<T *>(kv.vtbuf) + (size_t)img * kv.img_stride + (size_t)(col - 2 * kv.d) * kv.Lp + brow, o);   // (col - 2d = h*dh + c)
      } else {
#pragma unroll 1
        for (int e = 0; e < 8 && row + e < M; ++e) put(r + e, cl);
      }
    }
    if (first != 0)
      for (int u = threadIdx.x; u < 8 * BN; u += NT) {
        const int e = u & 7, cl = u >> 3, col = n0 + cl;
        const int r = e < first ? e : BM - 8 + e;
        if (col < N && col >= 2 * kv.d && m0 + r < M) put(r, cl);
      }
  }
}

// Cut of the tile grid over the 8 XCDs (see tile_of_id): the gx in {1, 2, 4, 8} for which an XCD's block needs the
// fewest operand rows; a cut that pads the grid by more than an eighth is priced four times.  *grid receives the
// workgroup count.
inline int xcd_cut(const GemmArgs &a, int BM, int BN, unsigned *grid) {
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  int best = 1;
  double best_cost = 1e300;
  const int64_t T = (int64_t)tiles_m * tiles_n;
  for (int gx = 1; gx <= 8; gx *= 2) {
    const int gy = 8 / gx;
    const int bm = (tiles_m + gx - 1) / gx, bn = (tiles_n + gy - 1) / gy;
    const int64_t padded = 8LL * bm * bn;
    double cost = (double)bm * BM + (double)bn * BN;          // operand rows per XCD (both operands have K columns)
    if (padded * 8 > T * 9) cost *= 4.0;                       // too many idle workgroup slots
    if (cost < best_cost) { best_cost = cost; best = gx; }
  }
  const int gy = 8 / best;
  const int bm = (tiles_m + best - 1) / best, bn = (tiles_n + gy - 1) / gy;
  *grid = (unsigned)(8 * bm * bn);
  // band height: the patch of G x (resident / G) tiles with the fewest operand rows.  From four rounds of tiles on
  // (16896x12288x3072: 256x256 1206 -> 1162 us, 128x192 1532 -> 1187, 128x128 1545 -> 1273); launches of fewer rounds keep N
  // fastest (4096x3456x1152, 128x128: 41 us against 46 in bands).
  const int resident = 32 * (BM * BN >= 256 * 128 ? 1 : 2);   // workgroups an XCD runs at a time
  int G = 1;
  if (bm * bn >= 4 * resident) {
    int best_rows = 1 << 30;
    for (int g = 1; g <= bm && g <= resident; g *= 2) {
      const int cols = resident / g < bn ? resident / g : bn;
      const int rows = resident / cols < bm ? resident / cols : bm;
      if (rows * BM + cols * BN < best_rows) { best_rows = rows * BM + cols * BN; G = g; }
    }
  }
  return best | G << 8;
}

inline bool vec_epilogue_ok(const GemmArgs &a) {
  auto al = [](const void *p, uintptr_t n) { return ((uintptr_t)p % n) == 0; };
  bool ok = (!a.bias || al(a.bias, 16));
  if (a.epilogue == 0) return ok && al(a.C, 16) && a.ldc % 8 == 0;
  ok = ok && al(a.C, 16) && a.ldc % 4 == 0 && al(a.R, 16) && a.ldr % 4 == 0 && (!a.gate || (al(a.gate, 16) && a.gate_stride % 4 == 0));
  if (a.C2) ok = ok && al(a.C2, 16) && a.ldc2 % 8 == 0;
  return ok;
}

// Fills the launch of `a` and, for NP = 2, `b` (same N and K) with BM x BN tiles; returns the workgroup count.
template <typename T, int NP>
inline unsigned make_launch(const GemmArgs &a, const GemmArgs *b, int BM, int BN, GemmLaunch<T, NP> *L) {
  unsigned total = 0;
  for (int i = 0; i < NP; ++i) {
    const GemmArgs &g = i ? *b : a;
    unsigned grid = 0;
    const int gx = xcd_cut(g, BM, BN, &grid);
    L->p[i] = GemmProblem<T>{(const T *)g.A, g.lda, (const T *)g.W, g.ldw, g.M, vec_epilogue_ok(g) ? 1 : 0, gx, make_epilogue<T>(g)};
    if (i == 0) L->grid0 = grid;
    total += grid;
  }
  L->N = a.N; L->K = a.K; L->grid = total;
  return total;
}

// go(number of problems, epilogue), both as integral constants; a pair's two GEMMs have the same epilogue (gemm_pair_one_launch)
template <typename F>
inline hipError_t for_launch_form(const GemmArgs &a, const GemmArgs *b, F &&go) {
  auto with = [&](auto em) { return b ? go(std::integral_constant<int, 2>{}, em) : go(std::integral_constant<int, 1>{}, em); };
  switch (gemm_epilogue_form(a)) {
    case EM_KV_ROUTE: return with(std::integral_constant<int, EM_KV_ROUTE>{});
    case EM_RESIDUAL: return with(std::integral_constant<int, EM_RESIDUAL>{});
    case EM_STORE_ERF: return with(std::integral_constant<int, EM_STORE_ERF>{});
    default: return with(std::integral_constant<int, EM_STORE>{});
  }
}

// tiles of a launch of one or two GEMMs
inline int64_t launch_tiles(const GemmArgs &a, const GemmArgs *b, int bm, int bn) {
  return (int64_t)((a.M + bm - 1) / bm + (b ? (b->M + bm - 1) / bm : 0)) * ((a.N + bn - 1) / bn);
}

}  // namespace

}  // namespace pf
