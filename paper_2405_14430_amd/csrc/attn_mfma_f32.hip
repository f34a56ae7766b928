// fp32 MFMA patch attention for head sizes 64 / 72 / 128 (gfx950): queries of a patch over all rows of the layer's K/V
// buffer, online softmax, fp32 throughout.
//
// Bound by the fp32 matrix rate (4 nq kv dh flops at 157 TFLOP/s).  Computed transposed with v_mfma_f32_16x16x4_f32 so that
// the score accumulators are the operands of the second product as they are:
//   S^T[kv][q] = K[kv][:] . Q[q][:]       A = K tile (LDS), B = Q fragments (registers)
//   O^T[c][q] += V^T[c][kv] P^T[kv][q]    A = V^T tile (LDS), B = P^T
// In the 16x16 accumulator layout lane l holds column (query) l % 16 and rows 4 g + r, g = l / 16, r = 0..3; the B operand of a
// K = 4 step takes k = g from lane group g, so register r of a score block is the operand for keys {r, 4 + r, 8 + r, 12 + r}
// and the matching A operands for r = 0..3 are four consecutive keys of a V^T row: one 16-byte LDS read for four MFMAs, no
// exchange between lanes.  The channels of the first product are grouped the same way.  16-wide blocks fit 72 channels (80
// rows of O^T; 32-wide blocks would compute 96).
//
// Workgroup: 4 waves x 16 queries, one head, one split of the keys; 32-key tiles go through registers into a double
// buffer (rows padded by 16 bytes: conflict-free 16-byte reads), one barrier per tile, the next tile's global loads in
// flight during the MFMAs of the current one.  512 queries x 16 heads x 4096 keys, dh = 72, fp32: 1386 us with the plain
// kernel (one query per thread, 512 one-wave workgroups); whole one-block PixArt-scale call 2501 -> 426 us with the MFMA
// GEMMs, the 64-token call 368 -> 45 us.
#include "common.h"
#include "ops.h"

namespace pf {

namespace {

constexpr int TQ = 64;   // queries per workgroup
constexpr int TK = 32;   // keys per tile
constexpr int NT = 256;

template <int DH>
struct FCfg {
  static constexpr int KS = DH / 16;                 // 16-channel steps of the first product
  static constexpr bool TAIL = DH % 16 == 8;         // and one of 8
  static constexpr int CB = (DH + 15) / 16;          // 16-channel blocks of O^T
  static constexpr int KLD = DH + 4, VLD = TK + 4;   // LDS row strides (floats)
  static constexpr int BUF = TK * KLD + DH * VLD;    // floats per buffer
  static constexpr int CH = TK * DH / 4;             // 16-byte chunks of a K (or V^T) tile
  static constexpr int NC = (CH + NT - 1) / NT;      // per thread
};

template <int DH>
__global__ __launch_bounds__(NT) void attn_mfma_f32_kernel(const float *__restrict__ q, int64_t ldq,
                                                           const float *__restrict__ kbuf, const float *__restrict__ vtbuf,
                                                           int kv_rows, int Lp, int H, float *__restrict__ out, int64_t ldo,
                                                           int nq, int splits, int qtiles, float *__restrict__ ws, int hpi) {
  // H counts heads over all images of the call (image-major, hpi heads per image); q / out rows are image-major too
  using C = FCfg<DH>;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;

  // workgroup id -> (head, query tile, split); all workgroups of a head on one XCD (ids are dealt round-robin to the 8)
  int L = blockIdx.x;
  const int per_xcd = gridDim.x >> 3;
  if (L < per_xcd * 8) L = (L & 7) * per_xcd + (L >> 3);
  const int per_head = qtiles * splits;
  const int h = L / per_head, rem = L - h * per_head;
  const int qt = rem / splits, sp = rem - qt * splits;
  const int qi = qt * TQ + wave * 16 + l16;

  const int tiles = (kv_rows + TK - 1) / TK;
  const int tps = (tiles + splits - 1) / splits;
  const int t_begin = sp * tps, t_end = min(tiles, t_begin + tps);
  const float *kh = kbuf + (size_t)h * Lp * DH;
  const float *vh = vtbuf + (size_t)h * DH * Lp;

  // tile staging: rows of the padded buffer past kv_rows are readable but may hold anything
  float4 kreg[C::NC], vreg[C::NC];
  auto fetch = [&](int t) {
#pragma unroll
    for (int i = 0; i < C::NC; ++i) {
      const int e = tid + i * NT;
      if (C::CH % NT != 0 && e >= C::CH) break;
      kreg[i] = *reinterpret_cast<const float4 *>(kh + (size_t)t * TK * DH + e * 4);
      vreg[i] = *reinterpret_cast<const float4 *>(vh + (size_t)(e >> 3) * Lp + t * TK + (e & 7) * 4);
    }
  };
  auto store = [&](int buf, int t) {
    float *kt = lds + buf * C::BUF, *vt = kt + TK * C::KLD;
#pragma unroll
    for (int i = 0; i < C::NC; ++i) {
      const int e = tid + i * NT;
      if (C::CH % NT != 0 && e >= C::CH) break;
      const int r = e / (DH / 4), c = e - r * (DH / 4);
      *reinterpret_cast<float4 *>(kt + r * C::KLD + c * 4) = kreg[i];
      float4 v = vreg[i];
      const int left = kv_rows - (t * TK + (e & 7) * 4);   // a weight of 0 must not meet a NaN of the padding
      if (left < 4) {
        if (left < 1) v.x = 0.f;
        if (left < 2) v.y = 0.f;
        if (left < 3) v.z = 0.f;
        v.w = 0.f;
      }
      *reinterpret_cast<float4 *>(vt + (e >> 3) * C::VLD + (e & 7) * 4) = v;
    }
  };
  if (t_begin < t_end) fetch(t_begin);

  // Q fragments, scaled: lane group g holds channels 16 s + 4 g .. + 3 of query qi (tail: 16 KS + 2 g, + 1)
  const float scale = 1.0f / sqrtf((float)DH);
  f32x4 qf[C::KS];
  float2 qtail = make_float2(0.f, 0.f);
  {
    const float *qp = q + ((size_t)(h / hpi) * nq + qi) * ldq + (size_t)(h % hpi) * DH;
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (qi < nq) v = *reinterpret_cast<const f32x4 *>(qp + s * 16 + g * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) qf[s][e] = v[e] * scale;
    }
    if constexpr (C::TAIL) {
      if (qi < nq) qtail = *reinterpret_cast<const float2 *>(qp + C::KS * 16 + g * 2);
      qtail.x *= scale; qtail.y *= scale;
    }
  }

  f32x4 o[C::CB];
#pragma unroll
  for (int cb = 0; cb < C::CB; ++cb) o[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;   // running maximum of the query; this lane's part of the sum

  if (t_begin < t_end) store(0, t_begin);
  for (int t = t_begin; t < t_end; ++t) {
    const int buf = (t - t_begin) & 1;
    __syncthreads();              // tile t is in LDS; everyone is done with the other buffer
    if (t + 1 < t_end) fetch(t + 1);
    const float *kt = lds + buf * C::BUF, *vt = kt + TK * C::KLD;
    f32x4 s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
      f32x4 a[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) a[b] = *reinterpret_cast<const f32x4 *>(kt + (b * 16 + l16) * C::KLD + ks * 16 + g * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int b = 0; b < 2; ++b) s[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][e], qf[ks][e], s[b], 0, 0, 0);
    }
    if constexpr (C::TAIL) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const float2 a = *reinterpret_cast<const float2 *>(kt + (b * 16 + l16) * C::KLD + C::KS * 16 + g * 2);
        s[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, qtail.x, s[b], 0, 0, 0);
        s[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, qtail.y, s[b], 0, 0, 0);
      }
    }
    if ((t + 1) * TK > kv_rows) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (t * TK + b * 16 + 4 * g + r >= kv_rows) s[b][r] = -INFINITY;
    }
    float tmax = s[0][0];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) tmax = fmaxf(tmax, s[b][r]);
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16, kWave));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, kWave));
    const float m_new = fmaxf(m, tmax);
    const float alpha = expf(m - m_new);   // 0 on the first tile
    m = m_new;
    float psum = 0.f;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[b][r] = expf(s[b][r] - m_new);
        psum += s[b][r];
      }
    l = l * alpha + psum;
#pragma unroll
    for (int cb = 0; cb < C::CB; ++cb)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[cb][r] *= alpha;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      f32x4 a[C::CB];
#pragma unroll
      for (int cb = 0; cb < C::CB; ++cb) {
        const int c = DH % 16 ? min(cb * 16 + l16, DH - 1) : cb * 16 + l16;   // rows past DH repeat the last (never stored)
        a[cb] = *reinterpret_cast<const f32x4 *>(vt + c * C::VLD + b * 16 + g * 4);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int cb = 0; cb < C::CB; ++cb) o[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[cb][r], s[b][r], o[cb], 0, 0, 0);
    }
    if (t + 1 < t_end) store(buf ^ 1, t + 1);
  }

  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);
  if (qi >= nq) return;
  if (splits == 1) {
    const float inv = 1.f / l;
    float *op = out + ((size_t)(h / hpi) * nq + qi) * ldo + (size_t)(h % hpi) * DH;
#pragma unroll
    for (int cb = 0; cb < C::CB; ++cb) {
      const int c = cb * 16 + 4 * g;
      if (c < DH) {   // (the caller's output rows are 8-byte aligned)
        *reinterpret_cast<float2 *>(op + c) = make_float2(o[cb][0] * inv, o[cb][1] * inv);
        *reinterpret_cast<float2 *>(op + c + 2) = make_float2(o[cb][2] * inv, o[cb][3] * inv);
      }
    }
  } else {   // partial result for the combine kernel: numerators, reference maximum, denominator
    const int d = H * DH;
    float *op = ws + ((size_t)sp * nq + qi) * d + (size_t)h * DH;
#pragma unroll
    for (int cb = 0; cb < C::CB; ++cb) {
      const int c = cb * 16 + 4 * g;
      if (c < DH) *reinterpret_cast<f32x4 *>(op + c) = o[cb];
    }
    if (g == 0) {
      float *ml = ws + (size_t)splits * nq * d + (((size_t)sp * nq + qi) * H + h) * 2;
      ml[0] = m;
      ml[1] = l;
    }
  }
}

template <int DH>
hipError_t launch(const AttnArgs &a, hipStream_t s) {
  constexpr int smem = 2 * FCfg<DH>::BUF * 4;
  if (hipError_t e = allow_dynamic_lds<&attn_mfma_f32_kernel<DH>, smem>(); e != hipSuccess) return e;
  const int B = a.batch > 1 ? a.batch : 1, qtiles = (a.nq + TQ - 1) / TQ;
  attn_mfma_f32_kernel<DH><<<dim3((unsigned)(qtiles * a.n_heads * B * a.splits)), NT, smem, s>>>(
      (const float *)a.q, a.ldq, (const float *)a.kbuf, (const float *)a.vtbuf, a.kv_rows, a.rows_padded, a.n_heads * B,
      (float *)a.out, a.ldo, a.nq, a.splits, qtiles, a.ws, a.n_heads);
  return hipGetLastError();
}

}  // namespace

bool attn_mfma_f32_head_size(int head_dim) { return head_dim == 64 || head_dim == 72 || head_dim == 128; }

// whole 32-row tiles of the padded buffers, 16-byte operand rows, 8-byte output rows; anything else stays with the plain kernel
bool attn_mfma_f32_supported(const AttnArgs &a) {
  return a.dt == DT_F32 && a.path != PATH_SIMT && attn_mfma_f32_head_size(a.head_dim) && a.rows_padded % TK == 0 &&
         a.kv_rows <= a.rows_padded && a.ldq % 4 == 0 && a.ldo % 2 == 0 &&
         (((uintptr_t)a.q | (uintptr_t)a.kbuf | (uintptr_t)a.vtbuf) & 15) == 0 && ((uintptr_t)a.out & 7) == 0;
}

hipError_t launch_attn_mfma_f32(const AttnArgs &a, hipStream_t s) {
  if (a.nq <= 0) return hipSuccess;
  if (a.head_dim == 64) return launch<64>(a, s);
  if (a.head_dim == 72) return launch<72>(a, s);
  return launch<128>(a, s);
}

}  // namespace pf
