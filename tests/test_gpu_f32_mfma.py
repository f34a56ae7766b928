"""fp32 MFMA GEMM and attention (GPU) at the edges of their tiles and dispatch rules, against float64 torch.

Bars: a sum of K products in fp32 is off by a random walk of K roundings of partial sums no larger than a few times the
result's rms: 2^-24 sqrt(K) per element typically, six times that at the largest of up to 10^6 elements, and a factor of two
for the epilogue.  A product of softmax weights and V adds the roundings of the score (|s| up to 30 here) to the exponent.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _pkg():
    import paper_2405_14430_amd.binding as B
    return B


def _err(got, ref):
    return float((got.double() - ref).abs().max() / ref.square().mean().sqrt())


# one K tile; ragged rows and columns of every variant (64x64: 1025 rows; K over four waves: 500 and 77 rows; over eight: the others);
# at most one tile per CU; many tiles; long K; K the kernels refuse
@pytest.mark.parametrize("M,N,K", [(1, 8, 32), (31, 40, 64), (33, 1000, 96), (65, 1544, 384), (300, 520, 6144), (1025, 1608, 160), (70, 72, 40), (500, 1160, 1152), (77, 4616, 1536)])
def test_gemm_f32(M, N, K):
    B = _pkg()
    print("gemm_f32", M, N, K, flush=True)
    name = B.load_library().pf_gemm_kernel_name(0, 0, M, N, K).decode()
    assert ("simt" in name) == (K % 32 != 0)
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N)
    A, W = torch.randn(M, K, generator=g, device="cuda"), torch.randn(N, K, generator=g, device="cuda") / math.sqrt(K)
    b, gate, R = (torch.randn(n, generator=g, device="cuda") for n in (N, N, M * N))
    lin = A.double() @ W.double().T + b.double()
    bar = 12 * 2.0 ** -24 * math.sqrt(K) + 4 * 2.0 ** -24
    half = N // 16 * 8
    ref = lin.clone()
    ref[:, half:] = torch.nn.functional.gelu(lin[:, half:], approximate="tanh")
    # the hardware exponential and reciprocal of the GELU: about 1 ulp each on the largest elements (5 rms)
    assert _err(B.pf_op_gemm(A, W, b, gelu_from=half), ref) <= bar + 32 * 2.0 ** -24
    R = R.view(M, N)
    got, copy = B.pf_op_gemm(A, W, b, epilogue=1, gate=gate, R=R, want_copy=True)
    assert _err(got, R.double() + gate.double() * lin) <= 4 * bar       # |gate| up to 4
    assert torch.equal(got, copy)


def test_gemm_f32_unaligned_operand_keeps_the_plain_kernel():
    """Rows that are not 16-byte aligned never reach the tile loads: a stage's weights may sit anywhere."""
    B = _pkg()
    from paper_2405_14430_amd import Stage
    import workloads as wl
    cfg = dict(wl.CONFIGS["K0f"], hidden=192)
    layers = wl.make_weights(cfg)
    a, b = Stage(cfg, layers), Stage(cfg, layers)
    moved = []
    for w in b._layers:
        for name in ("w_qkv", "w_o", "w_up", "w_down"):
            t = next(t for t in b._keep if t.data_ptr() == getattr(w, name))
            u = torch.empty(t.numel() + 1, device="cuda")
            u[1:] = t.flatten()
            moved.append(u)
            setattr(w, name, u.data_ptr() + 4)
    import ctypes as C
    b.destroy()
    assert b.lib.pf_stage_create(C.byref(b.c), b._layers, C.c_void_p(b.kv.data_ptr()), b.kv.numel(), C.c_void_p(b.ws.data_ptr()),
                                 b.ws.numel(), C.c_void_p(torch.cuda.current_stream().cuda_stream), C.byref(b.h)) == 0
    x = torch.randn(cfg["seq_img"], cfg["hidden"], device="cuda")
    cond = torch.randn(cfg["hidden"], device="cuda")
    ya, _ = a.kv_init(x, cond, want_output=True)
    yb, _ = b.kv_init(x, cond, want_output=True)
    assert _err(yb, ya.double()) <= 1e-4


@pytest.mark.parametrize("dh", [64, 72, 128])
@pytest.mark.parametrize("nq,kv_rows,splits", [(1, 1, 1), (63, 31, 1), (65, 33, 1), (100, 129, 2), (130, 300, 5), (64, 64, 3)])
def test_attention_f32(dh, nq, kv_rows, splits):
    """Rows past kv_rows hold NaN: neither the scores nor the zero weights may let them through."""
    B, H = _pkg(), 3
    print("attn_f32", dh, nq, kv_rows, splits, flush=True)
    assert B.load_library().pf_attention_kernel_name(0, 0, dh, nq, 0).decode() == "attn_mfma_f32_kernel"
    Lp = -(-kv_rows // 128) * 128
    g = torch.Generator(device="cuda").manual_seed(nq * 1000 + kv_rows + dh)
    q = 2.0 * torch.randn(nq, H * dh, generator=g, device="cuda")
    K, V = torch.randn(H, Lp, dh, generator=g, device="cuda"), torch.randn(H, dh, Lp, generator=g, device="cuda")
    K[:, kv_rows:], V[:, :, kv_rows:] = float("nan"), float("nan")
    s = torch.matmul(q.double().view(nq, H, dh).transpose(0, 1), K[:, :kv_rows].double().transpose(1, 2).contiguous()) / math.sqrt(dh)
    p = torch.softmax(s, -1)
    ref = torch.matmul(p, V[:, :, :kv_rows].double().transpose(1, 2).contiguous()).transpose(0, 1).reshape(nq, H * dh)
    got = B.pf_op_attention(q, K.contiguous(), V.contiguous(), kv_rows, Lp, H, dh, splits=splits)
    smax = float(s.abs().max())
    # exponent: score roundings 2^-24 (sqrt(dh) + 2) |s|; then the sums over the keys
    bar = 12 * 2.0 ** -24 * (smax * (math.sqrt(dh) / 4 + 2) + math.sqrt(kv_rows) + 4)
    assert _err(got, ref) <= bar
