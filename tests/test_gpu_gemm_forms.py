"""GEMM kernel instances (GPU) that other tests pass by: the erf GELU, whose epilogue is compiled on its own for every tile and
for one and two problems, and the 64x128 tile.  Against float64 torch.

Bars: an output of fp32 type is off by a random walk of K roundings of its partial sums (12 x 2^-24 sqrt(K) of the rms at the
largest of 10^6 elements) and the roundings of erf (4 x 2^-24 of elements up to 5 rms); one of bf16 type by one rounding, 2^-8
of the element, beside 1e-3 rms for sums taken in another order (test_gpu_ops.py)."""
import math

import numpy as np
import pytest
import torch

import workloads as wl
from oracle.pf_oracle import StageOracle

pytestmark = pytest.mark.gpu
F32, BF = torch.float32, torch.bfloat16


def _operands(M, N, K, dtype):
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 5 * K)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return r(M, K).to(dtype), (r(N, K) / math.sqrt(K)).to(dtype), r(N).to(dtype)


def _ok(got, ref, K):
    rms = ref.square().mean().sqrt()
    if got.dtype == F32:
        return bool(((got.double() - ref).abs() <= (12 * math.sqrt(K) + 32) * 2.0 ** -24 * rms).all())
    return bool(((got.double() - ref).abs() <= ref.abs() / 256 + 1e-3 * rms).all())


# every bf16 tile on ragged shapes, the kernel for other K; fp32: 64x64, K over four and over eight waves, the plain kernel
@pytest.mark.parametrize("dtype,M,N,K,tile", [(BF, 777, 650, 320, t) for t in range(0, 13)] + [(BF, 100, 72, 72, 0)] +
                         [(F32, 33, 1000, 96, 0), (F32, 500, 1160, 1152, 0), (F32, 1025, 1608, 160, 0), (F32, 70, 72, 40, 0)])
def test_erf_gelu(dtype, M, N, K, tile):
    from paper_2405_14430_amd import binding as B
    A, W, b = _operands(M, N, K, dtype)
    print("erf", dtype, M, N, K, tile, flush=True)
    lin = A.double() @ W.double().T + b.double()
    gf = N // 2 + 3                                   # inside a tile and inside a group of eight columns
    ref = lin.clone()
    ref[:, gf:] = torch.nn.functional.gelu(lin[:, gf:])
    got = B.pf_op_gemm(A, W, b, gelu_from=gf, gelu_tanh=0, tile=tile)
    assert _ok(got, ref, K)
    if dtype == F32:                                  # (fine enough to tell the two forms apart)
        assert not _ok(B.pf_op_gemm(A, W, b, gelu_from=gf, gelu_tanh=1), ref, K)
    shifted = torch.empty(N + 8, dtype=dtype, device="cuda")[1:1 + N].copy_(b)                  # the path without vector access
    assert _ok(B.pf_op_gemm(A, W, shifted, gelu_from=gf, gelu_tanh=0, tile=tile), ref, K)


@pytest.mark.parametrize("name,kw", [("C3s", {}), ("K2f", {}), ("C2x", {}), ("C4s", {})])
def test_stage_with_erf_gelu(name, kw):
    """One and two streams; the bars of the stage tests."""
    from paper_2405_14430_amd import Stage
    cfg = wl.variant(wl.CONFIGS[name], gelu_tanh=0, **kw)
    print("erf stage", name, flush=True)
    W, A = wl.make_weights(cfg), wl.make_activations(cfg)
    st, orc = Stage(cfg, W), StageOracle(cfg, W)
    tol, n, joint = 1e-4 if cfg["dtype"] == "f32" else 2e-2, wl.patch_rows(cfg), cfg["kind"] in (2, 3)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    err = lambda got, ref: float(np.max(np.abs(got.double().cpu().numpy() - ref)) / np.sqrt(np.mean(ref ** 2)))
    text = dev(A["text"]) if joint else dev(A["text"]).to(st.dt)
    st.kv_init(dev(A["x_prev"]), dev(A["cond"]), text)
    orc.kv_init(A["x_prev"], A["cond"], A["text"])
    got = st.patch_forward(dev(A["x"][:n]), dev(A["cond"]), 0, text=text if joint else None)
    ref = orc.patch_forward(A["x"][:n], A["cond"], 0, A["text"] if joint else None)
    for g, r in zip(got, ref) if joint else [(got, ref)]:
        assert err(g, r) <= tol


# launches the rule gives it; fewer K tiles than ring stages; ragged rows and columns; a single row
@pytest.mark.parametrize("M,N,K", [(512, 4608, 1536), (500, 4616, 1536), (130, 200, 64), (130, 200, 128), (130, 200, 192), (1, 8, 320), (65, 129, 448)])
def test_tile_64x128(M, N, K):
    from paper_2405_14430_amd import binding as B
    A, W, b = _operands(M, N, K, BF)
    g = torch.Generator(device="cuda").manual_seed(1)
    gate, R = torch.randn(N, generator=g, device="cuda"), torch.randn(M, N, generator=g, device="cuda")
    tile = 2
    print("64x128", M, N, K, flush=True)
    lin = A.double() @ W.double().T + b.double()
    got = B.pf_op_gemm(A, W, b, gelu_from=N // 2, tile=tile)
    ref = lin.clone()
    ref[:, N // 2:] = torch.nn.functional.gelu(lin[:, N // 2:], approximate="tanh")
    assert _ok(got, ref, K)
    x, copy = B.pf_op_gemm(A, W, b, epilogue=1, gate=gate, R=R, want_copy=True, tile=tile)
    ref = R.double() + gate.double() * lin
    assert bool(((x.double() - ref).abs() <= 4e-3 * ref.square().mean().sqrt()).all())          # |gate| up to 4
    assert torch.equal(copy, x.to(BF))


@pytest.mark.parametrize("dtype", [BF, F32])
@pytest.mark.parametrize("M,N,K", [(70, 130, 128), (300, 1156, 512), (33, 9, 64), (2100, 1203, 320), (500, 4611, 1536)])
def test_columns_behind_the_last_group_of_eight(dtype, M, N, K):
    """N no multiple of eight in rows that are: whole groups by vectors, the rest by elements, the columns behind untouched."""
    import ctypes as C
    from paper_2405_14430_amd import binding as B
    print("tail", dtype, M, N, K, flush=True)
    lib, ld = B.load_library(), (N + 7) // 8 * 8
    A, W, b = _operands(M, N, K, dtype)
    g = torch.Generator(device="cuda").manual_seed(2)
    bias, gate = torch.zeros(ld, dtype=dtype, device="cuda"), torch.randn(ld, generator=g, device="cuda")
    bias[:N] = b
    R = torch.randn(M, ld, generator=g, device="cuda")
    out, X, X2 = (torch.full((M, ld), 7.0, dtype=t, device="cuda") for t in (dtype, F32, dtype))
    p = lambda t: C.c_void_p(t.data_ptr())
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    dt = int(dtype == BF)
    assert lib.pf_op_gemm(dt, 0, p(A), K, p(W), K, p(bias), p(out), ld, M, N, K, 0, N // 2, 1, None, None, 0, None, 0, stream) == 0
    assert lib.pf_op_gemm(dt, 0, p(A), K, p(W), K, p(bias), p(X), ld, M, N, K, 1, N, 1, p(gate), p(R), ld, p(X2), ld, stream) == 0
    lin = A.double() @ W.double().T + b.double()
    ref = lin.clone()
    ref[:, N // 2:] = torch.nn.functional.gelu(lin[:, N // 2:], approximate="tanh")
    assert _ok(out[:, :N], ref, K)
    ref = R[:, :N].double() + gate[:N].double() * lin
    assert bool(((X[:, :N].double() - ref).abs() <= (4e-3 if dt else 4 * (12 * math.sqrt(K) + 32) * 2.0 ** -24) * ref.square().mean().sqrt()).all())
    assert torch.equal(X2[:, :N], X[:, :N].to(dtype))
    for t in (out, X, X2):
        assert bool((t[:, N:] == 7.0).all())
