"""K loops of the bf16 GEMM tiles at the lengths where their rings fill and drain (GPU), and the workgroups that read ahead for
launches that leave CUs idle.  Against float64 torch.

Bars: an output of bf16 type is off by one rounding, 2^-8 of the element, beside 1e-3 rms for fp32 sums taken in another order; one
of fp32 type by a random walk of K roundings of its partial sums, 12 x 2^-24 sqrt(K) of the rms at the largest of 10^6 elements."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
BF = torch.bfloat16
PIN = {"256x256": 1, "256x128": 3, "wavek": 6, "128x192": 10, "256x192": 11}


def _check(tile, M, N, K, pad=0, shift=0):
    from paper_2405_14430_amd import binding as B
    print("loop", tile, M, N, K, pad, shift, flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 5 * K + pad + shift)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    A = r(M, K + pad).to(BF)[:, :K]
    W = (r(N, K + pad) / math.sqrt(K)).to(BF)[:, :K]
    b = torch.empty(N + 8, dtype=BF, device="cuda")[shift:shift + N].copy_(r(N))
    gate, R = r(N), r(M, N)
    lin = A.double() @ W.double().T + b.double()
    got = B.pf_op_gemm(A, W, b, tile=PIN[tile])
    assert bool(((got.double() - lin).abs() <= lin.abs() / 256 + 1e-3 * lin.square().mean().sqrt()).all())
    x, copy = B.pf_op_gemm(A, W, b, epilogue=1, gate=gate, R=R, want_copy=True, tile=PIN[tile])
    ref = R.double() + gate.double() * lin
    bar = (12 * math.sqrt(K) + 32) * 2.0 ** -24 * gate.abs().max().double() * lin.square().mean().sqrt() + 2.0 ** -23 * ref.abs()
    assert bool(((x.double() - ref).abs() <= bar).all())
    assert torch.equal(copy, x.to(BF))
    none = B.pf_op_gemm(A, W, None, tile=PIN[tile])
    assert bool(((none.double() + b.double() - lin).abs() <= none.double().abs() / 256 + 1e-3 * lin.square().mean().sqrt()).all())


# one to seven and a few more K tiles: fewer than either ring holds, odd and even, past the first turn of both rings
@pytest.mark.parametrize("tile", ["256x256", "256x192", "256x128", "128x192"])
@pytest.mark.parametrize("nk", [1, 2, 3, 4, 5, 6, 7, 12, 17])
def test_loop_lengths(tile, nk):
    _check(tile, 300, 520, 64 * nk)


# a single row, rows and columns one past a tile, columns that are no multiple of eight, padded rows, an unaligned bias
@pytest.mark.parametrize("tile", ["256x256", "256x192", "256x128", "128x192", "wavek"])
@pytest.mark.parametrize("M,N,pad,shift", [(1, 8, 0, 0), (257, 385, 0, 0), (129, 194, 8, 0), (513, 264, 64, 1)])
def test_edges(tile, M, N, pad, shift):
    _check(tile, M, N, 448, pad, shift)


# read-ahead workgroups: fewer K tiles than workgroups, a block of the grid without rows, one tile, a full grid (none)
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (65, 1152, 1152), (512, 1152, 4608), (70, 1000, 192), (500, 1156, 1152), (1024, 1024, 1024)])
def test_read_ahead(M, N, K):
    _check("wavek", M, N, K)


# the most readers of an XCD and the fewest, two rounds of loads (the second one not full), XCDs without weight rows, too few readers (none), padded rows
@pytest.mark.parametrize("M,N,K,pad", [(64, 3072, 2048, 0), (700, 1150, 1152, 0), (60, 10200, 320, 0), (200, 3456, 1152, 0), (1, 136, 512, 8), (768, 1152, 256, 0), (130, 1536, 1536, 64)])
def test_read_ahead_readers(M, N, K, pad):
    _check("wavek", M, N, K, pad)
