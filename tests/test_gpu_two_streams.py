"""Calls with text rows (GPU) where their rows take a route of their own: both streams of a two-stream block in one launch,
text and image rows read and written where the caller keeps them, rows that are not 16-byte aligned, stacks of one layer, and
heads of 128 channels normalised in tiles of 64 rows.  Against the float64 oracle, at the stage's bars (fp32 1e-4, bf16 2e-2 of
the output's rms: see test_gpu_stage.py)."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle.pf_oracle import StageOracle

pytestmark = pytest.mark.gpu

CASES = [("C4s", dict(text_len=256, n_layers=2)), ("C4s", dict(text_len=256, n_layers=1)), ("C4n", dict(text_len=256, n_layers=3)),
         ("C4n", {}), ("K3n", dict(text_len=256)), ("C3s", dict(n_layers=1)), ("C3p", dict(n_layers=1)), ("C3n", dict(text_len=64)), ("K2n", {})]


def _dev(a, shift):
    """A device copy of `a` that starts `shift` floats past a 16-byte boundary."""
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    buf = torch.empty(t.numel() + 4, device="cuda")
    return buf[shift:shift + t.numel()].view(t.shape).copy_(t)


def _err(got, ref):
    return float(np.max(np.abs(got.double().cpu().numpy() - ref)) / np.sqrt(np.mean(ref ** 2)))


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("name,kw", CASES)
def test_calls_with_text_rows(name, kw, shift):
    from paper_2405_14430_amd import Stage
    cfg = wl.variant(wl.CONFIGS[name], **kw)
    print(name, kw, shift, flush=True)
    W, A = wl.make_weights(cfg), wl.make_activations(cfg)
    st, orc = Stage(cfg, W), StageOracle(cfg, W)
    tol = 1e-4 if cfg["dtype"] == "f32" else 2e-2
    n = wl.patch_rows(cfg)
    x_prev, cond, text = _dev(A["x_prev"], 0), _dev(A["cond"], 0), _dev(A["text"], shift)
    y, t = st.kv_init(x_prev, cond, text, want_output=True)
    ry, rt = orc.kv_init(A["x_prev"], A["cond"], A["text"])
    assert _err(y, ry) <= tol and _err(t, rt) <= tol
    x = _dev(A["x"][:n], 0)
    for out_text in (torch.empty_like(text), text):      # the text rows' output may be their input
        before = text.clone()
        y, t = st.patch_forward(x, cond, 0, text=text, text_out=out_text)
        ry, rt = orc.patch_forward(A["x"][:n], A["cond"], 0, A["text"])
        assert _err(y, ry) <= tol and _err(t, rt) <= tol
        assert out_text is text or torch.equal(text, before)
    assert torch.equal(x, torch.from_numpy(A["x"][:n]).cuda())
