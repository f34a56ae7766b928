"""Calls with text rows (GPU) whose output rows lie over input rows: y over x and text_out over text as the header allows, and
every other way of laying the four arrays into one buffer, where a call must have read its inputs before it writes over them.
Against the float64 oracle, at the stage's bars."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle.pf_oracle import StageOracle

pytestmark = pytest.mark.gpu


def _places(n, T):
    """First rows of (text, x, text_out, y) in one buffer of 2 * (n + T) rows."""
    return {"apart": (0, T, T + n, 2 * T + n), "aliased": (0, T, 0, T), "swapped": (0, T, n, 0), "text_out over x": (0, T, T + 3, T + n),
            "y over text": (n, n + T, 0, T), "y shifted": (0, T, T + n + 5, T + 5), "both shifted": (0, T, 5, T + 5)}


@pytest.mark.parametrize("place", list(_places(1, 1)))
@pytest.mark.parametrize("name,kw", [("C3s", {}), ("C3p", dict(n_layers=1)), ("K2f", {}), ("C4s", dict(text_len=256, n_layers=1)), ("C4s", {}), ("C3s", dict(batch=2))])
def test_output_rows_over_input_rows(name, kw, place):
    from paper_2405_14430_amd import Stage
    cfg = wl.variant(wl.CONFIGS[name], **kw)
    print(name, kw, place, flush=True)
    B, n, T, d = cfg.get("batch", 1), wl.patch_rows(cfg), cfg["text_len"], cfg["hidden"]
    W, acts = wl.make_weights(cfg), [wl.make_activations(dict(cfg, batch=1, seed=cfg["seed"] + 100 * b)) for b in range(B)]
    tol = 1e-4 if cfg["dtype"] == "f32" else 2e-2
    lead = (B,) if B > 1 else ()

    def dev(key, rows=slice(None)):
        a = np.stack([x[key][rows] for x in acts])
        return torch.from_numpy(np.ascontiguousarray(a.reshape(lead + a.shape[1:]), dtype=np.float32)).cuda()

    st = Stage(cfg, W)
    st.kv_init(dev("x_prev"), dev("cond"), dev("text"))
    buf = torch.full((2 * (n + T) * B, d), float("nan"), device="cuda")
    text, x, text_out, y = (buf[r * B:(r + k) * B].view(*lead, k, d) for r, k in zip(_places(n, T)[place], (T, n, T, n)))
    text.copy_(dev("text"))
    x.copy_(dev("x", slice(0, n)))
    st.patch_forward(x, dev("cond"), 0, text=text, out=y, text_out=text_out)
    for b, a in enumerate(acts):
        orc = StageOracle(dict(cfg, batch=1), W)
        orc.kv_init(a["x_prev"], a["cond"], a["text"])
        for got, ref in zip((y, text_out), orc.patch_forward(a["x"][:n], a["cond"], 0, a["text"])):
            got = (got[b] if B > 1 else got).double().cpu().numpy()
            assert float(np.max(np.abs(got - ref)) / np.sqrt(np.mean(ref ** 2))) <= tol
