"""Per-head norm and RoPE in the QKV projection's epilogue (GPU) on the tiles that the stages of a few hundred rows do not reach:
one layer at the real widths, ragged rows, against the float64 oracle.

Bars as in the stage tests; K and V rows are stored in bf16, one rounding (2^-8) of the value beside the bar."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle.pf_oracle import StageOracle

pytestmark = pytest.mark.gpu
TOL = 2e-2


# with the tile that the rule gives the image rows (the text rows of the first case are in the same GEMM)
@pytest.mark.parametrize("name,grid_h,grid_w,text,with_text,tile", [
    ("C4", 34, 59, 77, True, "256,256"), ("C4", 40, 35, 45, False, "128,128"), ("C4", 80, 51, 30, False, "128,128"),
    ("C3", 80, 50, 77, False, "256,192"), ("C3", 100, 60, 29, False, "256,256"), ("C3", 100, 80, 154, False, "128,192")])
def test_norm_and_rope_on_large_tiles(name, grid_h, grid_w, text, with_text, tile):
    from paper_2405_14430_amd import Stage, binding as B
    base = wl.CONFIGS[name]
    cfg = wl.variant(base, n_layers=1, n_patches=2, seq_img=grid_h * grid_w, grid_h=grid_h, grid_w=grid_w, text_len=text,
                     mlp_dim=base["hidden"], qk_norm=1, joint_rope=1 if name == "C3" else 0)
    rows = grid_h * grid_w // 2 + (text if with_text else 0)
    assert f"gemm_tile_kernel<{tile}," in B.load_library().pf_gemm_qkv_kernel_name(rows, cfg["hidden"], cfg["head_dim"], 1).decode()
    print("norm tiles", name, grid_h, grid_w, text, with_text, flush=True)
    W, A = wl.make_weights(cfg), wl.make_activations(cfg)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    st, orc = Stage(cfg, W), StageOracle(cfg, W)
    st.kv_init(None)
    orc.kv_init(None)
    n, p = wl.patch_rows(cfg), 0 if with_text else 1
    xp = A["x"][p * n:(p + 1) * n]
    got = st.patch_forward(dev(xp), dev(A["cond"]), p, text=dev(A["text"]) if with_text else None)
    ref = orc.patch_forward(xp, A["cond"], p, A["text"] if with_text else None)
    for g, r in zip(got, ref) if with_text else [(got, ref)]:
        assert np.max(np.abs(g.double().cpu().numpy() - r)) / np.sqrt(np.mean(r ** 2)) < TOL
    K, V, _ = st.kv_view(0)
    for buf, want in ((K, orc.kbuf[0]), (V, orc.vbuf[0])):
        g = buf.double().cpu().numpy().reshape(len(want), -1)
        assert np.max(np.abs(g - want) - 2.0 ** -8 * np.abs(want)) / np.sqrt(np.mean(want ** 2)) < TOL
        assert bool((np.abs(g).max(axis=1) > 0).sum() == n + (text if with_text else 0))   # the other rows stay zero
    st.destroy()
