"""Key splits of launches that run on the plain attention kernel (CPU, host-only query): the same kernel gets the same split
count whether it was asked for (kernel_path) or is what the head size falls back to."""
import ctypes as C

import pytest

from paper_2405_14430_amd import binding as B


def _splits(lib, kernel_path, dtype, head_dim, heads, side, patches, nq):
    hidden = heads * head_dim
    cfg = dict(kind=0, dtype=dtype, n_layers=1, hidden=hidden, n_heads=heads, head_dim=head_dim, mlp_dim=4 * hidden,
               seq_img=side * side, grid_h=side, grid_w=side, n_patches=patches)
    c = B.make_config(cfg, kernel_path)
    lw = (B.PfLayerWeights * 1)()
    for f in B._W_FIELDS:
        setattr(lw[0], f, 0x100000)
    h, out, need, have = C.c_void_p(), C.c_int(), C.c_size_t(), C.c_size_t()
    assert lib.pf_stage_create(C.byref(c), lw, C.c_void_p(0x200000), 1 << 40, C.c_void_p(0x300000), 1 << 40, None, C.byref(h)) == 0
    assert lib.pf_stage_attention_plan(h, nq, 0, C.byref(out), C.byref(need), C.byref(have)) == 0
    lib.pf_stage_destroy(h)
    return out.value


@pytest.mark.parametrize("head_dim", [8, 32, 48, 96, 112])
@pytest.mark.parametrize("heads", [2, 12, 24])
@pytest.mark.parametrize("side,patches", [(16, 4), (30, 3), (64, 16), (64, 8), (64, 4), (128, 8)])
def test_plain_kernel_launches_split_alike(head_dim, heads, side, patches):
    lib = B.load_library()
    for nq in (1, side * side // patches, side * side):
        args = ("f32", head_dim, heads, side, patches, nq)
        assert _splits(lib, B.PF_PATH_AUTO, *args) == _splits(lib, B.PF_PATH_SIMT, *args)
    # 1024 queries x 24 heads over 4096 keys: 384 workgroups of 64 queries, best split in four (3901 us against 5321 in two)
    if (heads, side, patches, head_dim) == (24, 64, 4, 48):
        assert _splits(lib, B.PF_PATH_AUTO, "f32", 48, 24, 64, 4, 1024) == 4
