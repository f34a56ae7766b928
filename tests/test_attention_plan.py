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


# us of an fp32 launch with its combine pass on the plain kernel, by split count (an MI355X)
MEASURED = {
    (48, 24, 1024, 64): {1: 4375, 2: 2300, 3: 1559, 4: 1182, 5: 976, 6: 1421, 8: 1195, 10: 1000, 12: 1225, 16: 974},
    (48, 12, 1024, 64): {1: 4305, 2: 2283, 3: 1545, 4: 1172, 5: 953, 6: 814, 8: 612, 10: 509, 12: 804, 16: 632},
    (32, 12, 512, 64): {1: 4077, 2: 2102, 3: 1443, 4: 1088, 5: 885, 6: 761, 8: 565, 10: 466, 12: 398, 16: 303},
    (48, 24, 4096, 64): {1: 4451, 2: 4486, 3: 4399, 4: 3435, 5: 3623, 6: 3696, 8: 3484, 10: 3891, 12: 4096, 16: 4219},
    (96, 12, 1024, 64): {1: 12953, 2: 6749, 3: 4514, 4: 3411, 5: 2805, 6: 4071, 8: 3351, 10: 2771, 12: 3401, 16: 2643},
    (96, 24, 1024, 64): {1: 13091, 2: 6750, 3: 8554, 4: 6629, 5: 5419, 6: 6312, 8: 5177, 10: 5394, 12: 5679, 16: 5258},
}


@pytest.mark.parametrize("head_dim,heads,nq,side", list(MEASURED))
def test_plain_kernel_splits_fill_the_chip(head_dim, heads, nq, side):
    us = MEASURED[head_dim, heads, nq, side]
    splits = _splits(B.load_library(), B.PF_PATH_AUTO, "f32", head_dim, heads, side, 4, nq)
    assert us[splits] <= 1.07 * min(us.values()), splits
