"""V^T rows of the fused K/V route (GPU) wherever they start in the buffer: the same rows are projected behind text of every
length mod 8, into patches that start anywhere mod 8, and with a second image, whose rows start elsewhere in a tile.  What
reaches the buffer is the same bits as behind 64 rows of text, and nothing else in the buffer changes."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("name,n,patches", [("C3s", 270, 4), ("C3n", 131, 2), ("C3r", 64, 3), ("K2f", 67, 3), ("C4s", 301, 2), ("K3f", 33, 3), ("C3s", 1100, 2)])
def test_rows_are_the_same_bits_at_every_offset(name, n, patches, batch):
    from paper_2405_14430_amd import Stage
    base = wl.variant(wl.CONFIGS[name], n_layers=1, n_patches=patches, seq_img=n * patches, grid_h=patches, grid_w=n, text_len=64, batch=batch)
    print(name, n, patches, batch, flush=True)
    W = wl.make_weights(base)
    g = torch.Generator(device="cuda").manual_seed(7)
    lead = (batch,) if batch > 1 else ()
    r = lambda *s: torch.randn(*lead, *s, generator=g, device="cuda")
    x, cond, text = r(n, base["hidden"]), r(base["hidden"]), r(72, base["hidden"])
    want = {}
    for T in range(64, 73):
        st = Stage(dict(base, text_len=T), W)
        for p in (0, patches - 1):
            st.kv_init()                                         # zeroes the buffers
            with_text = p == 0
            st.patch_forward(x, cond, p, text=text[..., :T, :].contiguous() if with_text else None)
            first, got = T + p * n, []
            for b in range(batch):
                K, V, _ = st.kv_view(0, b)
                for buf in (K, V):
                    got.append(buf[first:first + n].clone())
                    if with_text:
                        got.append(buf[:64].clone())
                        assert buf[:T].any(dim=-1).all()
                    buf[first:first + n] = 0
                    buf[:T if with_text else 0] = 0
            assert not st.kv.any()                               # the other rows and the padding
            for a, b in zip(got, want.setdefault(p, got)):
                assert torch.equal(a, b), (T, p)
