"""The GEMMs' tile rules and the banded tile walk (CPU, host-only queries).

The bf16 rule against measured launches: for shapes at the edges of its rounds - few rows
at wide outputs, one round and a little more, grids that an XCD's block of whole rows and columns pads - the tile it picks is
within an eighth of the fastest.  us per launch, plain store, isolated GEMMs with cold weights on an MI355X."""
import ctypes as C

import pytest

from paper_2405_14430_amd import binding as B

MEASURED = {
    (5362, 2048, 8192): {"<256,256,2,4,2,false>": 154.4, "<256,192,2,4,2,false>": 252.9, "<256,128,3,4,2,false>": 186.1, "<128,192,2,2,2,false>": 178.2, "<128,192,3,2,2,true>": 179.3, "<128,128,2,2,2,false>": 196.5, "<128,64,2,2,2,false>": 225.4, "<64,128,3,2,2,false>": 230.3},
    (10751, 1536, 7680): {"<256,256,2,4,2,false>": 294.8, "<256,192,2,4,2,false>": 252.2, "<256,128,3,4,2,false>": 275.4, "<128,192,2,2,2,false>": 251.7, "<128,192,3,2,2,true>": 250.4, "<128,128,2,2,2,false>": 299.6, "<128,64,2,2,2,false>": 331.9, "<64,128,3,2,2,false>": 334.2},
    (9409, 9216, 3072): {"<256,256,2,4,2,false>": 434.7, "<256,192,2,4,2,false>": 472.2, "<256,128,3,4,2,false>": 476.4, "<128,192,2,2,2,false>": 474.4, "<128,192,3,2,2,true>": 524.9, "<128,128,2,2,2,false>": 511.3, "<128,64,2,2,2,false>": 641.0, "<64,128,3,2,2,false>": 680.4},
    (431, 9216, 3072): {"<256,256,2,4,2,false>": 60.1, "<256,192,2,4,2,false>": 54.9, "<256,128,3,4,2,false>": 42.6, "<128,192,2,2,2,false>": 52.9, "<128,192,3,2,2,true>": 38.2, "<128,128,2,2,2,false>": 46.9, "<128,64,2,2,2,false>": 50.0, "<64,128,3,2,2,false>": 43.8},
    (512, 9216, 3072): {"<256,256,2,4,2,false>": 63.0, "<256,192,2,4,2,false>": 56.8, "<256,128,3,4,2,false>": 44.8, "<128,192,2,2,2,false>": 54.4, "<128,192,3,2,2,true>": 41.9, "<128,128,2,2,2,false>": 47.9, "<128,64,2,2,2,false>": 52.2, "<64,128,3,2,2,false>": 60.4},
    (5263, 1536, 1536): {"<256,256,2,4,2,false>": 34.0, "<256,192,2,4,2,false>": 32.0, "<256,128,3,4,2,false>": 43.3, "<128,192,2,2,2,false>": 36.2, "<128,192,3,2,2,true>": 39.1, "<128,128,2,2,2,false>": 44.7, "<128,64,2,2,2,false>": 41.1, "<64,128,3,2,2,false>": 38.7},
    (8283, 576, 2304): {"<256,256,2,4,2,false>": 43.0, "<256,192,2,4,2,false>": 40.1, "<256,128,3,4,2,false>": 30.5, "<128,192,2,2,2,false>": 38.8, "<128,192,3,2,2,true>": 29.4, "<128,128,2,2,2,false>": 34.9, "<128,64,2,2,2,false>": 35.4, "<64,128,3,2,2,false>": 40.9},
    (680, 6144, 1536): {"<256,256,2,4,2,false>": 33.5, "<256,192,2,4,2,false>": 31.0, "<256,128,3,4,2,false>": 24.3, "<128,192,2,2,2,false>": 29.1, "<128,192,3,2,2,true>": 22.3, "<128,128,2,2,2,false>": 25.4, "<128,64,2,2,2,false>": 27.9, "<64,128,3,2,2,false>": 32.7},
    (1038, 4608, 1152): {"<256,256,2,4,2,false>": 27.9, "<256,192,2,4,2,false>": 25.6, "<256,128,3,4,2,false>": 19.5, "<128,192,2,2,2,false>": 23.0, "<128,192,3,2,2,true>": 18.3, "<128,128,2,2,2,false>": 21.6, "<128,64,2,2,2,false>": 22.5, "<64,128,3,2,2,false>": 26.6},
    (7456, 768, 3840): {"<256,256,2,4,2,false>": 65.0, "<256,192,2,4,2,false>": 61.9, "<256,128,3,4,2,false>": 46.9, "<128,192,2,2,2,false>": 62.5, "<128,192,3,2,2,true>": 46.3, "<128,128,2,2,2,false>": 56.6, "<128,64,2,2,2,false>": 62.8, "<64,128,3,2,2,false>": 71.5},
    (2048, 9216, 3072): {"<256,256,2,4,2,false>": 132.7, "<256,192,2,4,2,false>": 115.0, "<256,128,3,4,2,false>": 123.4, "<128,192,2,2,2,false>": 113.3, "<128,192,3,2,2,true>": 117.0, "<128,128,2,2,2,false>": 132.0, "<128,64,2,2,2,false>": 149.2, "<64,128,3,2,2,false>": 167.8},
    (2560, 9216, 3072): {"<256,256,2,4,2,false>": 136.7, "<256,192,2,4,2,false>": 124.2, "<256,128,3,4,2,false>": 134.0, "<128,192,2,2,2,false>": 138.3, "<128,192,3,2,2,true>": 153.5, "<128,128,2,2,2,false>": 141.4, "<128,64,2,2,2,false>": 193.0, "<64,128,3,2,2,false>": 207.1},
    (16896, 9216, 3072): {"<256,256,2,4,2,false>": 745.6, "<256,192,2,4,2,false>": 805.5, "<256,128,3,4,2,false>": 861.7, "<128,192,2,2,2,false>": 838.5, "<128,192,3,2,2,true>": 941.2, "<128,128,2,2,2,false>": 901.5, "<128,64,2,2,2,false>": 1146.8, "<64,128,3,2,2,false>": 1187.4},
    (4096, 3456, 1152): {"<256,256,2,4,2,false>": 34.2, "<256,192,2,4,2,false>": 48.2, "<256,128,3,4,2,false>": 41.5, "<128,192,2,2,2,false>": 45.1, "<128,192,3,2,2,true>": 51.4, "<128,128,2,2,2,false>": 40.3, "<128,64,2,2,2,false>": 49.0, "<64,128,3,2,2,false>": 52.7},
    (3677, 8192, 2048): {"<256,256,2,4,2,false>": 106.2, "<256,192,2,4,2,false>": 126.0, "<256,128,3,4,2,false>": 127.5, "<128,192,2,2,2,false>": 131.7, "<128,192,3,2,2,true>": 152.1, "<128,128,2,2,2,false>": 127.9, "<128,64,2,2,2,false>": 158.3, "<64,128,3,2,2,false>": 170.8},
    (1024, 4608, 1536): {"<256,256,2,4,2,false>": 34.6, "<256,192,2,4,2,false>": 31.3, "<256,128,3,4,2,false>": 24.7, "<128,192,2,2,2,false>": 30.1, "<128,192,3,2,2,true>": 23.6, "<128,128,2,2,2,false>": 26.4, "<128,64,2,2,2,false>": 27.7, "<64,128,3,2,2,false>": 32.5},
    # fewer tiles, where the rule does not look at the epilogue: 430 to 528 tiles of 64x64, with a residual
    (633, 3072, 15360): {"gemm_wavek_kernel<64,64>": 107.1, "<64,64,4,2,2,false>": 120.5, "<64,128,3,2,2,false>": 116.4, "<64,64,2,2,2,false>": 166.0, "<128,64,2,2,2,false>": 177.8},
    (633, 3072, 12288): {"gemm_wavek_kernel<64,64>": 87.5, "<64,64,4,2,2,false>": 98.7, "<64,128,3,2,2,false>": 95.6, "<64,64,2,2,2,false>": 135.4, "<128,64,2,2,2,false>": 143.9},
    (569, 3072, 15360): {"gemm_wavek_kernel<64,64>": 107.4, "<64,64,4,2,2,false>": 92.4, "<64,128,3,2,2,false>": 115.2, "<64,64,2,2,2,false>": 165.3, "<128,64,2,2,2,false>": 177.5},
    (1275, 1536, 6144): {"gemm_wavek_kernel<64,64>": 45.7, "<64,64,4,2,2,false>": 50.0, "<64,128,3,2,2,false>": 49.3, "<64,64,2,2,2,false>": 67.2, "<128,64,2,2,2,false>": 72.6},
    (1339, 1536, 6144): {"gemm_wavek_kernel<64,64>": 63.4, "<64,64,4,2,2,false>": 64.0, "<64,128,3,2,2,false>": 51.5, "<64,64,2,2,2,false>": 67.8, "<128,64,2,2,2,false>": 73.4},
    (1211, 1536, 6144): {"gemm_wavek_kernel<64,64>": 45.5, "<64,64,4,2,2,false>": 40.0, "<64,128,3,2,2,false>": 49.8, "<64,64,2,2,2,false>": 68.1, "<128,64,2,2,2,false>": 73.2},
    (765, 2560, 10240): {"gemm_wavek_kernel<64,64>": 74.3, "<64,64,4,2,2,false>": 85.3, "<64,128,3,2,2,false>": 79.5, "<64,64,2,2,2,false>": 109.6, "<128,64,2,2,2,false>": 118.3},
    (1021, 2048, 8192): {"gemm_wavek_kernel<64,64>": 58.4, "<64,64,4,2,2,false>": 64.2, "<64,128,3,2,2,false>": 65.6, "<64,64,2,2,2,false>": 87.9, "<128,64,2,2,2,false>": 94.1},
    (1527, 1152, 4608): {"gemm_wavek_kernel<64,64>": 36.0, "<64,64,4,2,2,false>": 30.4, "<64,128,3,2,2,false>": 38.5, "<64,64,2,2,2,false>": 50.7, "<128,64,2,2,2,false>": 55.2},
    (1783, 1152, 4608): {"gemm_wavek_kernel<64,64>": 36.7, "<64,64,4,2,2,false>": 39.0, "<64,128,3,2,2,false>": 41.1, "<64,64,2,2,2,false>": 51.1, "<128,64,2,2,2,false>": 56.2},
    (1275, 1536, 1536): {"gemm_wavek_kernel<64,64>": 18.5, "<64,64,4,2,2,false>": 16.6, "<64,128,3,2,2,false>": 17.2, "<64,64,2,2,2,false>": 20.5, "<128,64,2,2,2,false>": 22.6},
}


@pytest.mark.parametrize("shape", list(MEASURED))
def test_rule_picks_a_tile_near_the_fastest(shape):
    us = MEASURED[shape]
    name = B.load_library().pf_gemm_kernel_name(1, 0, *shape).decode()
    assert us[name.replace("gemm_tile_kernel", "")] <= 1.125 * min(us.values()), (name, min(us, key=us.get))


# fp32 shapes of the GPU tests, one of every kernel and of the rule's edges (384 tiles of 64x64, 256 of 32x32, K = 6144)
@pytest.mark.parametrize("M,N,K,kernel", [
    (1025, 1608, 160, "gemm_f32_tile_kernel<64,64,3,2,2>"), (1024, 1536, 1152, "gemm_f32_tile_kernel<64,64,3,2,2>"),
    (1024, 1472, 1152, "gemm_f32_wavek_kernel<32,32,4>"), (500, 1160, 1152, "gemm_f32_wavek_kernel<32,32,4>"), (77, 4608, 1536, "gemm_f32_wavek_kernel<32,32,4>"),
    (512, 512, 1152, "gemm_f32_wavek_kernel<32,32,8>"), (33, 1000, 96, "gemm_f32_wavek_kernel<32,32,8>"), (300, 1544, 6144, "gemm_f32_wavek_kernel<32,32,8>"),
    (300, 1544, 6112, "gemm_f32_wavek_kernel<32,32,4>"), (70, 72, 40, "gemm_simt_kernel")])
def test_fp32_rule(M, N, K, kernel):
    assert B.load_library().pf_gemm_kernel_name(0, 0, M, N, K).decode() == kernel


# tile grids of at least four rounds per XCD, whose blocks are walked in bands: a lower last band (17 tile rows in bands of four),
# bands of both kinds of tiles, more rows than columns and the reverse
@pytest.mark.parametrize("M,N,bm,bn", [(16896, 12288, 256, 256), (16896, 9216, 256, 256), (65536, 3456, 128, 192), (16896, 3072, 128, 192), (17000, 9300, 128, 128), (3000, 60000, 128, 64), (30000, 20000, 64, 128)])
def test_banded_walk_covers_every_tile_once(M, N, bm, bn):
    lib = B.load_library()
    tiles_m, tiles_n = -(-M // bm), -(-N // bn)
    grid, tm, tn = C.c_uint(0), C.c_int(0), C.c_int(0)
    lib.pf_gemm_tile_map(M, N, bm, bn, 0, C.byref(grid), C.byref(tm), C.byref(tn))
    assert grid.value % 8 == 0
    seen, banded = set(), False
    for x in range(8):
        walk = []                                    # tiles of one XCD in the order of its workgroups
        for wg in range(x, grid.value, 8):
            if lib.pf_gemm_tile_map(M, N, bm, bn, wg, C.byref(grid), C.byref(tm), C.byref(tn)):
                walk.append((tm.value, tn.value))
        assert not seen.intersection(walk) and len(set(walk)) == len(walk)
        seen.update(walk)
        r0, c0 = min(t[0] for t in walk), min(t[1] for t in walk)
        rows, cols = max(t[0] for t in walk) - r0 + 1, max(t[1] for t in walk) - c0 + 1
        assert len(walk) == rows * cols              # a full rectangle
        # band height: rows before the second column; then whole bands, column by column, the last one maybe lower
        G = next((i for i, t in enumerate(walk) if t[1] != c0), len(walk))
        order = [(r0 + i, c0 + j) for b in range(0, rows, G) for j in range(cols) for i in range(b, min(b + G, rows))]
        assert walk == order
        banded = banded or G > 1
    assert banded and seen == {(i, j) for i in range(tiles_m) for j in range(tiles_n)}


# us of wave-split-K launches (residual; wide outputs of 64 rows: plain store), weights from HBM, without workgroups that read ahead and
# with as many as CUs were idle, up to 11 per XCD
READ_AHEAD = {
    (512, 1152, 4608): (20.5, 16.1), (256, 1152, 4608): (21.7, 15.5), (64, 3072, 15360): (66.7, 43.7), (375, 1536, 6144): (26.6, 19.8),
    (512, 1536, 6144): (26.6, 23.7), (576, 1152, 4608): (20.5, 19.0), (704, 1152, 4608): (20.8, 20.0), (64, 10240, 2560): (19.8, 18.5),
    (768, 1152, 4608): (20.7, 39.4), (768, 1152, 1152): (9.3, 10.3), (576, 1536, 6144): (26.7, 54.5), (640, 1536, 1536): (10.7, 11.5),
    (320, 3072, 15360): (63.3, 130.7), (320, 3072, 3072): (17.4, 20.1), (1100, 768, 3072): (15.0, 22.4), (64, 12288, 3072): (22.4, 23.9),
}


def _wavek_grid(lib, M, N):
    """(workgroups of the 64x64 tiles, tile rows and columns of an XCD's block)"""
    grid, tm, tn = C.c_uint(0), C.c_int(0), C.c_int(0)
    lib.pf_gemm_tile_map(M, N, 64, 64, 0, C.byref(grid), C.byref(tm), C.byref(tn))
    mine = [(tm.value, tn.value) for wg in range(0, grid.value, 8) if lib.pf_gemm_tile_map(M, N, 64, 64, wg, C.byref(grid), C.byref(tm), C.byref(tn))]
    return grid.value, len({t[0] for t in mine}), len({t[1] for t in mine})


@pytest.mark.parametrize("shape", list(READ_AHEAD))
def test_reads_ahead_where_it_was_faster(shape):
    without, with_readers = READ_AHEAD[shape]
    assert (B.load_library().pf_gemm_read_ahead(*shape) > 0) == (with_readers < without)


def test_read_ahead_is_bounded():
    """Over the grids of up to a tile per CU: never more workgroups than CUs, five to eleven readers per XCD (up to twenty only where
    all of the XCD's block stays in 3.5 MB of its L2), and a K tile of the block in two rounds of loads (each reader reads 1 / readers
    of the K tiles, and the launch lasts until it has)."""
    lib, on = B.load_library(), 0
    for tiles_m in range(1, 40):
        for tiles_n in range(1, 256 // tiles_m + 1):
            M, N = 64 * tiles_m - tiles_m % 3, 64 * tiles_n - tiles_n % 5
            grid, rows, cols = _wavek_grid(lib, M, N)
            for K in (1024, 2048, 6144, 2 ** 31 - 64):
                ahead, most = lib.pf_gemm_read_ahead(M, N, K), 20 if (rows + cols) * 64 * K * 2 <= 3.5 * 2 ** 20 else 11
                assert ahead % 8 == 0 and (ahead == 0 or (grid + ahead <= 256 and 5 <= ahead // 8 <= most and rows + cols <= 24))
                on += ahead > 0
    assert on > 2000 and lib.pf_gemm_read_ahead(0, 64, 64) == -6 and lib.pf_gemm_read_ahead(64, 64, 0) == -6


# us from HBM with eleven readers per XCD and with as many as CUs are idle, up to 20: short K, whose block stays in the L2, and long K
@pytest.mark.parametrize("shape,eleven,more", [((64, 6144, 2048), 11.9, 10.8), ((64, 6144, 1536), 11.0, 10.1), ((27, 6144, 2048), 11.0, 10.4),
                                               ((64, 3072, 15360), 43.5, 52.6), ((128, 3072, 15360), 42.1, 53.2), ((320, 1536, 6144), 18.2, 20.1)])
def test_more_readers_where_the_l2_keeps_what_they_read(shape, eleven, more):
    assert (B.load_library().pf_gemm_read_ahead(*shape) > 88) == (more < eleven)
