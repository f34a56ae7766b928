"""The GEMMs' tile rules and the banded tile walk (CPU, host-only queries).

The bf16 rule against measured launches: for shapes at the edges of its rounds - few rows
at wide outputs, one round and a little more, grids that an XCD's block of whole rows and columns pads - the tile it picks is
within an eighth of the fastest.  us per launch, plain store, isolated GEMMs with cold weights on an MI355X."""
import ctypes as C

import pytest

from paper_2405_14430_amd import binding as B

MEASURED = {
    (5362, 2048, 8192): {"<256,256,2,4,2,false>": 188.6, "<256,192,2,4,2,false>": 282.4, "<256,128,3,4,2,false>": 214.5, "<128,192,2,2,2,false>": 177.9, "<128,192,3,2,2,true>": 182.1, "<128,128,2,2,2,false>": 192.6, "<128,64,2,2,2,false>": 222.9, "<64,128,3,2,2,false>": 233.8},
    (10751, 1536, 7680): {"<256,256,2,4,2,false>": 340.0, "<256,192,2,4,2,false>": 287.9, "<256,128,3,4,2,false>": 310.3, "<128,192,2,2,2,false>": 247.4, "<128,192,3,2,2,true>": 249.3, "<128,128,2,2,2,false>": 295.4, "<128,64,2,2,2,false>": 326.9, "<64,128,3,2,2,false>": 344.4},
    (9409, 9216, 3072): {"<256,256,2,4,2,false>": 483.2, "<256,192,2,4,2,false>": 510.4, "<256,128,3,4,2,false>": 520.4, "<128,192,2,2,2,false>": 485.8, "<128,192,3,2,2,true>": 525.9, "<128,128,2,2,2,false>": 517.5, "<128,64,2,2,2,false>": 644.1, "<64,128,3,2,2,false>": 677.7},
    (431, 9216, 3072): {"<256,256,2,4,2,false>": 72.8, "<256,192,2,4,2,false>": 62.6, "<256,128,3,4,2,false>": 42.3, "<128,192,2,2,2,false>": 50.9, "<128,192,3,2,2,true>": 38.8, "<128,128,2,2,2,false>": 44.4, "<128,64,2,2,2,false>": 45.0, "<64,128,3,2,2,false>": 42.1},
    (512, 9216, 3072): {"<256,256,2,4,2,false>": 76.4, "<256,192,2,4,2,false>": 68.8, "<256,128,3,4,2,false>": 44.9, "<128,192,2,2,2,false>": 52.1, "<128,192,3,2,2,true>": 41.3, "<128,128,2,2,2,false>": 45.8, "<128,64,2,2,2,false>": 48.2, "<64,128,3,2,2,false>": 56.6},
    (5263, 1536, 1536): {"<256,256,2,4,2,false>": 39.8, "<256,192,2,4,2,false>": 32.4, "<256,128,3,4,2,false>": 48.1, "<128,192,2,2,2,false>": 34.9, "<128,192,3,2,2,true>": 39.7, "<128,128,2,2,2,false>": 44.3, "<128,64,2,2,2,false>": 39.8, "<64,128,3,2,2,false>": 36.9},
    (8283, 576, 2304): {"<256,256,2,4,2,false>": 53.1, "<256,192,2,4,2,false>": 41.7, "<256,128,3,4,2,false>": 34.0, "<128,192,2,2,2,false>": 33.1, "<128,192,3,2,2,true>": 28.7, "<128,128,2,2,2,false>": 30.9, "<128,64,2,2,2,false>": 33.9, "<64,128,3,2,2,false>": 38.9},
    (680, 6144, 1536): {"<256,256,2,4,2,false>": 42.5, "<256,192,2,4,2,false>": 37.1, "<256,128,3,4,2,false>": 24.8, "<128,192,2,2,2,false>": 29.1, "<128,192,3,2,2,true>": 22.9, "<128,128,2,2,2,false>": 25.2, "<128,64,2,2,2,false>": 26.4, "<64,128,3,2,2,false>": 30.8},
    (1038, 4608, 1152): {"<256,256,2,4,2,false>": 32.5, "<256,192,2,4,2,false>": 25.7, "<256,128,3,4,2,false>": 20.3, "<128,192,2,2,2,false>": 22.0, "<128,192,3,2,2,true>": 18.2, "<128,128,2,2,2,false>": 20.3, "<128,64,2,2,2,false>": 20.7, "<64,128,3,2,2,false>": 23.8},
    (7456, 768, 3840): {"<256,256,2,4,2,false>": 81.1, "<256,192,2,4,2,false>": 64.1, "<256,128,3,4,2,false>": 51.9, "<128,192,2,2,2,false>": 52.1, "<128,192,3,2,2,true>": 46.5, "<128,128,2,2,2,false>": 50.5, "<128,64,2,2,2,false>": 60.1, "<64,128,3,2,2,false>": 63.6},
    (2048, 9216, 3072): {"<256,256,2,4,2,false>": 153.0, "<256,192,2,4,2,false>": 129.7, "<256,128,3,4,2,false>": 136.9, "<128,192,2,2,2,false>": 117.1, "<128,192,3,2,2,true>": 120.4, "<128,128,2,2,2,false>": 130.9, "<128,64,2,2,2,false>": 150.3, "<64,128,3,2,2,false>": 163.8},
    (2560, 9216, 3072): {"<256,256,2,4,2,false>": 154.3, "<256,192,2,4,2,false>": 140.0, "<256,128,3,4,2,false>": 149.9, "<128,192,2,2,2,false>": 141.5, "<128,192,3,2,2,true>": 157.1, "<128,128,2,2,2,false>": 143.6, "<128,64,2,2,2,false>": 191.7, "<64,128,3,2,2,false>": 202.0},
    (16896, 9216, 3072): {"<256,256,2,4,2,false>": 850.0, "<256,192,2,4,2,false>": 916.2, "<256,128,3,4,2,false>": 967.2, "<128,192,2,2,2,false>": 881.2, "<128,192,3,2,2,true>": 989.4, "<128,128,2,2,2,false>": 944.0, "<128,64,2,2,2,false>": 1178.5, "<64,128,3,2,2,false>": 1215.3},
    (4096, 3456, 1152): {"<256,256,2,4,2,false>": 37.4, "<256,192,2,4,2,false>": 51.7, "<256,128,3,4,2,false>": 41.5, "<128,192,2,2,2,false>": 45.4, "<128,192,3,2,2,true>": 54.4, "<128,128,2,2,2,false>": 41.1, "<128,64,2,2,2,false>": 48.3, "<64,128,3,2,2,false>": 49.6},
    (3677, 8192, 2048): {"<256,256,2,4,2,false>": 116.7, "<256,192,2,4,2,false>": 130.7, "<256,128,3,4,2,false>": 138.0, "<128,192,2,2,2,false>": 131.0, "<128,192,3,2,2,true>": 150.2, "<128,128,2,2,2,false>": 128.1, "<128,64,2,2,2,false>": 159.4, "<64,128,3,2,2,false>": 165.9},
    (1024, 4608, 1536): {"<256,256,2,4,2,false>": 43.2, "<256,192,2,4,2,false>": 39.0, "<256,128,3,4,2,false>": 26.2, "<128,192,2,2,2,false>": 30.3, "<128,192,3,2,2,true>": 24.4, "<128,128,2,2,2,false>": 26.5, "<128,64,2,2,2,false>": 27.0, "<64,128,3,2,2,false>": 31.7},
    # fewer tiles, where the rule does not look at the epilogue: 430 to 528 tiles of 64x64, with a residual
    (633, 3072, 15360): {"gemm_wavek_kernel<64,64>": 106.8, "<64,64,4,2,2,false>": 120.1, "<64,128,3,2,2,false>": 119.1, "<64,64,2,2,2,false>": 162.9, "<128,64,2,2,2,false>": 177.2},
    (633, 3072, 12288): {"gemm_wavek_kernel<64,64>": 79.9, "<64,64,4,2,2,false>": 96.7, "<64,128,3,2,2,false>": 93.8, "<64,64,2,2,2,false>": 126.9, "<128,64,2,2,2,false>": 139.2},
    (569, 3072, 15360): {"gemm_wavek_kernel<64,64>": 103.0, "<64,64,4,2,2,false>": 93.7, "<64,128,3,2,2,false>": 115.2, "<64,64,2,2,2,false>": 161.6, "<128,64,2,2,2,false>": 175.8},
    (1275, 1536, 6144): {"gemm_wavek_kernel<64,64>": 46.0, "<64,64,4,2,2,false>": 50.5, "<64,128,3,2,2,false>": 51.7, "<64,64,2,2,2,false>": 67.1, "<128,64,2,2,2,false>": 74.2},
    (1339, 1536, 6144): {"gemm_wavek_kernel<64,64>": 64.0, "<64,64,4,2,2,false>": 65.3, "<64,128,3,2,2,false>": 53.6, "<64,64,2,2,2,false>": 66.9, "<128,64,2,2,2,false>": 74.4},
    (1211, 1536, 6144): {"gemm_wavek_kernel<64,64>": 45.7, "<64,64,4,2,2,false>": 43.1, "<64,128,3,2,2,false>": 51.1, "<64,64,2,2,2,false>": 67.0, "<128,64,2,2,2,false>": 74.3},
    (765, 2560, 10240): {"gemm_wavek_kernel<64,64>": 74.5, "<64,64,4,2,2,false>": 84.7, "<64,128,3,2,2,false>": 83.6, "<64,64,2,2,2,false>": 108.6, "<128,64,2,2,2,false>": 119.4},
    (1021, 2048, 8192): {"gemm_wavek_kernel<64,64>": 57.5, "<64,64,4,2,2,false>": 63.8, "<64,128,3,2,2,false>": 67.4, "<64,64,2,2,2,false>": 85.6, "<128,64,2,2,2,false>": 93.5},
    (1527, 1152, 4608): {"gemm_wavek_kernel<64,64>": 34.7, "<64,64,4,2,2,false>": 30.9, "<64,128,3,2,2,false>": 39.1, "<64,64,2,2,2,false>": 50.8, "<128,64,2,2,2,false>": 56.6},
    (1783, 1152, 4608): {"gemm_wavek_kernel<64,64>": 36.8, "<64,64,4,2,2,false>": 39.4, "<64,128,3,2,2,false>": 41.7, "<64,64,2,2,2,false>": 51.4, "<128,64,2,2,2,false>": 58.0},
    (1275, 1536, 1536): {"gemm_wavek_kernel<64,64>": 17.5, "<64,64,4,2,2,false>": 14.9, "<64,128,3,2,2,false>": 17.8, "<64,64,2,2,2,false>": 16.6, "<128,64,2,2,2,false>": 19.2},
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
