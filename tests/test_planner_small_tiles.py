"""Where automatic plans take the small tiles (64x64 and 32x256): shapes on both
sides of each limit, measured on both tiles (times in us, small tile / the other).
A plan without a GPU has one co-residency for every tile, so the limits that weigh
tiles against each other are checked with the device's own."""
import os
import subprocess
import sys

import pytest

from paper_2212_08964_amd import calibrate, skgemm as s

QUARTER16, QUARTER32 = (64, 64, 64), (64, 64, 32)


def info(M, N, K, la=0, lb=0, ta=s.BF16, num_cus=256, occupancy=3, tile=None):
    return s.Plan(M, N, K, la, lb, ta=ta, num_cus=num_cus, occupancy=occupancy, tile=tile).info()


def on_device(*args, **kw):
    return info(*args, num_cus=0, occupancy=0, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,la,lb,quarter", [
    (1647, 457, 3961, 0, 0, False),      # rows off 16 bytes, 62 slabs: 28.3 / 21.9
    (2413, 351, 3327, 0, 0, False),      # 52: 25.4 / 21.0
    (256, 4096, 2802, 0, 1, False),      # 44: 21.0 / 18.8
    (640, 1392, 3688, 0, 1, False),      # rows on 16 bytes, 58: 22.9 / 19.1
    (2539, 265, 3032, 0, 1, False),      # 48: 19.9 / 18.1
    (1920, 320, 2944, 0, 0, True),       # rows on 128 bytes, 46: 13.9 / 16.4
    (1792, 384, 3584, 0, 1, True),       # 56: 14.9 / 17.6
    (576, 896, 4032, 0, 0, True),        # 63: 15.2 / 18.1
    (1400, 472, 2040, 0, 1, True),       # rows on 16 bytes, 32 slabs
    (1024, 1024, 1024, 0, 0, True),      # one workgroup per CU
])
def test_quarter_split_limits(M, N, K, la, lb, quarter):
    assert (on_device(M, N, K, la, lb)["tile"][:3] == QUARTER16) == quarter


def test_quarter_split_over_two_per_cu():
    """A split the model would spread over more than two workgroups per CU keeps to
    two, in whole shares a tile; with one share it is data-parallel."""
    i = info(960, 832, 3456)
    assert i["tile"][:3] == QUARTER16 and i["t"] == 195 and i["grid"] == i["g_sk"] == 390
    for M, N, K in [(1856, 320, 1984), (768, 768, 1600), (832, 832, 2048), (1408, 384, 1536)]:
        i = info(M, N, K)
        assert i["tile"][:3] == QUARTER16 and i["grid"] <= 512 and i["g_sk"] % i["t"] == 0, (M, N, K)
    assert info(1647, 457, 3961)["tile"][:3] != QUARTER16 != info(256, 4096, 2802, 0, 1)["tile"][:3]
    # named, the tile keeps the model's own split
    assert info(960, 832, 3456, tile=QUARTER16)["grid"] > 512
    assert info(2145, 158, 5418)["tile"][:3] != QUARTER16           # 85 slabs


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,la,lb,quarter", [
    (384, 384, 1024, 0, 0, True), (300, 500, 2000, 0, 0, True),
    (510, 859, 5621, 0, 0, False),       # 176 slabs over a third of the CUs: 56.0 / 53.3
    (768, 2304, 768, 0, 0, False),       # more than a tile and a half per CU: 34.4 / 34.0
    (512, 2048, 4416, 1, 0, False),      # 1024 workgroups of 138 slabs: 87.9 / 81.2
    (369, 2405, 3279, 1, 0, False),      # 912 of 103: 68.4 / 63.4
    (3008, 192, 3840, 1, 1, True),       # a quarter of the 128x128 tiles is padding: 47.5 / 60.8
])
def test_quarter_fp32_limits(M, N, K, la, lb, quarter):
    assert (on_device(M, N, K, la, lb, ta=s.F32)["tile"][:3] == QUARTER32) == quarter


@pytest.mark.parametrize("M,N,K,stream", [
    (1, 32000, 4096, False),      # 1000 tiles of 16 slabs: 49.3 / 45.4
    (16, 50304, 2048, False),     # 1572 of 8: 51.2 / 33.2
    (16, 128256, 5120, False),    # 4008 of 20, sixteen waves: 262.8 / 218.7
    (1, 28672, 3072, False),      # 896 of 12: 36.9 / 32.3
    (22, 17088, 4991, False),     # 534 of 20, a short third wave: 1.17x
    (3, 17280, 6403, False),      # 540 of 26, the same: 1.10x
    (1, 9249, 1214, False),       # rows off 8 bytes
    (1, 50304, 8192, True),       # 32 slabs, seven waves: 151.6 / 189.7
    (16, 128256, 8192, True),     # sixteen: 348.6 / 407.0
    (1, 32000, 5120, True),       # 20 slabs, last wave nearly full: 60.4 / 67.3
    (1, 50304, 5120, True),       # seven waves: 107.2 / 115.3
    (1, 16384, 4096, True),       # two full waves: 25.7 / 26.4
    (4, 9983, 9984, True),        # more than 32 slabs
    (16, 8192, 300, True),        # one wave
])
def test_streaming_waves(M, N, K, stream):
    """Above one streaming tile per CU the number of slabs and the fill of the last
    wave decide."""
    i = info(M, N, K, 0, 1, occupancy=2)
    assert (i["tile"][:3] == (32, 32, 256)) == stream


@pytest.mark.parametrize("K,stream", [(4096, True), (8192, True), (8256, False), (11840, False)])
def test_streaming_64_rows(K, stream):
    """33 to 64 rows: up to 32 slabs (49x5120x11840: 40.2 / 33.0)."""
    assert (info(49, 5120, K, 0, 1, occupancy=2)["tile"][:3] == (64, 32, 256)) == stream


@pytest.mark.parametrize("M,N,K,tile", [
    (64, 704, 64, None), (64, 1230, 64, None), (33, 900, 128, None), (64, 900, 192, None),      # 1.06-1.21x
    (64, 900, 256, (64, 32, 256)), (40, 5000, 448, (64, 32, 256)),
    (32, 900, 64, None), (9, 900, 128, None), (9, 900, 129, (32, 32, 256)), (32, 3000, 200, (32, 32, 256)),
    (8, 900, 64, None), (1, 900, 3, None), (8, 900, 65, (32, 32, 256)), (1, 3000, 96, (32, 32, 256)),
    (8, 900, 0, None)])
def test_streaming_short_k(M, N, K, tile):
    """A small part of a slab: the other tiles, in either role of the small operand."""
    stream = [(32, 32, 256), (64, 32, 256)]
    for i in (info(M, N, K, 0, 1, occupancy=2), s.Plan(N, M, K, 0, 1, lc=1, ta=s.BF16, num_cus=256, occupancy=2).info()):
        assert i["tile"][:3] == tile if tile else i["tile"][:3] not in stream


@pytest.mark.gpu
@pytest.mark.parametrize("ta,tile", [(s.BF16, QUARTER16), (s.F32, QUARTER32)])
def test_quarter_integer_shapes_take_the_tile(ta, tile):
    """The shapes whose automatic products, single and batched by three, are compared
    bit by bit with the oracle as this tile's."""
    for M, N, K in [(500, 300, 1000), (130, 131, 77)]:
        assert on_device(M, N, K, 0, 1, ta=ta)["tile"][:3] == tile
        assert s.BatchedPlan(3, M, N, K, 0, 1, 0, ta, s.F32).info()["tile"][:3] == tile


@pytest.mark.parametrize("tile", calibrate.SMALL_TILES)
@pytest.mark.parametrize("M,N,K", [(32, 4096, 4096), (30, 1000, 333), (500, 300, 1000), (1024, 1024, 1024), (64, 9000, 2500),
                                   (700, 900, 8192)])
def test_calibration_terms(tile, M, N, K):
    """calibrate.estimate_terms and the plan's constants give the planner's own
    estimate (which its log prints, or its HBM bound where that is larger)."""
    code = ("from paper_2212_08964_amd import skgemm as s, calibrate as c\n"
            f"p = s.Plan({M}, {N}, {K}, lb=s.COL_MAJOR, ta=s.BF16, num_cus=256, occupancy=3, tile={tile})\n"
            "print(sum(x * y for x, y in zip(c.estimate_terms(p.info()), p.model_constants())))")
    out = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, SKGEMM_LOG="1"), capture_output=True, text=True,
                         cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), timeout=120)
    assert out.returncode == 0, out.stderr
    logged = float(out.stderr.split("est_us=")[1].split()[0])
    i = info(M, N, K, 0, 1, tile=tile)
    hbm = 2.0 * (M * K + N * K + M * N) / 6.0e6
    partials = 2.0 * 4 * i["BM"] * i["BN"] * (i["g_sk"] - i["sk_tiles"]) / 6.0e6 if i["g_sk"] else 0.0
    assert logged == pytest.approx(max(float(out.stdout), hbm + partials), abs=0.02)
