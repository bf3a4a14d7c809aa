"""The streaming 16-bit tiles (32x32x256 and 64x32x256: few rows, both operands
K-contiguous) against the float64 oracle: parity at the edges of the tile and of
its k-slabs, integer inputs bit-exact under every schedule, padded leading
dimensions with NaN in the gaps, the schedule trace, and the rule that picks
the tiles.

Tolerances as for the other 16-bit tiles: the products are exact in FP32 and K
of them are added in FP32, so 1e-5 relative Frobenius error with FP32 output;
one rounding to the output type (2^-8 for bfloat16) more, so 1e-2, with 16-bit
output."""
import numpy as np
import pytest
import torch

import workloads as W
from helpers import oracle_plan_for, records_to_schedule, to_f64
from oracle import gemm as og
from oracle import schedule as S

TILES = [(32, 32, 256), (64, 32, 256)]


def sk():
    from paper_2212_08964_amd import skgemm
    return skgemm


def dev():
    return torch.device("cuda:0")


def operands(M, N, K, dtype, seed, integer=False, pad=0):
    """A (M x K) row-major and B (K x N) column-major, rows `pad` elements apart
    (NaN in the gap)."""
    g = W.rng(seed)
    make = W.integer_f32 if integer else W.normal_f32
    out = []
    for rows in (M, N):
        buf = torch.full((rows, K + pad), float("nan"), dtype=dtype, device=dev())
        buf[:, :K] = torch.from_numpy(make(g, (rows, K))).to(dtype).to(dev())
        out.append(buf[:, :K])
    return out[0], out[1].t()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 33, 255), (16, 4096, 2048), (31, 257, 256), (32, 32, 257), (7, 100, 8),
                                   (33, 31, 1000), (64, 1000, 4096), (63, 2049, 777), (20, 40, 8192)])
def test_stream_parity(dtype, pad, shape):
    M, N, K = shape
    A, B = operands(M, N, K, dtype, M + N + K, pad=pad)
    ref = og.gemm_f64(to_f64(A), to_f64(B))
    for tile in ([None] + TILES) if M <= 32 else [None, TILES[1]]:
        for pol in ("auto", "dp", "sk"):
            C32 = sk().matmul(A, B, policy=pol, out_dtype=torch.float32, tile=tile)
            C16 = sk().matmul(A, B, policy=pol, tile=tile)
            torch.cuda.synchronize()
            assert og.rel_frobenius(to_f64(C32), ref) <= 1e-5, (tile, pol)
            assert og.rel_frobenius(to_f64(C16), ref) <= 1e-2, (tile, pol)


@pytest.mark.gpu
@pytest.mark.parametrize("tile", TILES)
def test_stream_integer_exact_every_schedule_and_trace(tile):
    """Integer inputs are exact under every schedule, rows above the tile's
    height and beta included; the trace equals the enumerator's schedule."""
    M, N, K = 100, 700, 3000
    A, B = operands(M, N, K, torch.bfloat16, 3, integer=True)
    ref = og.gemm_f64(to_f64(A), to_f64(B))
    for pol in ["auto", "paper", "dp", "sk", "dp_1tile_sk", "2tile_sk_dp"]:
        for fg in ([0] if pol != "sk" else [0, 1, 5, 47, 176, 200]):
            plan = sk().get_plan(M, N, K, 0, 1, 0, sk().BF16, sk().F32, pol, fg, 2, tile)
            info = plan.info()
            assert info["tile"][:3] == tile and info["occupancy"] == 1
            tr = torch.full((plan.trace_capacity() * 8,), -7, dtype=torch.int32, device=dev())
            C = torch.ones((M, N), dtype=torch.float32, device=dev())
            sk().matmul(A, B, out=C, beta=2.0, policy=pol, force_g=fg, tile=tile, trace=tr)
            torch.cuda.synchronize()
            assert np.array_equal(to_f64(C), ref + 2.0), (pol, fg)
            recs = [tuple(int(v) for v in r) for r in tr.cpu().numpy().reshape(-1, 8) if r[0] != -7]
            o = oracle_plan_for(info, plan.model_constants(), info["policy_name"], force_g=info["g_sk"])
            assert records_to_schedule(recs, info["grid"]) == S.enumerate_schedule(o), (pol, fg)
            C2 = sk().matmul(A, B, out_dtype=torch.float32, policy=pol, force_g=fg, tile=tile)
            torch.cuda.synchronize()
            assert np.array_equal(to_f64(C2), ref), (pol, fg)


def test_stream_rule():
    """Automatic plans take the streaming tiles exactly where the rule says:
    both operands K-contiguous, at most 32 rows (but for a short last wave of
    short tiles), or at most 64 with rows on 128-byte lines and at most one tile
    per CU; never for other policies, layouts, types, batches or groups, nor
    where the options ask for another tile or for eight waves."""
    s = sk()
    kw = dict(num_cus=256, occupancy=2)

    def tile(M, N, K, lb=s.COL_MAJOR, ta=s.BF16, **k):
        return s.Plan(M, N, K, lb=lb, ta=ta, **{**kw, **k}).info()["tile"][:3]

    for ta in (s.BF16, s.F16):
        for M, N, K in [(1, 1, 1), (32, 8192, 8192)]:
            assert tile(M, N, K, ta=ta) == TILES[0]
        assert tile(33, 8192, 4096, ta=ta) == tile(64, 100, 64, ta=ta) == TILES[1]
        for M, N, K in [(64, 8193, 4096), (33, 4096, 4100), (65, 4096, 4096), (16, 10000, 1000), (16, 20000, 333)]:
            assert tile(M, N, K, ta=ta) not in TILES
    assert tile(8192, 16, 4096, la=s.ROW_MAJOR, lc=s.COL_MAJOR) == TILES[0]      # 16 rows as launched
    for k in [dict(lb=s.ROW_MAJOR), dict(la=s.COL_MAJOR), dict(policy="dp"), dict(policy="sk"), dict(ta=s.F32),
              dict(tile=(128, 128, 64)), dict(policy="auto", force_g=7), dict(tile=(0, 0, 0, 8))]:
        assert tile(16, 4096, 4096, **k) not in TILES, k
    assert s.BatchedPlan(4, 16, 4096, 4096, lb=s.COL_MAJOR, ta=s.BF16, **kw).info()["tile"][:3] not in TILES
    assert s.GroupedPlan([16], [4096], [4096], lb=s.COL_MAJOR, ta=s.BF16, **kw).info()["tile"][:3] not in TILES
    for t in TILES:          # no kernel reads an MN-contiguous operand
        with pytest.raises(s.SkgemmError) as e:
            tile(16, 4096, 4096, lb=s.ROW_MAJOR, tile=t)
        assert e.value.status == s.ERR_UNSUPPORTED


@pytest.mark.parametrize("M,N,K,stream", [(24, 17000, 2176, False), (1, 8700, 2176, False), (24, 17000, 2048, True),
                                          (1, 8192, 2176, True), (24, 17000, 4096, True), (1, 9663, 2900, True)])
def test_stream_rule_padded_last_slab(M, N, K, stream):
    """Above one tile per CU, short tiles whose last slab is mostly padding stay
    on the other tiles."""
    s = sk()
    p = s.Plan(M, N, K, lb=s.COL_MAJOR, ta=s.BF16, num_cus=256, occupancy=2)
    assert (p.info()["tile"][:3] in TILES) == stream
