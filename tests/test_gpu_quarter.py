"""The quarter-size tiles (64x64x64 for 16-bit types, 64x64x32 for FP32) against
the float64 oracle: parity at the edges of the tile and of its k-slabs in every
layout, integer inputs bit-exact under every schedule, padded leading dimensions
with NaN in the gaps, batches, the schedule trace, and the rule that picks them.

Tolerances as for the other tiles of these types: K products added in FP32, so
1e-5 relative Frobenius error with FP32 output (2e-5 for FP32 inputs); one
rounding to the output type (2^-8 for bfloat16) more with 16-bit output, 1e-2."""
import itertools

import numpy as np
import pytest
import torch

import workloads as W
from helpers import oracle_plan_for, records_to_schedule, to_f64
from oracle import gemm as og
from oracle import schedule as S

TILES = {torch.bfloat16: (64, 64, 64), torch.float16: (64, 64, 64), torch.float32: (64, 64, 32)}


def sk():
    from paper_2212_08964_amd import skgemm
    return skgemm


def dev():
    return torch.device("cuda:0")


def operand(rows, cols, col_major, dtype, seed, integer=False, pad=0):
    """rows x cols in the given order, lines `pad` elements apart (NaN in the gap)."""
    r, c = (cols, rows) if col_major else (rows, cols)
    make = W.integer_f32 if integer else W.normal_f32
    buf = torch.full((r, c + pad), float("nan"), dtype=dtype, device=dev())
    buf[:, :c] = torch.from_numpy(make(W.rng(seed), (r, c))).to(dtype).to(dev())
    return buf[:, :c].t() if col_major else buf[:, :c]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", list(TILES))
@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 65, 31), (64, 64, 64), (65, 63, 33), (129, 190, 65), (100, 300, 1000),
                                   (512, 512, 96), (257, 1023, 2049)])
def test_quarter_parity(dtype, pad, shape):
    M, N, K = shape
    for ca, cb in itertools.product([False, True], repeat=2):
        A = operand(M, K, ca, dtype, M + K, pad=pad)
        B = operand(K, N, cb, dtype, N + K + 1, pad=pad)
        ref = og.gemm_f64(to_f64(A), to_f64(B))
        for pol in ("auto", "dp", "sk"):
            C = sk().matmul(A, B, policy=pol, out_dtype=torch.float32, tile=TILES[dtype])
            torch.cuda.synchronize()
            assert og.rel_frobenius(to_f64(C), ref) <= (2e-5 if dtype == torch.float32 else 1e-5), (ca, cb, pol)
            if dtype != torch.float32:
                C = sk().matmul(A, B, policy=pol, tile=TILES[dtype])
                torch.cuda.synchronize()
                assert og.rel_frobenius(to_f64(C), ref) <= 1e-2, (ca, cb, pol)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_quarter_integer_exact_every_schedule_and_trace(dtype):
    """Integer inputs are exact under every schedule, beta included; the trace
    equals the enumerator's schedule."""
    M, N, K = 300, 200, 700
    code = {torch.bfloat16: sk().BF16, torch.float32: sk().F32}[dtype]
    for ca, cb in [(False, False), (True, True)]:
        A, B = operand(M, K, ca, dtype, 3, integer=True), operand(K, N, cb, dtype, 4, integer=True)
        ref = og.gemm_f64(to_f64(A), to_f64(B))
        for pol in ["auto", "paper", "dp", "sk", "dp_1tile_sk", "2tile_sk_dp"]:
            for fg in ([0] if pol != "sk" else [0, 1, 7, 41, 100]):
                plan = sk().get_plan(M, N, K, int(ca), int(cb), 0, code, sk().F32, pol, fg, 2, TILES[dtype])
                info = plan.info()
                assert info["tile"][:3] == TILES[dtype]
                tr = torch.full((plan.trace_capacity() * 8,), -7, dtype=torch.int32, device=dev())
                C = torch.ones((M, N), dtype=torch.float32, device=dev())
                sk().matmul(A, B, out=C, beta=2.0, policy=pol, force_g=fg, tile=TILES[dtype], trace=tr)
                torch.cuda.synchronize()
                assert np.array_equal(to_f64(C), ref + 2.0), (pol, fg)
                recs = [tuple(int(v) for v in r) for r in tr.cpu().numpy().reshape(-1, 8) if r[0] != -7]
                o = oracle_plan_for(info, plan.model_constants(), info["policy_name"], force_g=info["g_sk"])
                assert records_to_schedule(recs, info["grid"]) == S.enumerate_schedule(o), (pol, fg)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_quarter_automatic_and_batched(dtype):
    """Automatic plans that take the tile, single and batched, integer exact."""
    for M, N, K in [(500, 300, 1000), (130, 131, 77)]:
        A, B = operand(M, K, False, dtype, 5, integer=True), operand(K, N, True, dtype, 6, integer=True)
        C = sk().matmul(A, B, out_dtype=torch.float32)
        Ab, Bb = torch.stack([A, -A, A + 1]), torch.stack([B, B, 2 - B])
        Cb = sk().batched_matmul(Ab, Bb, out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert np.array_equal(to_f64(C), og.gemm_f64(to_f64(A), to_f64(B)))
        for i in range(3):
            assert np.array_equal(to_f64(Cb[i]), og.gemm_f64(to_f64(Ab[i]), to_f64(Bb[i])))


def test_quarter_rule():
    """Automatic plans of small problems take the quarter-size tiles; not with 64
    rows or columns or more than two tiles per CU (16-bit types), other policies,
    options, types or groups, nor for a tile named in part."""
    s = sk()
    kw = dict(num_cus=256, occupancy=2)

    def tile(M, N, K, ta=s.BF16, **k):
        return s.Plan(M, N, K, ta=ta, **{**kw, **k}).info()["tile"][:3]

    for M, N, K in [(1024, 1024, 1024), (512, 512, 512), (200, 300, 700)]:
        assert tile(M, N, K) == tile(M, N, K, ta=s.F16) == (64, 64, 64)
    assert tile(384, 384, 1024, ta=s.F32) == tile(141, 574, 128, ta=s.F32) == (64, 64, 32)
    for M, N, K in [(64, 1000, 1000), (1000, 64, 1000), (2048, 2048, 512), (1536, 1536, 512), (8192, 8192, 8192)]:
        assert tile(M, N, K) != (64, 64, 64), (M, N, K)
    for k in [dict(policy="dp"), dict(policy="sk"), dict(force_g=7), dict(tile=(0, 0, 0, 4)), dict(tile=(0, 0, 0, 8)),
              dict(tile=(128, 128, 64)), dict(tile=(64, 0, 0)), dict(tile=(0, 0, 64))]:
        assert tile(1024, 1024, 1024, **k) != (64, 64, 64), k
    assert s.GroupedPlan([512], [512], [512], ta=s.BF16, **kw).info()["tile"][:3] != (64, 64, 64)
    for ta, t in [(s.F64, (64, 64, 64)), (s.F32, (64, 64, 64)), (s.BF16, (64, 64, 32))]:
        with pytest.raises(s.SkgemmError) as e:
            tile(512, 512, 512, ta=ta, tile=t)
        assert e.value.status == s.ERR_UNSUPPORTED


@pytest.mark.parametrize("M,N,K,large", [(2556, 1675, 2416, True), (2556, 1675, 2432, False), (1297, 3957, 3360, True),
                                         (512, 2000, 3001, False), (192, 1136, 5059, False)])
def test_small_fp8_tile_rule(M, N, K, large):
    """Automatic FP8 plans weigh the small tile's misaligned runs where K is not a
    multiple of 128; with whole lines, and for small products, it stays."""
    s = sk()
    kw = dict(lb=s.COL_MAJOR, ta=s.F8E4M3, tc=s.BF16, num_cus=256, occupancy=2)
    assert (s.Plan(M, N, K, **kw).info()["tile"][:3] == (256, 256, 128)) == large
    assert s.Plan(M, N, K, **kw, tile=(128, 128, 128)).info()["tile"][:3] == (128, 128, 128)
