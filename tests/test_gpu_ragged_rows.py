"""The kernels for operands whose rows do not start on 16 bytes (the eight-wave
128x128 16-bit tile with more than 16 slabs a workgroup, the small FP8 tile): odd
leading dimensions, aligned ones from a misaligned base, NaN in the gaps, every
layout, edges of the tile and its slabs, batches with odd strides, every schedule,
with and without a trace.

Integer inputs of at most 2 in magnitude are exact in FP32 sums of these lengths, so
results are compared bit by bit with the FP64 product."""
import itertools

import pytest
import torch

from helpers import oracle_plan_for, records_to_schedule
from oracle import schedule as S

pytestmark = pytest.mark.gpu

TILE16, TILE8 = (128, 128, 64, 8), (128, 128, 128)
E4M3 = torch.float8_e4m3fn


def sk():
    from paper_2212_08964_amd import skgemm
    return skgemm


def operand(rows, cols, col_major, dtype, seed, pad, shift, batch=None):
    """Integers in [-2, 2]; lines `pad` elements apart (NaN between), `shift` elements
    past a 256-byte boundary; batches one element more apart."""
    r, c = (cols, rows) if col_major else (rows, cols)
    n, one = batch or 1, r * (c + pad) + 1
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    buf = torch.full((n * one + shift,), float("nan"), device="cuda:0").to(dtype)
    out = buf[shift:shift + n * one].view(n, one)[:, :r * (c + pad)].view(n, r, c + pad)[:, :, :c]
    out.copy_(torch.randint(-2, 3, (n, r, c), generator=g, device="cuda:0").to(torch.float32).to(dtype))
    out = out.transpose(1, 2) if col_major else out
    return out if batch else out[0]


def product(A, B):
    return (A.float().double() @ B.float().double()).float()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("pad,shift", [(0, 0), (3, 0), (0, 1), (5, 7)])
@pytest.mark.parametrize("M,N,K", [(2177, 2049, 1091), (2176, 2048, 1152), (2049, 2300, 1089), (1100, 4000, 1500)])
def test_ragged_16(dtype, pad, shift, M, N, K):
    for ca, cb in itertools.product([False, True], repeat=2):
        A = operand(M, K, ca, dtype, M + K, pad, 0)
        B = operand(K, N, cb, dtype, N + K, pad, shift)
        ref = product(A, B)
        # (more workgroups than CUs: fewer run the three-stage tile)
        for pol, fg in (("auto", 0), ("dp", 0), ("sk", 0), ("sk", 301), ("dp_1tile_sk", 0)):
            C = sk().matmul(A, B, policy=pol, force_g=fg, tile=TILE16, out_dtype=torch.float32)
            assert torch.equal(C, ref), (ca, cb, pol, fg)
        C = sk().matmul(A, B, policy="dp", tile=TILE16)
        assert torch.equal(C, ref.to(dtype)), (ca, cb)


@pytest.mark.parametrize("pad,shift", [(0, 0), (3, 0), (0, 1), (0, 8)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (127, 129, 31), (128, 128, 128), (300, 257, 130), (129, 300, 1001), (200, 390, 3000)])
def test_ragged_fp8(pad, shift, M, N, K):
    A, B = operand(M, K, False, E4M3, M + K, pad, shift), operand(K, N, True, E4M3, N + K, pad, 0)
    ref = product(A, B)
    one, two = torch.tensor([1.0], device="cuda:0"), torch.tensor([2.0], device="cuda:0")
    for pol, fg in (("auto", 0), ("dp", 0), ("sk", 0), ("sk", 5), ("dp_1tile_sk", 0)):
        assert torch.equal(sk().matmul(A, B, policy=pol, force_g=fg, tile=TILE8), ref), (pol, fg)
    assert torch.equal(sk().matmul(A, B, tile=TILE8, scale_a=one, scale_b=two, out_dtype=torch.bfloat16),
                       (2 * ref).to(torch.bfloat16))


@pytest.mark.parametrize("cb", [False, True])
def test_ragged_batches(cb):
    A, B = operand(130, 1200, False, torch.bfloat16, 1, 0, 0, 70), operand(1200, 136, cb, torch.bfloat16, 2, 0, 0, 70)
    assert B.stride(0) % 8                       # rows on 16 bytes, matrices not
    C = sk().batched_matmul(A, B, out_dtype=torch.float32, tile=TILE16)
    assert torch.equal(C, torch.stack([product(a, b) for a, b in zip(A, B)]))
    A, B = operand(140, 256, False, E4M3, 1, 0, 0, 3), operand(256, 136, True, E4M3, 2, 0, 0, 3)
    C = sk().batched_matmul(A, B, tile=TILE8)
    assert torch.equal(C, torch.stack([product(a, b) for a, b in zip(A, B)]))


@pytest.mark.parametrize("kind", ["16", "fp8"])
def test_ragged_trace(kind):
    """The trace equals the enumerator's schedule."""
    dtype, code, tile, cb = ((torch.bfloat16, sk().BF16, TILE16, False), (E4M3, sk().F8E4M3, TILE8, True))[kind == "fp8"]
    M, N, K = ((2100, 2200, 1091), (300, 260, 2051))[kind == "fp8"]
    A, B = operand(M, K, False, dtype, 3, 0, 0), operand(K, N, cb, dtype, 4, 0, 0)
    for pol, fg in (("dp", 0), ("sk", 300 if kind == "16" else 7), ("sk", 0), ("dp_1tile_sk", 0)):
        plan = sk().get_plan(M, N, K, 0, int(cb), 0, code, sk().F32, pol, fg, 2, tile)
        info = plan.info()
        tr = torch.full((plan.trace_capacity() * 8,), -7, dtype=torch.int32, device="cuda:0")
        C = sk().matmul(A, B, out_dtype=torch.float32, policy=pol, force_g=fg, tile=tile, trace=tr)
        assert torch.equal(C, product(A, B)), (pol, fg)
        recs = [tuple(int(v) for v in r) for r in tr.cpu().numpy().reshape(-1, 8) if r[0] != -7]
        o = oracle_plan_for(info, plan.model_constants(), info["policy_name"], force_g=info["g_sk"])
        assert records_to_schedule(recs, info["grid"]) == S.enumerate_schedule(o), (pol, fg)
