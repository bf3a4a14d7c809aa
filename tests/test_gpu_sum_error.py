"""FP32 sums of the quarter-size and streaming tiles are no less exact than those of
the larger tiles, whose plans cut the same product's k into more shares.

Both errors are measured against 64 bits on the same inputs.  The rounding errors of
a sum of N terms in blocks of n have a variance that goes with n + N / n; the small
tiles' blocks keep to its least, so their error is at most the other tile's.  The
sample of at least 4096 results fixes each error to 1.1 %, so the ratio may pass 1
by 3 %."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SMALL = {torch.float32: (64, 64, 32), torch.bfloat16: (64, 64, 64), torch.float16: (64, 64, 64)}
LARGE = {torch.float32: (128, 128, 32), torch.bfloat16: (128, 128, 64), torch.float16: (128, 128, 64)}


def sk():
    from paper_2212_08964_amd import skgemm
    return skgemm


def normal(*shape, dtype, scale=1.0):
    return (torch.randn(shape, device="cuda:0") * scale).to(dtype)


def error(C, ref):
    return float((C.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("dtype,M,N,K", [
    (torch.float32, 384, 384, 1024), (torch.float32, 300, 500, 2000), (torch.float32, 512, 512, 512),
    (torch.float32, 256, 1152, 673), (torch.float32, 1219, 146, 128), (torch.float32, 321, 341, 4415),
    (torch.bfloat16, 1024, 1024, 1024), (torch.bfloat16, 640, 1280, 1827), (torch.bfloat16, 768, 910, 1024),
    (torch.float16, 1152, 1036, 979), (torch.float16, 200, 300, 5000), (torch.bfloat16, 300, 200, 128)])
def test_quarter_sums(dtype, M, N, K):
    torch.manual_seed(M + N + K)
    A, B = normal(M, K, dtype=dtype), normal(K, N, dtype=dtype, scale=K ** -0.5)
    ref = A.double() @ B.double()
    small, large = (error(sk().matmul(A, B, out_dtype=torch.float32, tile=t), ref) for t in (SMALL[dtype], LARGE[dtype]))
    auto = error(sk().matmul(A, B, out_dtype=torch.float32), ref)
    assert small <= 1.03 * large and auto <= 1.03 * large, (small, auto, large)


@pytest.mark.parametrize("batch,M,N,K", [(26, 115, 256, 1442), (5, 430, 256, 1179), (12, 195, 278, 1920)])
def test_quarter_sums_batched(batch, M, N, K):
    torch.manual_seed(K)
    A, B = normal(batch, M, K, dtype=torch.bfloat16), normal(batch, K, N, dtype=torch.bfloat16, scale=K ** -0.5)
    ref = torch.stack([a.double() @ b.double() for a, b in zip(A, B)])
    small, large = (error(sk().batched_matmul(A, B, out_dtype=torch.float32, tile=t), ref)
                    for t in (SMALL[torch.bfloat16], LARGE[torch.bfloat16]))
    assert small <= 1.03 * large, (small, large)


@pytest.mark.parametrize("tile", [(32, 32, 256), (64, 32, 256)])
@pytest.mark.parametrize("M,N,K", [(1, 4352, 6784), (2, 4313, 4332), (31, 6746, 4224), (16, 2048, 1024), (8, 1000, 300)])
def test_streaming_sums(tile, M, N, K):
    torch.manual_seed(M + N + K)
    A, B = normal(M, K, dtype=torch.bfloat16), normal(N, K, dtype=torch.bfloat16, scale=K ** -0.5).t()
    ref = A.double() @ B.double()
    small, large = (error(sk().matmul(A, B, out_dtype=torch.float32, tile=t), ref) for t in (tile, (64, 256, 64)))
    assert small <= 1.03 * large, (small, large)
