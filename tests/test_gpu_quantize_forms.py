"""The quantiser's routes: matrices without gaps (any length, as one row), padded
rows, misaligned starts, both orders, more work than one sweep of the grid.

The scale is absmax / 448 in FP32 and the codes are the correctly rounded E4M3
values of x / s, so both are compared exactly with the quotient rounded on the
CPU."""
import pytest
import torch

E4M3 = torch.float8_e4m3fn


def sk():
    from paper_2212_08964_amd import skgemm
    return skgemm


def reference(x):
    """(codes, scale) of a CPU tensor, in FP32 throughout."""
    v = x.float()
    fin = torch.where(torch.isfinite(v), v.abs(), torch.zeros_like(v))
    m = fin.max() if v.numel() else torch.tensor(0.0)
    s = torch.tensor(1.0) if m == 0 else m / torch.tensor(448.0)
    return torch.clamp(v / s, -448.0, 448.0).to(E4M3), s


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("shape", [(1, 1), (1, 15), (1, 17), (3, 5), (16, 16), (33, 257), (64, 4099), (7, 8193),
                                   (1023, 1025), (4096, 4608), (1, 70001)])
@pytest.mark.parametrize("pad,shift", [(0, 0), (16, 0), (3, 0), (0, 1)])
def test_quantizer_routes(dtype, shape, pad, shift):
    rows, cols = shape
    g = torch.Generator().manual_seed(rows + cols)
    x = torch.randn(shape, generator=g).to(dtype)
    # the largest magnitude last, where a remainder could be missed
    x[-1, -1] = -9.0
    buf = torch.full((rows * (cols + pad) + shift,), 50.0, dtype=dtype, device="cuda:0")
    X = buf[shift:].view(rows, cols + pad)[:, :cols]
    X.copy_(x)
    q0, s0 = reference(x)
    for layout in ("row", "col"):
        q, s = sk().quantize_e4m3(X, layout)
        torch.cuda.synchronize()
        assert torch.equal(s.cpu(), s0.reshape(1))
        assert torch.equal(q.cpu().contiguous().view(torch.uint8), q0.view(torch.uint8)), layout
    q, s = sk().quantize_e4m3(X.t(), "col")      # column-major in and out
    torch.cuda.synchronize()
    assert torch.equal(s.cpu(), s0.reshape(1))
    assert torch.equal(q.t().cpu().contiguous().view(torch.uint8), q0.view(torch.uint8))
