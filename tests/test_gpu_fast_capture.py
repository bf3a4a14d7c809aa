"""Repeated calls under HIP graph capture: matmul, batched_matmul and conv2d go past the
layout inference and the plan lookup there too, the quantiser allocates its own buffer;
each replay computes the present contents of the captured tensors, with eager calls of
the same signatures and synchronisations between the replays."""
import pytest
import torch

from paper_2212_08964_amd import skgemm as s

pytestmark = pytest.mark.gpu


def rand(*shape, dtype=torch.bfloat16):
    return torch.randint(-2, 3, shape, device="cuda:0").to(dtype)       # exact in FP32 accumulation


def cases():
    """Name: (input tensors, call on them); splits with partial tiles among them."""
    one = lambda: torch.tensor([2.0], device="cuda:0")
    return {
        "matmul": ([rand(300, 2100), rand(2100, 200)], lambda A, B: s.matmul(A, B, out_dtype=torch.float32)),
        "decode": ([rand(5, 4096), rand(900, 4096)], lambda A, B: s.matmul(A, B.t(), out_dtype=torch.float32)),
        "scaled": ([rand(130, 1030), rand(90, 1030), one(), one()],
                   lambda A, B, a, b: s.matmul(A, B.t(), out_dtype=torch.float32, scale_a=a, scale_b=b)),
        "batched": ([rand(3, 130, 1100), rand(3, 1100, 70)], lambda A, B: s.batched_matmul(A, B, out_dtype=torch.float32)),
        "conv": ([rand(2, 9, 7, 64), rand(40, 3, 3, 64)], lambda x, w: s.conv2d(x, w, padding=(1, 1), out_dtype=torch.float32)),
        "quantize": ([rand(300, 1111)], lambda x: torch.cat([v.view(torch.uint8).flatten() for v in s.quantize_e4m3(x)])),
    }


@pytest.mark.parametrize("name", ["matmul", "decode", "scaled", "batched", "conv", "quantize"])
def test_replays(name):
    torch.manual_seed(0)
    tensors, call = cases()[name]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(3):                      # the signature is known, the stream has its workspace
            call(*tensors)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        out = call(*tensors)
    for i in range(4):
        for t in tensors:
            if t.dtype == torch.bfloat16:
                t.copy_(rand(*t.shape) * (i + 1 if name == "quantize" else 1))
        want = call(*tensors).clone()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), i
        if name == "matmul":
            assert torch.equal(out, tensors[0].float() @ tensors[1].float())
