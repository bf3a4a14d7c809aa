"""Automatic FP8 plans that take the large tile for rows off 128 bytes: calls that only
the small tile can run (a leading dimension whose 256-row slab is beyond 32-bit
offsets, a workspace, or the library's own array, too small for 256x256 partial
tiles) still run, on the small tile's plan."""
import ctypes

import pytest
import torch

from paper_2212_08964_amd import skgemm as s


def ints(rows, cols, seed, ld=None):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    v = torch.randint(-2, 3, (rows, cols), generator=g, device="cuda:0").to(torch.float32).to(torch.float8_e4m3fn)
    if ld is None:
        return v
    buf = torch.empty(rows * ld, dtype=torch.uint8, device="cuda:0").view(torch.float8_e4m3fn).view(rows, ld)
    buf[:, :cols] = v
    return buf[:, :cols]


@pytest.mark.skipif(torch.cuda.is_available(), reason="made-up addresses: only where nothing can be launched")
def test_accepted_without_a_gpu():
    """Past the checks the launch fails for want of a device (ERR_HIP)."""
    M, N, K = 129, 129, 9000001
    plan = s.Plan(M, N, K, lb=s.COL_MAJOR, ta=s.F8E4M3, tc=s.F32, num_cus=256, occupancy=2)
    assert plan.info()["tile"][:3] == (256, 256, 128)
    small = s.Plan(M, N, K, lb=s.COL_MAJOR, ta=s.F8E4M3, tc=s.F32, num_cus=256, occupancy=2, tile=(128, 128, 128))
    assert plan.workspace_size() >= small.workspace_size()
    assert plan.trace_capacity() >= small.trace_capacity()

    def status(**k):
        a = dict(lda=K, ldb=K, ws=1 << 20, nws=plan.workspace_size()) | k
        return s.lib().skgemm_run(plan.handle, 1 << 20, a["lda"], 1 << 20, a["ldb"], 1 << 20, N, 1.0, 0.0, None, None,
                                  ctypes.c_void_p(a["ws"]), a["nws"], None)

    assert status() == s.ERR_HIP
    assert status(nws=small.workspace_size()) == s.ERR_HIP
    assert status(lda=16777000) == s.ERR_HIP
    assert status(lda=17000000) == s.ERR_UNSUPPORTED           # beyond the small tile's, too
    assert status(lda=K - 1) == s.ERR_INVALID_ARG
    assert status(nws=small.workspace_size() - 1) == s.ERR_WORKSPACE


@pytest.mark.skipif(torch.cuda.is_available(), reason="made-up addresses: only where nothing can be launched")
@pytest.mark.parametrize("M,N,K", [(1922, 8252, 4018), (2786, 7310, 3898)])
def test_library_array_without_a_gpu(M, N, K):
    """The large tile's plan needs less than the small tile's: a leading dimension that
    only the latter can run gets as far as looking for the library's array (ERR_HIP)."""
    plan = s.Plan(M, N, K, lb=s.COL_MAJOR, ta=s.F8E4M3, tc=s.F32, num_cus=256, occupancy=2)
    small = s.Plan(M, N, K, lb=s.COL_MAJOR, ta=s.F8E4M3, tc=s.F32, num_cus=256, occupancy=2, tile=(128, 128, 128))
    assert plan.info()["tile"][:3] == (256, 256, 128)
    assert plan.info()["fixup_ws_bytes"] < small.info()["fixup_ws_bytes"] <= 64 << 20

    def status(lda):
        return s.lib().skgemm_run_noalloc(plan.handle, 1 << 20, lda, 1 << 20, K, 1 << 20, N, 1.0, 0.0, None, None, None)

    assert status(K) == s.ERR_HIP
    assert status(8400003) == s.ERR_HIP
    assert status(K - 1) == s.ERR_INVALID_ARG
    assert status(17000000) == s.ERR_UNSUPPORTED


@pytest.mark.gpu
def test_library_array_of_the_other_tile():
    """The same call on the GPU (rows 8400003 elements apart)."""
    M, N, K, ld = 1922, 8252, 4018, 8400003
    plan = s.Plan(M, N, K, lb=s.COL_MAJOR, ta=s.F8E4M3, tc=s.F32)
    A, B = ints(M, K, 1, ld=ld), ints(N, K, 2).t()
    C = torch.empty((M, N), device="cuda:0")
    plan.run_noalloc(A.data_ptr(), ld, B.data_ptr(), K, C.data_ptr(), N, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(C, A.float() @ B.float())


@pytest.mark.gpu
def test_large_leading_dimension():
    M, N, K = 682, 4164, 7133
    assert s.Plan(M, N, K, lb=s.COL_MAJOR, ta=s.F8E4M3, tc=s.F32).info()["tile"][:3] == (256, 256, 128)
    A, B = ints(M, K, 1, ld=8400003), ints(N, K, 2).t()
    ref = A.float() @ B.float()
    assert torch.equal(s.matmul(A, B), ref)
    assert torch.equal(s.matmul(A.contiguous(), B), ref)


@pytest.mark.gpu
def test_library_array():
    M, N, K = 682, 4164, 7133
    plan = s.Plan(M, N, K, lb=s.COL_MAJOR, ta=s.F8E4M3, tc=s.F32)
    assert plan.info()["fixup_ws_bytes"] > 64 << 20
    A, B = ints(M, K, 1), ints(N, K, 2).t()
    C = torch.empty((M, N), device="cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    for _ in range(3):
        C.zero_()
        plan.run_noalloc(A.data_ptr(), K, B.data_ptr(), K, C.data_ptr(), N, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(C, A.float() @ B.float())
