"""TSMTTSM calls of few blocks, whose last block sums them in the same launch:
grids around the largest such one, widths with fewer and more entries than a
block has threads, calls in a row, on two streams, without allocation and in
graph replays (the counter starts every launch at zero).  Integer inputs make
every sum exact, so each result must equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_03136_amd import _lib, api, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NUMPY = {"r64": np.float64, "c128": np.complex128, "r32": np.float32, "c64": np.complex64}


def pair(K, M, N, dt, seed=95):
    cplx = dt in ("c128", "c64")
    A = inputs.host_integers(K, M, seed, inputs.STREAM_A, cplx)
    B = inputs.host_integers(K, N, seed, inputs.STREAM_B, cplx)
    dev = [torch.from_numpy(np.ascontiguousarray(x.astype(NUMPY[dt]))).to(DEV) for x in (A, B)]
    return dev[0], dev[1], oracle.tsmttsm(A, B)


@pytest.mark.parametrize("dt", ["r64", "c128", "r32", "c64"])
@pytest.mark.parametrize("M,N", [(1, 2), (2, 2), (3, 3), (4, 4), (1, 16), (7, 5), (8, 8), (16, 9), (16, 16)])
def test_grids_and_widths(dt, M, N):
    for K in (300, 10007, 40000):
        print("small %s %dx%d K=%d" % (dt, M, N, K), flush=True)
        A, B, ref = pair(K, M, N, dt)
        wide = torch.full((M, N + 3), 5, dtype=api._SMALL[A.dtype], device=DEV)
        for grid in (0, 2, 3, 17, 63, 64, 65):
            assert _lib.tsg_set_grid_limit(grid) == 0
            try:
                first, again = api.tsmttsm(A, B), api.tsmttsm(A, B)
                api.tsmttsm(A, B, out=wide[:, :N])
            finally:
                _lib.tsg_set_grid_limit(0)
            assert np.array_equal(first.cpu().numpy(), ref), (K, grid)
            assert torch.equal(first, again) and torch.equal(first, wide[:, :N]), (K, grid)
            assert bool((wide[:, N:] == 5).all())


def test_streams_growth_and_no_alloc():
    """Two streams count in their own workspaces, one that grew starts a new
    count, and the no-alloc calls have theirs."""
    cases = [pair(10007, 4, 4, "r64"), pair(9000, 8, 8, "c128"), pair(2000, 3, 3, "r64", 96)]
    big = pair(200000, 64, 64, "c128")
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    got = []
    for turn in range(6):
        for s in streams:
            with torch.cuda.stream(s):
                got += [(api.tsmttsm(A, B), ref) for A, B, ref in (cases + [big] if turn == 3 else cases)]
    torch.cuda.synchronize()
    for C, ref in got:
        assert np.array_equal(C.cpu().numpy(), ref)
    assert _lib.tsg_init(0) == 0
    for A, B, ref in cases * 2:
        out = torch.empty(ref.shape, dtype=A.dtype, device=DEV)
        assert _lib.tsg_tsmttsm_noalloc(api._DT[A.dtype], 0, A.shape[0], A.shape[1], B.shape[1], A.data_ptr(), A.shape[1],
                                        B.data_ptr(), B.shape[1], out.data_ptr(), out.shape[1],
                                        torch.cuda.current_stream().cuda_stream) == 0
        assert np.array_equal(out.cpu().numpy(), ref)


def test_replays():
    A, B, ref = pair(10007, 4, 4, "r64")
    out = torch.empty(4, 4, dtype=torch.float64, device=DEV)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        api.tsmttsm(A, B, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        api.tsmttsm(A, B, out=out)
    for turn in range(4):
        out.fill_(-1.0)
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), ref), turn
        with torch.cuda.stream(s):
            assert np.array_equal(api.tsmttsm(A, B).cpu().numpy(), ref), turn
