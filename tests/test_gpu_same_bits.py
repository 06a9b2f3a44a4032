"""One product by every route gives the same bits: eagerly (few blocks: summed
by the last of them in the same launch), without allocation and replayed from a
graph (slots summed by a second kernel).  Uniform inputs, whose sums depend on
the order of the additions; grids whose slots are fewer, as many and more than
a block's slices."""
import pytest
import torch

from paper_1905_03136_amd import _lib, api, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TYPES = {"r64": torch.float64, "c128": torch.complex128, "r32": torch.float32, "c64": torch.complex64}


@pytest.mark.parametrize("dt", list(TYPES))
@pytest.mark.parametrize("M,N", [(1, 1), (1, 2), (2, 2), (3, 3), (4, 4), (5, 5), (6, 6), (7, 7), (8, 8), (7, 5), (16, 9),
                                 (16, 16)])
def test_eager_no_alloc_and_graph(dt, M, N):
    assert _lib.tsg_init(0) == 0
    cplx = TYPES[dt].is_complex
    s = torch.cuda.Stream()
    for K in (300, 2500, 10007, 16384, 40000):
        print("bits %s %dx%d K=%d" % (dt, M, N, K), flush=True)
        A = inputs.device_uniform(K, M, 99, inputs.STREAM_A, cplx, DEV).to(TYPES[dt])
        B = inputs.device_uniform(K, N, 99, inputs.STREAM_B, cplx, DEV).to(TYPES[dt])
        out, fixed = (torch.empty(M, N, dtype=api._SMALL[TYPES[dt]], device=DEV) for _ in range(2))
        torch.cuda.synchronize()
        for grid in (0, 2, 5, 17, 33, 64):
            assert _lib.tsg_set_grid_limit(grid) == 0
            try:
                with torch.cuda.stream(s):
                    eager = api.tsmttsm(A, B)
                    assert _lib.tsg_tsmttsm_noalloc(api._DT[A.dtype], 0, K, M, N, A.data_ptr(), M, B.data_ptr(), N,
                                                    fixed.data_ptr(), N, s.cuda_stream) == 0
                torch.cuda.synchronize()
                g = torch.cuda.CUDAGraph()
                with torch.cuda.graph(g, stream=s):
                    api.tsmttsm(A, B, out=out)
            finally:
                _lib.tsg_set_grid_limit(0)
            for turn in range(3):
                out.fill_(-1.0)
                torch.cuda.synchronize()
                with torch.cuda.stream(s):
                    g.replay()
                torch.cuda.synchronize()
                assert torch.equal(out, eager), ("graph", K, grid, turn)
            assert torch.equal(fixed, eager), ("no-alloc", K, grid)
