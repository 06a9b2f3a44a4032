"""The TSMTTSM kernels that stage their rows in LDS by direct loads: row counts
around a stage, widths around a 16-column block and a group of four, either
matrix the wider, padded rows, both products of a matrix with itself, and the
layouts they leave to the other kernels.  Integer inputs make every product
and sum exact, so each result must equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_03136_amd import _lib, api, codegen, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NUMPY = {"r64": np.float64, "c128": np.complex128, "r32": np.float32, "c64": np.complex64}
WIDTHS = [(17, 1), (4, 32), (32, 31), (33, 33), (48, 13), (21, 47), (49, 64), (64, 64), (61, 37), (3, 62)]
ROWS = [1, 7, 64, 65, 127, 4099]


def placed(x, dt, pad=0, shift=0):
    """x on the device with `pad` more columns a row, `shift` elements past an aligned start."""
    k, w = x.shape
    buf = torch.zeros(k * (w + pad) + shift, dtype=torch.from_numpy(np.zeros(1, NUMPY[dt])).dtype, device=DEV)
    v = buf[shift:].view(k, w + pad)[:, :w]
    v.copy_(torch.from_numpy(np.ascontiguousarray(x.astype(NUMPY[dt]))))
    return v


def check(A, B, dA, dB, op):
    ref = oracle.tsmttsm(A.conj() if op == "C" else A, B)
    for grid in (0, 3):
        assert _lib.tsg_set_grid_limit(grid) == 0
        try:
            got = api.tsmttsm(dA, dB, op=op).cpu().numpy()
        finally:
            _lib.tsg_set_grid_limit(0)
        assert np.array_equal(got, ref), (A.shape, B.shape, op, grid)


@pytest.mark.parametrize("dt", ["r64", "c128", "r32", "c64"])
@pytest.mark.parametrize("M,N", WIDTHS)
def test_rows_widths_and_layouts(dt, M, N):
    cplx = dt in ("c128", "c64")
    tdt = torch.from_numpy(np.zeros(1, NUMPY[dt])).dtype
    assert "_lds_dma" in api.kernel_name("tsmttsm", tdt, M, N)
    for K in ROWS:
        print("stage %s %dx%d K=%d" % (dt, M, N, K), flush=True)
        A = inputs.host_integers(K, M, 91, inputs.STREAM_A, cplx)
        B = inputs.host_integers(K, N, 91, inputs.STREAM_B, cplx)
        dA, dB = placed(A, dt), placed(B, dt)
        for op in ("T", "C") if cplx else ("T",):
            check(A, B, dA, dB, op)
        # rows padded to whole 16-byte chunks, to odd strides, and a start off
        # the alignment
        es = np.dtype(NUMPY[dt]).itemsize
        pad = lambda w: 16 // es + (-w) % (16 // es)  # noqa: E731
        check(A, B, placed(A, dt, pad(M)), placed(B, dt, pad(N)), "T")
        check(A, B, placed(A, dt, pad(M)), dB, "T")
        check(A, B, placed(A, dt, 1), dB, "T")
        check(A, B, dA, placed(B, dt, 0, 1), "T")


@pytest.mark.parametrize("dt", ["r64", "c128", "r32", "c64"])
@pytest.mark.parametrize("M", [17, 32, 40, 48, 49, 64])
def test_matrix_with_itself(dt, M):
    cplx = dt in ("c128", "c64")
    for K in ROWS:
        print("gram %s %d K=%d" % (dt, M, K), flush=True)
        A = inputs.host_integers(K, M, 92, inputs.STREAM_A, cplx)
        for pad in (0, 16, 1):
            dA = placed(A, dt, pad)
            for op in ("T", "C") if cplx else ("T",):
                check(A, A, dA, dA, op)
            # another view of the same rows: two matrices
            check(A, A, dA, placed(A, dt, pad), "T")


def test_leading_dimension_beyond_the_offsets_falls_back():
    """A leading dimension whose tile would not fit 32-bit offsets is left to
    the other kernels (three rows of it, so that the matrix stays small)."""
    K, M, ld = 3, 24, 1 << 23
    A = inputs.host_integers(K, M, 93, inputs.STREAM_A)
    buf = torch.zeros(K * ld, dtype=torch.float64, device=DEV)
    dA = buf.view(K, ld)[:, :M]
    dA.copy_(torch.from_numpy(A))
    check(A, A, dA, dA, "T")


def test_every_class_is_registered():
    names = {_lib.tsg_variant_name(i) for i in range(_lib.tsg_variant_count())}
    missing = [codegen.variant_name(v) for v in codegen.stage_variants() if codegen.variant_name(v) not in names]
    assert not missing, missing
