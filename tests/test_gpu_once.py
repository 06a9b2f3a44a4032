"""The TSMM kernels of one small tile a wave: row counts around their tiles
(16 to 128 rows a wave, up to 16 waves a block), widths around slices and
groups of four and blocks of 16 columns, old values read or not, each form of
the small operand, padded rows, the layouts they leave to the other kernels,
and memory around the result untouched.  Integer inputs make every product,
sum and stored result exact, so each result must equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_03136_amd import _lib, api, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NUMPY = {"r64": np.float64, "c128": np.complex128, "r32": np.float32, "c64": np.complex64}
# every class of 4, 8, 16 and more columns has its own widths in the table
WIDTHS = [(1, 1), (4, 4), (3, 16), (16, 5), (9, 12), (17, 20), (31, 30), (40, 33), (25, 47), (64, 4), (5, 64),
          (63, 39), (36, 56), (57, 61)]
ROWS = [1, 15, 16, 17, 129, 1023, 4111]


def placed(x, dt, pad=0, shift=0):
    """(view, buffer): x on the device with `pad` more columns a row, `shift`
    elements past an aligned start, 7 around and after it."""
    k, w = x.shape
    n = k * (w + pad)
    buf = torch.full((n + shift + 64,), 7, dtype=torch.from_numpy(np.zeros(1, NUMPY[dt])).dtype, device=DEV)
    v = buf[shift:shift + n].view(k, w + pad)[:, :w]
    v.copy_(torch.from_numpy(np.ascontiguousarray(x.astype(NUMPY[dt]))))
    return v, buf


def check(A, X, old, dt, la, lb, alpha=1.0, beta=0.0, conjA=False, opC="N"):
    ref = alpha * oracle.tsmm(A.conj() if conjA else A, X)
    if beta:
        ref = ref + beta * old
    small = {"N": X, "T": X.T, "C": X.conj().T}[opC]
    dX = torch.from_numpy(np.ascontiguousarray(small)).to(DEV)
    for grid in (0, 3):
        dA = placed(A, dt, *la)[0]
        start = old if beta else np.full(old.shape, np.nan)
        out, buf = placed(start, dt, *lb)
        assert _lib.tsg_set_grid_limit(grid) == 0
        try:
            api.tsmm(dA, dX, out=out, alpha=alpha, beta=beta, conjA=conjA, opC=opC)
        finally:
            _lib.tsg_set_grid_limit(0)
        what = (dt, A.shape, X.shape, la, lb, alpha, beta, conjA, opC, grid)
        assert np.array_equal(out.cpu().numpy(), ref), what
        out.fill_(7)
        assert bool((buf == 7).all()), what


@pytest.mark.parametrize("dt", ["r64", "c128", "r32", "c64"])
@pytest.mark.parametrize("M,N", WIDTHS)
def test_rows_widths_forms_and_layouts(dt, M, N):
    cplx = dt in ("c128", "c64")
    es = np.dtype(NUMPY[dt]).itemsize
    chunk = lambda w: 16 // es + (-w) % (16 // es)  # noqa: E731: whole 16-byte chunks a row
    for K in ROWS:
        print("once %s %dx%d K=%d" % (dt, M, N, K), flush=True)
        A = inputs.host_integers(K, M, 93, inputs.STREAM_A, cplx)
        X = inputs.host_integers(M, N, 93, inputs.STREAM_C, cplx)
        old = inputs.host_integers(K, N, 93, inputs.STREAM_B, cplx)
        check(A, X, old, dt, (0, 0), (0, 0))
        check(A, X, old, dt, (0, 0), (0, 0), alpha=2.0, beta=-1.0, opC="T")
        check(A, X, old, dt, (chunk(M), 0), (chunk(N), 0), beta=1.0)
        if cplx:
            check(A, X, old, dt, (0, 0), (0, 0), conjA=True, opC="C")
            check(A, X, old, dt, (0, 0), (chunk(N), 0), beta=2.0, conjA=True)
        # odd strides and starts off the alignment
        check(A, X, old, dt, (1, 0), (1, 0))
        check(A, X, old, dt, (0, 1), (0, 0), beta=1.0)
        check(A, X, old, dt, (0, 0), (0, 1))


@pytest.mark.parametrize("dt", ["r64", "c128", "r32", "c64"])
def test_route(dt):
    """Contiguous matrices of widths with no kernel of their own take these
    kernels; a narrow non-square pair in binary64 keeps its exact widths."""
    tdt = torch.from_numpy(np.zeros(1, NUMPY[dt])).dtype
    for M, N in [(3, 16), (17, 20), (9, 12), (64, 4), (28, 7)]:
        assert "_mfma_once_" in api.kernel_name("tsmm", tdt, M, N), (M, N)
    assert ("_once_" in api.kernel_name("tsmm", tdt, 3, 8)) == (dt in ("r32", "c64"))


@pytest.mark.parametrize("M,N", [(8, 8), (20, 24), (40, 33)])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_bad_row_stays_in_its_row(M, N, bad):
    """Columns past a width are operands too: what lies there (the next row's
    values) must not reach a result."""
    A = inputs.host_integers(1024, M, 94, inputs.STREAM_A, False)
    A[[0, 37, 512, 1023]] = bad
    X = inputs.host_integers(M, N, 94, inputs.STREAM_C, False)
    got = api.tsmm(placed(A, "r64")[0], torch.from_numpy(X).to(DEV)).cpu().numpy()
    clean = np.ones(1024, bool)
    clean[[0, 37, 512, 1023]] = False
    assert np.array_equal(got[clean], A[clean] @ X)
    assert not np.isfinite(got[~clean]).all(axis=1).any()


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("M,N", [(17, 17), (33, 33), (16, 40), (46, 46), (48, 48), (64, 64), (40, 64)])
def test_wide_complex_updates(dt, M, N):
    """Wide complex updates take a kernel that reads the old values with A, of
    their own widths or of a range."""
    for K in (1, 130, 4111):
        print("update %s %dx%d K=%d" % (dt, M, N, K), flush=True)
        A = inputs.host_integers(K, M, 95, inputs.STREAM_A, True)
        X = inputs.host_integers(M, N, 95, inputs.STREAM_C, True)
        old = inputs.host_integers(K, N, 95, inputs.STREAM_B, True)
        for la, lb in (((0, 0), (0, 0)), ((3, 0), (2, 0)), ((0, 1), (1, 1))):
            check(A, X, old, dt, la, lb, alpha=-1.0, beta=1.0)
            check(A, X, old, dt, la, lb, beta=2.0, conjA=True, opC="C")
