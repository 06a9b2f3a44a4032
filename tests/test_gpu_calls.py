"""The native torch calls: what they take, with the strides, streams and
threads of a plain call, what they leave to the Python functions, and that both
give the same results and errors."""
import threading

import numpy as np
import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

import oracle
from paper_1905_03136_amd import _calls, _lib, api, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TYPES = [torch.float64, torch.complex128, torch.float32, torch.complex64]


def tall(K, M, dt, stream=inputs.STREAM_A):
    return torch.from_numpy(inputs.host_integers(K, M, 97, stream, dt.is_complex)).to(DEV).to(dt)


def wide(x):
    return x.cpu().to(torch.complex128 if x.is_complex() else torch.float64).numpy()


@pytest.fixture(autouse=True)
def bound():
    api._bind()


@pytest.mark.parametrize("dt", TYPES)
@pytest.mark.parametrize("K", [1, 2, 1000])
def test_plain_calls(dt, K):
    for acc in ("f64", "f32") if dt in (torch.float32, torch.complex64) else ("f64",):
        base = tall(K, 12, dt)
        A, B = base[:, 1:6], tall(K, 7, dt, inputs.STREAM_B)
        X = tall(5, 7, api._SMALL[dt], inputs.STREAM_C)
        out = torch.zeros(5, 9, dtype=api._SMALL[dt], device=DEV)
        for op in ("T", "C"):
            C = _calls.tsmttsm(A, B, op, None, acc)
            ref = oracle.tsmttsm(wide(A).conj() if op == "C" else wide(A), wide(B))
            assert C.dtype == api._SMALL[dt] and np.array_equal(C.cpu().numpy(), ref)
            assert _calls.tsmttsm(torch.nn.Parameter(A), B, op, out[:, :7], acc).data_ptr() == out.data_ptr()
            assert torch.equal(out[:, :7], C) and not C.requires_grad
        for opC, small in (("N", X), ("T", X.T.contiguous()), ("C", X.conj().resolve_conj().T.contiguous())):
            for conjA in (False, True):
                P = _calls.tsmm(A, small, None, 2.0, 0.0, conjA, opC, acc)
                ref = 2.0 * oracle.tsmm(wide(A).conj() if conjA else wide(A), X.cpu().numpy())
                assert P.dtype == dt and np.array_equal(wide(P), ref)
                W = B.clone()
                assert _calls.tsmm(A, small, W, 2.0, -1.0, conjA, opC, acc) is W
                assert np.array_equal(wide(W), ref - wide(B))


class Sub(torch.Tensor):
    pass


class Mode(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def test_what_they_leave_to_python():
    A, B, X = tall(50, 4, torch.float64), tall(50, 3, torch.float64), tall(4, 3, torch.float64)
    no = NotImplemented
    for bad in (A.cpu(), A.as_subclass(Sub), A.int(), A[:, ::2], A[:0], A[:, :0], A[0], A[None], A.to(torch.float16), 3, None):
        assert _calls.tsmttsm(bad, B, "T", None, "f64") is no
        assert _calls.tsmttsm(B, bad, "T", None, "f64") is no
        assert _calls.tsmm(bad, X, None, 1.0, 0.0, False, "N", "f64") is no
        assert _calls.tsmm(A, bad, None, 1.0, 0.0, False, "N", "f64") is no
    assert _calls.tsmttsm(A, B[:49], "T", None, "f64") is no
    assert _calls.tsmttsm(A, B.float(), "T", None, "f64") is no
    assert _calls.tsmttsm(A, B, "H", None, "f64") is no and _calls.tsmttsm(A, B, "T", None, "f32") is no
    assert _calls.tsmttsm(A, B, "T", X[:3], "f64") is no and _calls.tsmttsm(A, B, "T", X.float(), "f64") is no
    assert _calls.tsmm(A, X, None, 1.0, 1.0, False, "N", "f64") is no
    assert _calls.tsmm(A, X, None, 1, 0.0, False, "N", "f64") is no
    assert _calls.tsmm(A, X, None, 1.0, 0.0, 0, "N", "f64") is no
    assert _calls.tsmm(A, X, B[:40], 1.0, 0.0, False, "N", "f64") is no
    wide65 = torch.zeros(50, 65, dtype=torch.float64, device=DEV)
    assert _calls.tsmttsm(wide65, B, "T", None, "f64") is no
    Z = torch.zeros(50, 2, dtype=torch.complex128, device=DEV)
    assert _calls.tsmttsm(Z.conj(), Z, "T", None, "f64") is no
    with Mode():
        assert _calls.tsmttsm(A, B, "T", None, "f64") is no
    ref = api.tsmttsm(A, B)
    with Mode():
        assert torch.equal(api.tsmttsm(A, B), ref)
    assert torch.equal(api.tsmttsm(A.as_subclass(Sub), B).as_subclass(torch.Tensor), ref)
    assert torch.equal(api.tsmttsm(A, B, op="H"), ref)
    assert torch.equal(api.tsmm(A, X, alpha=2), api.tsmm(A, X, alpha=2.0))
    with pytest.raises(ValueError):
        api.tsmm(A, X, beta=1.0)
    with pytest.raises(ValueError):
        api.tsmttsm(A[:, ::2], B)
    with pytest.raises(_lib.TsgError):
        api.tsmttsm(wide65, B)
    assert _lib.tsg_force_variant(_lib.tsg_variant_name(0)) == 0
    try:
        with pytest.raises(_lib.TsgError, match="forced variant"):
            api.tsmttsm(tall(50, 61, torch.complex128), tall(50, 59, torch.complex128))
    finally:
        _lib.tsg_force_variant("")


def test_streams_and_threads():
    A, B = tall(100000, 8, torch.float64), tall(100000, 8, torch.float64, inputs.STREAM_B)
    ref = oracle.tsmttsm(wide(A), wide(B))
    torch.cuda.synchronize()
    got = []

    def work():
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(20):
                x = A * 2.0
                C = api.tsmttsm(x, B)
                x.zero_()
                got.append(C)
        s.synchronize()

    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(got) == 80
    for C in got:
        assert np.array_equal(C.cpu().numpy(), 2.0 * ref)
