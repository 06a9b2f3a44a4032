"""Every kernel that brings its rows straight into LDS, forced by name: TSMM of
one small tile a wave (tsmm_once) and staged TSMTTSM (tsmttsm_stage).

Rows: less than a tile, one tile, and for three blocks several tiles of every
wave with a ragged one at the end.  Widths: the class's largest, one less and
its smallest (both ways round for TSMTTSM); rows contiguous and, where they are
whole 16-byte chunks, padded; old values of TSMM read and not (those that are not are NaN),
rows of NaN and infinities, memory around the result untouched.  Integer inputs
make every product, sum and stored result exact, so each result must equal
numpy's bit for bit."""
import numpy as np
import pytest
import torch

from paper_1905_03136_amd import _lib, api, codegen, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NUMPY = {"r64": np.float64, "c128": np.complex128, "r32": np.float32, "c64": np.complex64}
TORCH = {"r64": torch.float64, "c128": torch.complex128, "r32": torch.float32, "c64": torch.complex64}
ONCE = {codegen.variant_name(v): v for v in codegen.once_variants()}
STAGE = {codegen.variant_name(v): v for v in codegen.stage_variants()}


def registered(name):
    if name not in {_lib.tsg_variant_name(i) for i in range(_lib.tsg_variant_count())}:
        pytest.skip("spills registers: not in the library")


def pads(dt, *widths):
    """Pads of the matrices' rows: none, and for rows of whole 16-byte chunks one chunk more of each."""
    es = np.dtype(NUMPY[dt]).itemsize
    each = [(0, 16 // es) if w * es % 16 == 0 else (0,) for w in widths]
    return [(a, b) for a in each[0] for b in each[1]]


def placed(x, dt, pad):
    """(view, buffer): x with `pad` more columns a row, 7 around it."""
    k, w = x.shape
    buf = torch.full((k * (w + pad) + 64,), 7, dtype=TORCH[dt], device=DEV)
    v = buf[:k * (w + pad)].view(k, w + pad)[:, :w]
    v.copy_(x)
    return v, buf


def dev(x, dt):
    with np.errstate(invalid="ignore"):
        return torch.from_numpy(np.ascontiguousarray(x.astype(NUMPY[dt]))).to(DEV)


def forced(name, grid, call):
    assert _lib.tsg_force_variant(name) == 0 and _lib.tsg_set_grid_limit(grid) == 0
    try:
        return call()
    finally:
        _lib.tsg_set_grid_limit(0)
        _lib.tsg_force_variant(None)


def wave_lds(c, M, N, es, beta):
    piece = lambda w: -(-16 * c["U"] * w * es // 1024) * 1040  # noqa: E731
    return max(piece(M), piece(N)) + 256 + (piece(N) + 256 if beta else 0)


@pytest.mark.parametrize("name", sorted(ONCE))
def test_one_tile_tsmm(name):
    registered(name)
    v = ONCE[name]
    c, dt = v["cfg"], v["dt"]
    cplx = dt in ("c128", "c64")
    es = np.dtype(NUMPY[dt]).itemsize
    am, an = codegen.once_above(v)
    rows = 16 * c["U"]
    long = 6 * rows * c["WPB"] + rows + 5
    for M, N in sorted({(v["maxM"], v["maxN"]), (max(am + 1, v["maxM"] - 1), max(an + 1, v["maxN"] - 1)), (am + 1, an + 1)}):
        for K in (rows - 3, rows, long):
            print("%s %dx%d K=%d" % (name, M, N, K), flush=True)
            A = inputs.host_integers(K, M, 101, inputs.STREAM_A, cplx)
            X = inputs.host_integers(M, N, 101, inputs.STREAM_C, cplx)
            old = inputs.host_integers(K, N, 101, inputs.STREAM_B, cplx)
            AX = A @ X
            dX = torch.from_numpy(X).to(DEV)
            flat, prior, none = dev(A, dt), dev(old, dt), dev(np.full(old.shape, np.nan), dt)
            refs = dev(AX, dt), dev(AX + old, dt)
            for la, lb in pads(dt, M, N):
                dA = placed(flat, dt, la)[0]
                for beta in (0.0, 1.0):
                    lds = codegen.once_c_bytes(dt, c) + (2 if c["DB"] else 1) * c["WPB"] * wave_lds(c, M, N, es, beta)
                    for grid in (0, 3) if K == long else (0,):
                        out, buf = placed(prior if beta else none, dt, lb)
                        what = (name, M, N, K, la, lb, beta, grid)
                        call = lambda: api.tsmm(dA, dX, out=out, beta=beta)  # noqa: E731
                        if lds > codegen.LDS_BYTES:
                            with pytest.raises(_lib.TsgError, match="forced variant"):
                                forced(name, grid, call)
                            continue
                        forced(name, grid, call)
                        assert torch.equal(out, refs[int(beta)]), what
                        out.fill_(7)
                        assert bool((buf == 7).all()), what
        # rows that are not finite reach their own results only
        bad = A.copy()
        at = [0, 1, rows - 1, rows, K // 2, K - 1]
        bad[at] = [[np.nan if r % 2 else np.inf] for r in range(len(at))]
        clean = np.ones(K, bool)
        clean[at] = False
        got = forced(name, 0, lambda: api.tsmm(dev(bad, dt), dX)).cpu().numpy()
        assert np.array_equal(got[clean], AX[clean]), (name, M, N)
        assert not np.isfinite(got[~clean]).any(), (name, M, N)


@pytest.mark.parametrize("name", sorted(STAGE))
def test_staged_tsmttsm(name):
    registered(name)
    v = STAGE[name]
    c, dt = v["cfg"], v["dt"]
    cplx = dt in ("c128", "c64")
    wide, narrow, sym = v["maxM"], v["maxN"], bool(c.get("SYM"))
    if sym:
        widths = [(w, w) for w in sorted({narrow, narrow - 3})]  # (its groups of four: up to maxN columns)
    else:
        widths = [(wide, narrow), (wide - 15, narrow - 3), (wide - 1, max(narrow - 1, narrow - 3))]
        widths = [p for p in widths if p[0] >= p[1]]
        widths += [(n, m) for m, n in widths[:1]]
    rt = c["RT"]
    for M, N in dict.fromkeys(widths):
        for K in (rt - 1, rt, 3 * 7 * rt + rt // 2 + 1):
            print("%s %dx%d K=%d" % (name, M, N, K), flush=True)
            A = inputs.host_integers(K, M, 102, inputs.STREAM_A, cplx)
            B = A if sym else inputs.host_integers(K, N, 102, inputs.STREAM_B, cplx)
            flat, other = dev(A, dt), dev(B, dt)
            for op in ("T", "C") if cplx else ("T",):
                ref = torch.from_numpy((A.conj() if op == "C" else A).T @ B).to(DEV)
                for la, lb in pads(dt, M, N):
                    dA = placed(flat, dt, la)[0]
                    dB = dA if sym else placed(other, dt, lb)[0]
                    for grid in (0, 1, 3):
                        out = torch.full((M, N + 2), 7, dtype=api._SMALL[TORCH[dt]], device=DEV)
                        forced(name, grid, lambda: api.tsmttsm(dA, dB, op=op, out=out[:, :N]))
                        what = (name, M, N, K, op, la, lb, grid)
                        assert torch.equal(out[:, :N], ref), what
                        assert bool((out[:, N:] == 7).all()), what


@pytest.mark.parametrize("dt,M,N", [("r64", 17, 20), ("r64", 3, 16), ("c128", 9, 12), ("r32", 16, 5), ("r32", 31, 30), ("c64", 20, 20)])
def test_unforced_calls_around_the_row_rule(dt, M, N):
    """As many rows as the dispatch wants for these kernels, and one less."""
    u = int(api.kernel_name("tsmm", TORCH[dt], M, N).split("_once_u")[1].split("_")[0])
    cplx = dt in ("c128", "c64")
    for tiles in (1024, 4096, 6144):
        for K in (16 * u * tiles - 1, 16 * u * tiles):
            print("%s %dx%d K=%d" % (dt, M, N, K), flush=True)
            A = inputs.host_integers(K, M, 103, inputs.STREAM_A, cplx)
            X = inputs.host_integers(M, N, 103, inputs.STREAM_C, cplx)
            old = inputs.host_integers(K, N, 103, inputs.STREAM_B, cplx)
            dA, dX, AX = dev(A, dt), torch.from_numpy(X).to(DEV), A @ X
            assert torch.equal(api.tsmm(dA, dX), dev(AX, dt))
            assert torch.equal(api.tsmm(dA, dX, out=dev(old, dt), beta=1.0), dev(AX + old, dt))
