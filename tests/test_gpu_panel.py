"""The blocked path's panels and products at the sizes where they can go
wrong: panels of one to a few 16-row blocks and ragged last panels, a matrix
that ends where its allocation ends, and products with every tile shape,
ragged in rows, columns and depth.

L = [[I, 0], [C, I]] with small integers gives X = B - N B (N the part below
the diagonal blocks) exactly, in every data type, so those results are compared
bit for bit with torch's product of the same integers."""
import numpy as np
import pytest

import workloads as W
from parity import assert_parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
hs = pytest.importorskip("paper_2608_25469_amd")

DT = {"d": torch.float64, "z": torch.complex128, "s": torch.float32, "c": torch.complex64}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    hs.lib()


@pytest.mark.parametrize("cx", [False, True], ids=["real", "complex"])
@pytest.mark.parametrize("ib", [16, 32, 256, 0])
def test_ragged_panels(cx, ib):
    """Last panels of 1, 2, 7, 8, 9, 15, 16, 17 rows after whole ones, and
    lone panels around the steps of the kernel's sizes (128, 256, 512 rows);
    1, 15, 16, 17 and 33 columns."""
    span = ib or (256 if cx else 512)
    sizes = [span * k + r for k, r in ((1, 1), (2, 2), (1, 7), (1, 8), (1, 9), (1, 15), (1, 16), (1, 17))]
    if ib == 0:
        sizes += [65, 127, 128, 129, 255, 256, 257] + ([] if cx else [511, 512])
    for j, m in enumerate(s for s in sizes if s > 64 or ib):
        n = (1, 15, 16, 17, 33)[j % 5]
        unit = j % 3 == 0
        L, B = W.problem(900 + j, m, n, cx)
        alpha = complex(-0.5, 1.0) if cx else -0.75
        Ld, Bd = hs.to_colmajor(L), hs.to_colmajor(B, ld=m + j % 3)
        hs.trsm(Ld, Bd, alpha, unit=unit, block_size=ib, path=2)
        torch.cuda.synchronize()
        assert_parity(L, B, hs.from_colmajor(Bd), alpha, unit=unit, tag=("panel", m, n, cx, ib))


def _ints(shape, dt, lo, hi, g):
    t = torch.randint(lo, hi + 1, shape, generator=g, device="cuda").to(DT[dt])
    if dt in "zc":
        t = torch.complex(t.real, torch.randint(lo, hi + 1, shape, generator=g, device="cuda").to(t.real.dtype))
    return t


@pytest.mark.parametrize("dt", list("dzsc"))
@pytest.mark.parametrize("m,m1,n", [(577, 512, 30), (1030, 700, 33), (1531, 530, 127), (1100, 1024, 700),
                                    (2050, 1000, 1025), (3001, 1501, 2333), (4250, 2200, 4099)])
def test_products_exact(dt, m, m1, n):
    g = torch.Generator(device="cuda").manual_seed(m + n)
    Ls = torch.full((m, m), float("nan"), dtype=DT[dt], device="cuda")   # row j: column j of L
    Ls = torch.triu(torch.zeros_like(Ls)) + torch.tril(Ls, -1)
    Ls.diagonal().fill_(1)
    C = _ints((m - m1, m1), dt, -2, 2, g)
    Ls[:m1, m1:] = C.t()
    B = hs.colmajor(m, n, DT[dt])
    B.copy_(_ints((m, n), dt, -3, 3, g))
    want = B.clone()
    want[m1:] -= C @ want[:m1].contiguous()
    hs.trsm(Ls.t(), B, 1.0)
    torch.cuda.synchronize()
    assert torch.equal(B, want), (dt, m, m1, n)


def test_mixed_products_exact():
    """The same through the mixed mode, whose products round their operands
    to FP32 (small integers are exact)."""
    for m, m1, n in ((1100, 700, 37), (2300, 1100, 1300), (4200, 2100, 4097)):
        g = torch.Generator(device="cuda").manual_seed(m)
        Ls = torch.eye(m, dtype=torch.float64, device="cuda")
        C = _ints((m - m1, m1), "d", -2, 2, g)
        Ls[:m1, m1:] = C.t()
        B = hs.colmajor(m, n, torch.float64)
        B.copy_(_ints((m, n), "d", -3, 3, g))
        want = B.clone()
        want[m1:] -= C @ want[:m1].contiguous()
        hs.trsm(Ls.t(), B, 1.0, mixed=True)
        torch.cuda.synchronize()
        assert torch.equal(B, want), (m, m1, n)


@pytest.mark.parametrize("dt", list("dzsc"))
def test_chains_on_two_streams_and_with_infinities(dt):
    """Chains (one launch, workgroups handing X on): several at once on two
    streams give the bits each gives alone, and infinities and NaNs in B stay
    in their columns and end where a lone solve ends."""
    g = torch.Generator(device="cuda").manual_seed(5)
    cases = []
    for m, n in ((1300, 40), (2049, 17), (700, 333)):
        Ls = torch.triu(_ints((m, m), dt, -2, 2, g), 1) / m   # row j: column j of L
        Ls.diagonal().fill_(1.5)
        B = hs.colmajor(m, n, DT[dt])
        B.copy_(_ints((m, n), dt, -3, 3, g))
        B[m // 3, 2] = float("inf")
        B[m // 2, 5] = float("nan")
        alone = B.clone()
        hs.trsm(Ls.t(), alone, 1.0)
        cases.append((Ls, B, alone))
    torch.cuda.synchronize()
    sides = [torch.cuda.Stream() for _ in range(2)]
    outs = []
    for rep in range(4):
        for k, (Ls, B, _) in enumerate(cases):
            X = B.clone()
            torch.cuda.synchronize()
            hs.trsm(Ls.t(), X, 1.0, stream=sides[(rep + k) % 2])
            outs.append((k, X))
    torch.cuda.synchronize()
    for k, X in outs:
        a, b = (torch.view_as_real(t.resolve_conj()) if t.is_complex() else t for t in (X, cases[k][2]))
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)), (dt, k)
    for Ls, B, alone in cases:
        fine = [c for c in range(B.shape[1]) if c not in (2, 5)]
        ref = torch.linalg.solve_triangular(Ls.t().to(DT["z" if dt in "zc" else "d"]).contiguous(),
                                            B[:, fine].to(DT["z" if dt in "zc" else "d"]).contiguous(), upper=False)
        # forward error of a solve with kappa < 10: a few units in the last place times m
        eps = 2.0 ** (-52 if dt in "dz" else -23)
        assert (alone[:, fine] - ref).abs().max().item() <= 10 * B.shape[0] * eps * ref.abs().max().item()
        assert not torch.isfinite(alone[B.shape[0] // 3, 2].abs()) and torch.isnan(alone[B.shape[0] // 2, 5].abs())


def _colmajor(t, ld=None):
    out = hs.colmajor(t.shape[0], t.shape[1], t.dtype, ld=ld)
    out.copy_(t)
    return out


@pytest.mark.parametrize("side,uplo,trans", [("R", "L", "T"), ("R", "L", "C"), ("R", "U", "N"), ("R", "L", "N"), ("R", "U", "C"),
                                             ("L", "U", "N"), ("L", "L", "C")])
@pytest.mark.parametrize("dt", list("dz"))
def test_right_hand_sides_at_strides(dt, side, uplo, trans):
    """One launch reading B where it lies (transposed, reversed, conjugated; k
    up to a panel, and chains) gives the bits of the same solve on a gathered
    copy."""
    g = torch.Generator(device="cuda").manual_seed(11)
    for k, nr in ((65, 1), (130, 17), (257, 40), (512, 33), (700, 257), (1299, 15)):
        # op(A) or op(A)^T as a lower triangle, by the library's own rules
        T = torch.tril(_ints((k, k), dt, -3, 3, g), -1) / k + 1.5 * torch.eye(k, dtype=DT[dt], device="cuda")
        opT = T if side == "L" else T.t()                     # op(A) if no reversal is needed
        lower_op = (uplo == "L") == (trans == "N")
        if lower_op != (side == "L"):                         # the operator is the reversed one
            opT = opT.flip(0, 1)
        A = {"N": opT, "T": opT.t(), "C": opT.mH}[trans]
        assert torch.equal(A, torch.tril(A) if uplo == "L" else torch.triu(A))
        rev = lower_op != (side == "L")
        B = _ints((k, nr), dt, -3, 3, g)                      # the gathered right-hand side
        want = hs.colmajor(k, nr, DT[dt])
        want.copy_(B)
        hs.trsm(_colmajor(T), want, 0.5)
        S = B.flip(0) if rev else B
        S = S if side == "L" else S.t()
        X = _colmajor(S, S.shape[0] + 3)
        hs.trsm_general(_colmajor(A), X, 0.5, side=side, uplo=uplo, trans=trans)
        torch.cuda.synchronize()
        R = X if side == "L" else X.t()
        R = R.flip(0) if rev else R
        assert torch.equal(R, want), (dt, side, uplo, trans, k, nr)


@pytest.mark.parametrize("cx", [False, True], ids=["real", "complex"])
@pytest.mark.parametrize("m,n", [(500, 33), (1300, 40)])
def test_waits_that_give_up_leave_nan(cx, m, n):
    """A wavefront that gives up its wait (here after two looks) forms NaN
    from then on: whatever then is not NaN is what a whole solve gives."""
    import ctypes
    m //= 2 if cx else 1
    L, B = W.problem(7, m, n, cx)
    Ld, Bd, want = hs.to_colmajor(L), hs.to_colmajor(B), hs.to_colmajor(B)
    hs.trsm(Ld, want)
    f = hs.lib().hsma_internal_short_waits
    i64, vp = ctypes.c_int64, ctypes.c_void_p
    f.argtypes = [ctypes.c_int, i64, i64, vp, i64, vp, i64, ctypes.c_int, vp]
    for looks, gives_up in ((1, True), (1 << 20, False)):
        X = Bd.clone()
        assert X.stride() == Bd.stride()
        assert f(cx, m, n, Ld.data_ptr(), m, X.data_ptr(), m, looks, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        a, b = (torch.view_as_real(t) if cx else t for t in (X, want))
        there = ~torch.isnan(a)
        assert torch.equal(a[there], b[there]), (m, n, cx, looks)
        assert bool(there.all()) != gives_up, (m, n, cx, looks)


@pytest.mark.parametrize("dt", list("dzsc"))
@pytest.mark.parametrize("m,n", [(100, 40), (256, 30), (500, 33), (1100, 20)])
def test_error_of_a_solve(dt, m, n):
    """Panels and chains against extended precision, where the terms beside the
    diagonal are small (diagonal in [1, 2], N(0, 1) right-hand sides): no more
    than four roundings of an X at its own size, of 0.425 u each in the root mean
    square (complex: a little more, its products are not exact), so 0.85 u and
    0.9 u.  And infinities stay where a product with the inverse of a diagonal
    block leaves them, in their own row."""
    if dt in "zc":
        m //= 2
    wide = np.clongdouble if dt in "zc" else np.longdouble
    L, B = W.problem(m, m, n, dt in "zc")
    cast = {"d": np.float64, "z": np.complex128, "s": np.float32, "c": np.complex64}[dt]
    r = np.random.default_rng(m)
    d = r.uniform(1, 2, m) + (1j * r.uniform(-0.5, 0.5, m) if dt in "zc" else 0)
    L = (np.tril(L, -1) / np.abs(np.tril(L, -1)).max() / m + np.diag(d)).astype(cast)
    B = (r.normal(size=(m, n)) + (1j * r.normal(size=(m, n)) if dt in "zc" else 0)).astype(cast)
    X = B.astype(wide) * wide(-0.75)
    for k in range(m):
        X[k] /= wide(L[k, k])
        X[k + 1:] -= np.outer(L[k + 1:, k].astype(wide), X[k])
    Ld, Bd = hs.to_colmajor(L), hs.to_colmajor(B)
    hs.trsm(Ld, Bd, -0.75, path=2)
    torch.cuda.synchronize()
    got = hs.from_colmajor(Bd).astype(wide)
    err = float(np.sqrt((np.abs(got - X) ** 2).sum() / (np.abs(X) ** 2).sum()))
    u = 2.0 ** (-53 if dt in "dz" else -24)
    assert err <= 0.5 * (1.8 if dt in "zc" else 1.7) * u, (dt, m, n, err / u)
    B[m // 2, 3] = np.inf
    B[m // 3, 5] = -np.inf
    Bd = hs.to_colmajor(B)
    hs.trsm(Ld, Bd, path=2)
    torch.cuda.synchronize()
    got = hs.from_colmajor(Bd)
    assert np.isinf(got[m // 2, 3]) and np.isinf(got[m // 3, 5]), (dt, m, n)
    assert np.isfinite(np.delete(got, [3, 5], 1)).all(), (dt, m, n)
    Bd = hs.to_colmajor(B)
    hs.trsm(Ld, Bd, path=2, unit=True)
    torch.cuda.synchronize()
    got = hs.from_colmajor(Bd)
    assert np.isinf(got[m // 2, 3]) and np.isinf(got[m // 3, 5]), (dt, m, n)
    assert np.isfinite(np.delete(got, [3, 5], 1)).all(), (dt, m, n)
    if dt in "ds":   # an infinite pivot: its X is 0, and what follows stands
        L[m // 2, m // 2] = np.inf
        B[m // 2, 3] = B[m // 3, 5] = 1
        Bd = hs.to_colmajor(B)
        hs.trsm(hs.to_colmajor(L), Bd, path=2)
        torch.cuda.synchronize()
        got = hs.from_colmajor(Bd)
        assert (got[m // 2] == 0).all() and np.isfinite(got).all(), (dt, m, n)


@pytest.mark.parametrize("n", [16400, 32768, 65541])
@pytest.mark.parametrize("dt,m", [("d", 65), ("d", 128), ("d", 129), ("d", 300), ("z", 40), ("z", 64), ("z", 150),
                                  ("s", 65), ("s", 256), ("s", 300), ("c", 64), ("c", 65), ("c", 200)])
def test_many_columns(dt, m, n):
    """Panels of many strips (several a workgroup, panels of another height from
    32768 columns): the bits of the same panels on a thousand columns."""
    span = {"d": 128, "z": 64, "s": 256, "c": 128}[dt]
    g = torch.Generator(device="cuda").manual_seed(m)
    Ls = torch.tril(_ints((m, m), dt, -3, 3, g), -1) / m + 1.5 * torch.eye(m, dtype=DT[dt], device="cuda")
    L = _colmajor(Ls)
    B = hs.colmajor(m, n, DT[dt], ld=m + 1)
    B.copy_(_ints((m, n), dt, -3, 3, g))
    X = hs.colmajor(m, n, DT[dt], ld=m + 1)
    X.copy_(B)
    hs.trsm(L, X, 0.5, path=2, unit=m == 129)
    for c in (0, n // 2, n - 1000):
        want = _colmajor(B[:, c:c + 1000])
        hs.trsm(L, want, 0.5, path=2, unit=m == 129, block_size=span if n >= 32768 and m > span else 0)
        torch.cuda.synchronize()
        assert torch.equal(X[:, c:c + 1000], want), (dt, m, n, c)


@pytest.mark.parametrize("dt,k", [("d", 100), ("z", 66), ("d", 200)])
def test_many_rows_from_the_right(dt, k):
    """The same where B is read at strides (X L^H = B)."""
    nr, g = 70001, torch.Generator(device="cuda").manual_seed(k)
    L = _colmajor(torch.tril(_ints((k, k), dt, -3, 3, g), -1) / k + 1.5 * torch.eye(k, dtype=DT[dt], device="cuda"))
    B = _ints((nr, k), dt, -3, 3, g)
    X, want = _colmajor(B), _colmajor(B.mH)
    hs.trsm_general(L, X, 0.5, side="R", uplo="L", trans="C")
    hs.trsm(L, want, 0.5)
    torch.cuda.synchronize()
    assert torch.equal(X, want.mH), (dt, k)


def test_more_columns_than_one_launch_of_strips():
    """2^27 columns and more: a workgroup of 512 for each strip of 16 would be
    more threads than a launch can have."""
    m, n = 65, (1 << 27) + 17
    Ls = torch.eye(m, device="cuda") + torch.diag(torch.ones(m - 1, device="cuda"), 1)   # row j: column j of L
    B = torch.ones((n, m), device="cuda").t()
    hs.trsm(Ls.t(), B)
    torch.cuda.synchronize()
    want = (1 - torch.arange(m, device="cuda") % 2).float()
    for c in range(0, n, 1 << 24):
        assert bool((B[:, c:c + (1 << 24)] == want[:, None]).all()), c


@pytest.mark.parametrize("dt", list("dzsc"))
def test_chains_that_overlap(dt):
    """Chains enqueued in turn on two streams with no wait between them, so that
    two run at once and workspace passes from stream to stream while in use: the
    bits of each alone."""
    g = torch.Generator(device="cuda").manual_seed(17)
    cases = []
    for m, n in ((1300, 40), (2049, 17), (700, 333), (3000, 100)):
        L = _colmajor(torch.tril(_ints((m, m), dt, -2, 2, g), -1) / m + 1.5 * torch.eye(m, dtype=DT[dt], device="cuda"))
        B = _colmajor(_ints((m, n), dt, -3, 3, g))
        alone = B.clone()
        hs.trsm(L, alone)
        torch.cuda.synchronize()
        cases.append((L, B, alone, [B.clone() for _ in range(6)]))
    sides = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for rep in range(6):
        for k, (L, _, _, X) in enumerate(cases):
            hs.trsm(L, X[rep], stream=sides[(rep + k) % 2])
    torch.cuda.synchronize()
    for k, (_, _, alone, X) in enumerate(cases):
        for rep, x in enumerate(X):
            assert torch.equal(x, alone), (dt, k, rep)
