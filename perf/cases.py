"""Performance cases: the solves that programs have this library do, through
its Python binding.

Each case is a dict of plain values.  ``prepare`` makes what a program holds
before the call (matrices on the GPU, a batch plan), ``run`` is one pass
through the public entry points, ``work`` the bytes and operations that the
pass cannot do without, and ``exact`` its result in 64 bits from torch alone.

Kinds of case:

* ``trsm``: one solve ``X = alpha inv(L) B``, real or complex, double or
  single.  Solves are in place, as the entry point defines them, so a repeated
  pass solves the previous pass's result again; the diagonal of L lies
  in [1, 2] and |alpha| <= 1, so values stay finite.
* ``mixed``: updates on the FP32 matrix cores, with refinement steps.
* ``general``: the other sides, triangles and operators.
* ``potrf``: Cholesky factorization of a copy of A.
* ``plan``: a prepared batch of small problems, executed again and again.
* ``served``: one batch of mixed sizes handed over as it comes (no plan), with
  the size distribution of the serving workload.

L's strict lower triangle is U(-1, 1)/m, its diagonal U(1, 2) (complex: the
imaginary parts U(-1, 1)/m and U(-1/2, 1/2)) and B is N(0, 1), the
distributions of the library's workloads.  The triangle that must not be read
holds other random numbers.
"""
import math
import random

import torch

import paper_2608_25469_amd as hsma

DTYPES = {"d": torch.float64, "z": torch.complex128, "s": torch.float32, "c": torch.complex64}
REAL_OF = {"d": torch.float64, "z": torch.float64, "s": torch.float32, "c": torch.float32}
ESIZE = {"d": 8, "z": 16, "s": 4, "c": 8}

# The largest listed solve, in multiply-add pairs of real numbers.
MOST_FLOPS = 16384.0 ** 3


def listed():
    return [
        # The smallest call in daily use: one 32 x 32 solve, bound by latency.
        dict(name="trsm_d_32", kind="trsm", dtype="d", m=32, n=32, lda=32, ldb=32, unit=False, alpha=1.0),
        # An ordinary mid-sized solve with sizes and leading dimensions of no
        # special form.
        dict(name="trsm_d_500x300", kind="trsm", dtype="d", m=500, n=300, lda=517, ldb=500, unit=False, alpha=-0.75),
        # The same in complex data, with a unit diagonal (an LU factor's L).
        dict(name="trsm_z_1000x257", kind="trsm", dtype="z", m=1000, n=257, lda=1003, ldb=1000, unit=True, alpha=1.0),
        # A tall factor with a few hundred right-hand sides.
        dict(name="trsm_d_4096x256", kind="trsm", dtype="d", m=4096, n=256, lda=4096, ldb=4096, unit=False, alpha=1.0),
        # The largest real and complex solves the library is quoted on.
        dict(name="trsm_d_16384", kind="trsm", dtype="d", m=16384, n=16384, lda=16384, ldb=16384, unit=False, alpha=-1.0),
        dict(name="trsm_z_8192", kind="trsm", dtype="z", m=8192, n=8192, lda=8192, ldb=8192, unit=False, alpha=-1.0),
        # Single precision.
        dict(name="trsm_s_4096", kind="trsm", dtype="s", m=4096, n=4096, lda=4096, ldb=4096, unit=False, alpha=1.0),
        # Mixed precision with one refinement step.
        dict(name="mixed_d_8192x4096", kind="mixed", dtype="d", m=8192, n=4096, lda=8192, ldb=8192, steps=1, alpha=1.0),
        # X op(A) = B with the upper triangle stored, as after an LU
        # factorization from the other side; ragged sizes.
        dict(name="general_d_RUT_2500x1777", kind="general", dtype="d", side="R", uplo="U", trans="T", m=2500, n=1777,
             lda=1777, ldb=2500, unit=False, alpha=1.0),
        # Cholesky factorization.
        dict(name="potrf_d_4096", kind="potrf", dtype="d", m=4096, lda=4096),
        # 10 000 small complex problems, m, n ~ U{8..64}, in one plan.
        dict(name="plan_z_10000", kind="plan", dtype="z", count=10000, lo=8, hi=64, shapes=1),
        # 96 requests of the serving mix in one call: m log-uniform in
        # [8, 4096], n in [1, 512], 30 % complex.
        dict(name="served_96", kind="served", count=96, m_hi=4096, n_hi=512, shapes=4),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _ld(rng, m):
    """Tight, rounded up, or odd leading dimensions."""
    return m + rng.choice([0, 0, 0, 1, 3, (-m) % 16])


def draw(rng):
    kind = rng.choices(["trsm", "mixed", "general", "potrf", "plan", "served"], [8, 1, 2, 2, 2, 1])[0]
    if kind == "trsm":
        dt = rng.choice(["d", "d", "z", "z", "s", "c"])
        while True:
            m = _log_int(rng, 8, 16384 if dt in "ds" else 8192)
            n = _log_int(rng, 1, 16384 if dt in "ds" else 8192)
            if float(m) * m * n * (4 if dt in "zc" else 1) <= MOST_FLOPS:
                break
        return dict(kind=kind, dtype=dt, m=m, n=n, lda=_ld(rng, m), ldb=_ld(rng, m), unit=rng.random() < 0.25,
                    alpha=rng.choice([1.0, 1.0, -1.0, 0.5]))
    if kind == "mixed":
        m = _log_int(rng, 1024, 8192)
        return dict(kind=kind, dtype="d", m=m, n=_log_int(rng, 64, 4096), lda=_ld(rng, m), ldb=_ld(rng, m),
                    steps=rng.choice([0, 1, 1, 2]), alpha=1.0)
    if kind == "general":
        dt = rng.choice(["d", "d", "z", "s"])
        m, n, side = _log_int(rng, 16, 6000), _log_int(rng, 16, 6000), rng.choice("LR")
        k = m if side == "L" else n
        return dict(kind=kind, dtype=dt, side=side, uplo=rng.choice("LU"), trans=rng.choice("NTC"), m=m, n=n,
                    lda=_ld(rng, k), ldb=_ld(rng, m), unit=rng.random() < 0.25, alpha=rng.choice([1.0, -0.5]))
    if kind == "potrf":
        dt = rng.choice("dz")
        m = _log_int(rng, 32, 12000 if dt == "d" else 6000)
        return dict(kind=kind, dtype=dt, m=m, lda=_ld(rng, m))
    if kind == "plan":
        lo = _log_int(rng, 2, 24)
        return dict(kind=kind, dtype=rng.choice("dz"), count=_log_int(rng, 300, 20000), lo=lo,
                    hi=rng.randint(max(lo, 8), 64), shapes=rng.randrange(1 << 20))
    return dict(kind=kind, count=_log_int(rng, 8, 128), m_hi=_log_int(rng, 256, 4096), n_hi=_log_int(rng, 16, 512),
                shapes=rng.randrange(1 << 20))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _uniform(shape, dt, g):
    """U(-1, 1) in every component."""
    t = torch.empty(shape, dtype=DTYPES[dt], device="cuda")
    (torch.view_as_real(t) if t.is_complex() else t).uniform_(-1.0, 1.0, generator=g)
    return t


def _diagonal(m, dt, g):
    d = torch.empty(m, dtype=REAL_OF[dt], device="cuda").uniform_(1.0, 2.0, generator=g)
    if dt in "zc":
        im = torch.empty(m, dtype=REAL_OF[dt], device="cuda").uniform_(-0.5, 0.5, generator=g)
        d = torch.complex(d, im)
    return d


def _triangle(m, ld, dt, g):
    """m x m, column-major with leading dimension ld; the same distribution on
    both sides of the diagonal, so that either triangle can be the stored one."""
    store = _uniform((m, ld), dt, g)
    store /= m
    A = store[:, :m].t()
    A.diagonal().copy_(_diagonal(m, dt, g))
    return A


def _rhs(m, n, ld, dt, g):
    store = torch.empty((n, ld), dtype=DTYPES[dt], device="cuda")
    (torch.view_as_real(store) if store.is_complex() else store).normal_(generator=g)
    return store[:, :m].t()


def _spd(case, seed):
    """Hermitian positive definite: a scaled random Hermitian matrix (spectral
    norm below 1.2) on a diagonal of U(2, 3)."""
    dt, m, g = case["dtype"], case["m"], _gen(seed)
    store = torch.empty((m, case["lda"]), dtype=DTYPES[dt], device="cuda")
    R = _uniform((m, m), dt, g)
    A = store[:, :m].t()
    A.copy_((R + R.mH) * (0.5 / math.sqrt(m)))
    d = torch.empty(m, dtype=REAL_OF[dt], device="cuda").uniform_(2.0, 3.0, generator=g)
    A.diagonal().copy_(d)
    return A


def _plan_shapes(case):
    r = random.Random(case["shapes"])
    return [(r.randint(case["lo"], case["hi"]), r.randint(case["lo"], case["hi"])) for _ in range(case["count"])]


def _served_shapes(case):
    """(m, n, dtype, alpha) of each request."""
    r = random.Random(case["shapes"])
    out = []
    for _ in range(case["count"]):
        m, n = _log_int(r, 8, case["m_hi"]), _log_int(r, 1, case["n_hi"])
        out.append((m, n, "z" if r.random() < 0.3 else "d", r.choice([1.0, -1.0, 0.5, -0.75])))
    return out


def _offsets(sizes, align):
    offs, pos = [], 0
    for k in sizes:
        offs.append(pos)
        pos += (k + align - 1) // align * align
    return offs, max(pos, 1)


def _pools(shapes, dt, g):
    """All L's and all B's of one data type, each in one pool with every
    matrix at a 256-byte boundary.  Returns the pools and the views."""
    al = 256 // ESIZE[dt]
    lo, lsz = _offsets([m * m for m, _ in shapes], al)
    bo, bsz = _offsets([m * n for m, n in shapes], al)
    pl = _uniform((lsz,), dt, g)
    pb = torch.empty(bsz, dtype=DTYPES[dt], device="cuda")
    (torch.view_as_real(pb) if pb.is_complex() else pb).normal_(generator=g)
    if shapes:
        ms = torch.tensor([m for m, _ in shapes], device="cuda")
        start = torch.tensor(lo, device="cuda")
        room = torch.tensor(lo[1:] + [lsz], device="cuda") - start
        pl /= torch.repeat_interleave(ms, room)
        # Diagonal entry k of problem i is at start_i + k (m_i + 1).
        which = torch.repeat_interleave(torch.arange(len(shapes), device="cuda"), ms)
        first = torch.cumsum(ms, 0) - ms
        k = torch.arange(which.numel(), device="cuda") - first[which]
        pl[start[which] + k * (ms[which] + 1)] = _diagonal(which.numel(), dt, g)
    vl = [pl[o:o + m * m].view(m, m).t() for o, (m, _) in zip(lo, shapes)]
    vb = [pb[o:o + m * n].view(n, m).t() for o, (m, n) in zip(bo, shapes)]
    return pl, pb, vl, vb


def _served_pools(case, seed):
    shapes, g = _served_shapes(case), _gen(seed)
    pools = {}
    for dt in "dz":
        pools[dt] = _pools([(m, n) for m, n, d, _ in shapes if d == dt], dt, g)
    return shapes, pools


# |alpha| < 1, so that plans executed again and again stay finite.
PLAN_ALPHA = {"d": 0.875, "z": complex(0.8, 0.4)}


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("trsm", "mixed"):
        g = _gen(seed)
        return dict(case=case, L=_triangle(case["m"], case["lda"], case["dtype"], g),
                    B=_rhs(case["m"], case["n"], case["ldb"], case["dtype"], g))
    if kind == "general":
        g = _gen(seed)
        k = case["m"] if case["side"] == "L" else case["n"]
        return dict(case=case, A=_triangle(k, case["lda"], case["dtype"], g),
                    B=_rhs(case["m"], case["n"], case["ldb"], case["dtype"], g))
    if kind == "potrf":
        A = _spd(case, seed)
        W = hsma.colmajor(case["m"], case["m"], A.dtype, ld=case["lda"])
        return dict(case=case, A=A, W=W)
    if kind == "plan":
        pl, pb, vl, vb = _pools(_plan_shapes(case), case["dtype"], _gen(seed))
        plan = hsma.BatchPlan([(L, B, PLAN_ALPHA[case["dtype"]]) for L, B in zip(vl, vb)])
        return dict(case=case, plan=plan, pool_l=pl, out=pb)
    shapes, pools = _served_pools(case, seed)
    nxt = {dt: iter(zip(pools[dt][2], pools[dt][3])) for dt in "dz"}
    probs = [hsma.problem_struct(*next(nxt[dt]), alpha) for _, _, dt, alpha in shapes]
    return dict(case=case, probs=probs, pools=pools, out=[pools[dt][1] for dt in "dz"])


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "trsm":
        return hsma.trsm(state["L"], state["B"], alpha=c["alpha"], unit=c["unit"])
    if kind == "mixed":
        return hsma.trsm(state["L"], state["B"], alpha=c["alpha"], mixed=True, refine_steps=c["steps"])
    if kind == "general":
        return hsma.trsm_general(state["A"], state["B"], alpha=c["alpha"], side=c["side"], uplo=c["uplo"],
                                 trans=c["trans"], unit=c["unit"])
    if kind == "potrf":
        state["W"].copy_(state["A"])   # the factorization is in place; the program keeps A
        return hsma.potrf(state["W"])
    if kind == "plan":
        state["plan"].execute()
        return state["out"]
    hsma.trsm_batched(state["probs"])
    return state["out"]


# ---------------------------------------------------------------------------
# Work and exact results
# ---------------------------------------------------------------------------

def _solve_work(m, n, dt):
    """m^2 n flops in real data and 4 m^2 n + 2 m n in complex; the triangle
    read once, B read and written once."""
    fl = 4.0 * m * m * n + 2.0 * m * n if dt in "zc" else float(m) * m * n
    return ESIZE[dt] * (m * (m + 1) / 2.0 + 2.0 * m * n), fl


def work(case):
    kind = case["kind"]
    if kind == "potrf":
        m = case["m"]
        # The copy of A (read and written) and the triangle read and written.
        by = ESIZE[case["dtype"]] * (2.0 * m * m + m * (m + 1.0))
        return {"bytes": by, "flops": m ** 3 / 3.0 * (4 if case["dtype"] == "z" else 1)}
    if kind == "general":
        k, o = (case["m"], case["n"]) if case["side"] == "L" else (case["n"], case["m"])
        each = [_solve_work(k, o, case["dtype"])]
    elif kind == "plan":
        each = [_solve_work(m, n, case["dtype"]) for m, n in _plan_shapes(case)]
    elif kind == "served":
        each = [_solve_work(m, n, dt) for m, n, dt, _ in _served_shapes(case)]
    else:
        by, fl = _solve_work(case["m"], case["n"], case["dtype"])
        # A refinement step is a residual (one triangular product) and a
        # second solve.
        each = [(by, fl * (1 + 2 * case.get("steps", 0)))]
    return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}


def _solve(L, B, alpha, unit, upper=False):
    """alpha inv(T) B in 64 bits for the stated triangle T of L."""
    dt = torch.complex128 if L.is_complex() else torch.float64
    T = L.to(dt)
    T = T.triu() if upper else T.tril()
    return torch.linalg.solve_triangular(T, alpha * B.to(dt), upper=upper, unitriangular=unit)


def _padded(vl, vb, alphas):
    """Many small problems in one batched solve, each padded with an identity
    block to the largest size."""
    m, n = max(v.shape[0] for v in vb), max(v.shape[1] for v in vb)
    T = torch.eye(m, dtype=vl[0].dtype).repeat(len(vl), 1, 1)
    R = torch.zeros((len(vl), m, n), dtype=vb[0].dtype)
    for i, (L, B, a) in enumerate(zip(vl, vb, alphas)):
        k = L.shape[0]
        T[i, :k, :k] = L.tril()
        R[i, :k, :B.shape[1]] = a * B
    X = torch.linalg.solve_triangular(T, R, upper=False)
    return [X[i, :B.shape[0], :B.shape[1]] for i, B in enumerate(vb)]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("trsm", "mixed"):
        s = prepare(case, seed)
        return _solve(s["L"], s["B"], case["alpha"], case.get("unit", False))
    if kind == "general":
        s = prepare(case, seed)
        A = s["A"].triu() if case["uplo"] == "U" else s["A"].tril()
        A = {"N": A, "T": A.mT, "C": A.mH}[case["trans"]]
        upper = (case["uplo"] == "U") == (case["trans"] == "N")
        if case["side"] == "L":
            return _solve(A, s["B"], case["alpha"], case["unit"], upper)
        return _solve(A.mT, s["B"].mT, case["alpha"], case["unit"], not upper).mT
    if kind == "potrf":
        A = _spd(case, seed)
        return torch.linalg.cholesky(A.tril() + A.tril(-1).mH) + A.triu(1)
    if kind == "plan":
        _, pb, vl, vb = _pools(_plan_shapes(case), case["dtype"], _gen(seed))
        out = pb.cpu()
        cl, cb = [v.cpu() for v in vl], [v.cpu() for v in vb]
        al = 256 // ESIZE[case["dtype"]]
        offs, _ = _offsets([v.numel() for v in cb], al)
        for o, X in zip(offs, _padded(cl, cb, [PLAN_ALPHA[case["dtype"]]] * len(cl))):
            out[o:o + X.numel()] = X.t().reshape(-1)
        return out
    shapes, pools = _served_pools(case, seed)
    out = []
    for dt in "dz":
        _, pb, vl, vb = pools[dt]
        res = pb.clone()
        mine = [s for s in shapes if s[2] == dt]
        offs, _ = _offsets([m * n for m, n, _, _ in mine], 256 // ESIZE[dt])
        for o, (m, n, _, a), L, B in zip(offs, mine, vl, vb):
            res[o:o + m * n] = _solve(L, B, a, False).t().reshape(-1)
        out.append(res)
    return out
