"""The 2-D kernels with a launch per step or vector operation, on the small
grids that one launch otherwise solves: chosen by tgdk_ctx_one_launch (OFF),
and taken when the one-launch kernels find the chip held by others (CLOSED, the
gates closed from the start): the same bits, and the oracle's solution."""
import contextlib

import numpy as np
import pytest
import torch

import workloads as W
from oracle import gmres as OG, operators as O

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"


def tg():
    import paper_2005_03070_amd as m
    return m


def _t(a):
    return torch.tensor(a, device=DEV)


@contextlib.contextmanager
def launches(mode):
    L = tg()._lib
    tg().one_launch(mode)
    try:
        yield
    finally:
        tg().one_launch(L.ONE_LAUNCH_ON)


def _off_and_closed(f):
    """f's results with a launch per step; the same bits with closed gates."""
    L = tg()._lib
    with launches(L.ONE_LAUNCH_OFF):
        off = f()
    with launches(L.ONE_LAUNCH_CLOSED):
        closed = f()
    for a, b in zip(off, closed):
        assert torch.equal(a, b)
    return off


def _space(op, k, store=torch.float64, transpose=False):
    nx, ny = op.dims
    x, y = [np.arange(1, d + 1) / (d + 1) for d in (nx, ny)]
    cols = [np.outer(np.sin((1 + j // 3) * np.pi * y), np.sin((1 + j % 3) * np.pi * x)).reshape(-1) for j in range(k)]
    return tg().defl_from_basis(op, _t(np.stack(cols) + 1e-3 * W.rng(5).standard_normal((k, op.n))), store=store,
                                transpose=transpose)


def _residual(oop, x, b, transpose=False):
    A = O.apply_transpose if transpose else O.apply
    return np.linalg.norm(b - A(oop, x.cpu().numpy())) / np.linalg.norm(b)


# one tile, several, and a chip full (256 tiles)
@pytest.mark.parametrize("dims", [(63, 40), (130, 190), (1024, 1000)])
@pytest.mark.parametrize("precision,k", [("fp64", 0), ("fp64", 5), ("fp32_ir", 0), ("fp32_ir", 3)])
def test_bicgstab(dims, precision, k):
    beta = (10.0, 4.0)
    oop, op = O.const_cd(dims, beta), tg().Operator.const_cd(dims, beta, device=DEV)
    b = W.rhs(op.n, 11)
    space = _space(op, k, torch.float32 if precision == "fp32_ir" else torch.float64) if k else None
    budget = dict(ncyc=3, max_extra=0, maxit_cycle=25) if dims[0] == 1024 else dict(max_extra=100)
    reps = []

    def f():
        x, r = tg().solve(op, _t(b), defl=space, precision=precision, rtol=1e-10, **budget)
        reps.append((r[0].status, r[0].cycles, r[0].mvp_inner, r[0].relres_true))
        return [x]

    x, = _off_and_closed(f)
    assert reps[0] == reps[1]
    res = _residual(oop, x, b)
    if dims[0] != 1024:
        assert reps[0][0] == 0 and res <= 1.01e-10
    assert reps[0][3] == pytest.approx(res, rel=0.05)


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
def test_bicgstab_per_row_coefficients(transpose, precision):
    dims, beta = (130, 70), (8.0, 3.0)
    kc = W.kfield(dims, 3)
    oop, op = O.div_k(dims, kc, beta), tg().Operator.div_k(dims, _t(kc), beta)
    b = W.rhs(op.n, 13)
    space = _space(op, 6, transpose=transpose)
    x, = _off_and_closed(lambda: [tg().solve(op, _t(b), defl=space, precision=precision, rtol=1e-10, max_extra=100,
                                             transpose=transpose)[0]])
    assert _residual(oop, x, b, transpose) <= 1.01e-10


def test_bicgstab_batch_resume_and_fixed_scratch():
    dims, beta = (130, 100), (20.0, 5.0)
    oop, op = O.const_cd(dims, beta), tg().Operator.const_cd(dims, beta, device=DEV)
    B = np.stack([W.rhs(op.n, 40 + j) for j in range(5)])
    space = _space(op, 6)
    kw = dict(defl=space, rtol=1e-9, ncyc=8, max_extra=100)

    def f():
        X, reps = tg().solve(op, _t(B), **kw)
        Y, _ = tg().solve_noalloc(op, _t(B), **kw)
        z, r = tg().solve(op, _t(B[0]), max_cycles_call=3, **kw)
        z, r = tg().solve(op, _t(B[0]), x0=z, icyc0=r[0].cycles, nu0=r[0].nu0, **kw)
        assert all(q.status == 0 for q in reps) and r[0].status == 0
        return [X, Y, z]

    X, Y, z = _off_and_closed(f)
    assert torch.equal(X, Y)
    for j in range(5):
        assert _residual(oop, X[j], B[j]) <= 1.01e-9
    assert _residual(oop, z, B[0]) <= 1.01e-9


@pytest.mark.parametrize("s,precision,store", [(1, "fp64", torch.float64), (4, "fp64", torch.float64),
                                               (4, "fp32_ir", torch.float32), (8, "fp64", torch.float64)])
def test_idr(s, precision, store):
    dims, beta = (130, 100), (6.0, 3.0)
    oop, op = O.const_cd(dims, beta), tg().Operator.const_cd(dims, beta, device=DEV)
    b = W.rhs(op.n, 19)
    space, shadow = _space(op, 5, store), _t(W.shadow_draw(op.n, s, 7))
    start = _t(0.01 * W.rhs(op.n, 20))

    def f():
        x, r = tg().solve_idr(op, _t(b), s=s, shadow=shadow, defl=space, precision=precision, x0=start, rtol=1e-9,
                              max_extra=100)
        assert r.status == 0
        return [x]

    x, = _off_and_closed(f)
    r0 = np.linalg.norm(b - O.apply(oop, start.cpu().numpy())) / np.linalg.norm(b)
    assert _residual(oop, x, b) <= 1.01e-9 * min(1.0, r0)


@pytest.mark.parametrize("dims,m", [((7, 5), 20), ((130, 190), 33)])
def test_gmres(dims, m):
    oop, op = O.const_cd(dims, (5.0, 2.0)), tg().Operator.const_cd(dims, (5.0, 2.0), device=DEV)
    b = W.rhs(op.n, 12)
    x, = _off_and_closed(lambda: [tg().solve(op, _t(b), method="gmres", m3=m, rtol=1e-13, max_extra=2)[0]])
    xo, _ = OG.gmres_proj(oop, b, rtol=1e-13, m=m, maxcyc=2)
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-10 * np.linalg.norm(xo)  # as with one launch a cycle


# tiles of 64 rows with 47 and 48 of their 64 columns in the grid: launches per
# step, and one launch a cycle
@pytest.mark.parametrize("nx", [47, 48])
def test_gmres_on_narrow_grids(nx):
    dims = (nx, 8300)
    oop, op = O.const_cd(dims, (5.0, 2.0)), tg().Operator.const_cd(dims, (5.0, 2.0), device=DEV)
    b = W.rhs(op.n, 12)
    x, _ = tg().solve(op, _t(b), method="gmres", m3=12, rtol=1e-13, max_extra=2)
    xo, _ = OG.gmres_proj(oop, b, rtol=1e-13, m=12, maxcyc=2)
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-10 * np.linalg.norm(xo)
    off, = _off_and_closed(lambda: [tg().solve(op, _t(b), method="gmres", m3=12, rtol=1e-13, max_extra=2)[0]])
    assert torch.equal(x, off) == (nx == 47)  # (the sums of the one-launch steps have another order)


def test_coarse_setup():
    dims = (63, 66)
    oop, op = O.const_cd(dims, (4.0, 1.0)), tg().Operator.const_cd(dims, (4.0, 1.0), device=DEV)
    b = W.rhs(op.n, 9)

    def f():
        x, space, rep = tg().coarse_setup(op, _t(b), 40, 12, nev=8, rtolev=1e-9, rtol=1e-11, maxcyc=80)
        V, H = space.basis()
        return [x, V, _t(H)]

    x, V, H = _off_and_closed(f)
    assert _residual(oop, x, b) <= 1e-10
    V = V.cpu().numpy()
    np.testing.assert_allclose(V @ V.T, np.eye(len(V)), atol=1e-12)
    AV = np.stack([O.apply(oop, v) for v in V])
    np.testing.assert_allclose(H.cpu().numpy(), V @ AV.T, atol=1e-12 * O.norm1(oop))


def test_instances_of_two_sizes():
    ops = [tg().Operator.const_cd(d, (6.0, 3.0), device=DEV) for d in ((63, 40), (400, 300), (64, 64))]
    bs = [_t(W.rhs(o.n, 50 + j)) for j, o in enumerate(ops)]
    xs = _off_and_closed(lambda: tg().solve_instances(ops, None, bs, rtol=1e-9, max_extra=100)[0])
    for o, b, x in zip(ops, bs, xs):
        assert _residual(O.const_cd(o.dims, (6.0, 3.0)), x, b.cpu().numpy()) <= 1.01e-9


def test_one_launch_is_the_default_and_bad_modes_are_refused():
    L = tg()._lib
    op = tg().Operator.const_cd((63, 40), (6.0, 3.0), device=DEV)
    b = _t(W.rhs(op.n, 11))
    x = tg().solve(op, b, rtol=1e-9, max_extra=100)[0]
    with launches(L.ONE_LAUNCH_ON):
        y = tg().solve(op, b, rtol=1e-9, max_extra=100)[0]
    assert torch.equal(x, y)
    for mode in (-1, 3):
        with pytest.raises(L.TgdkError):
            tg().one_launch(mode)
