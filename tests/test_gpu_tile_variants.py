"""The one-launch kernels' tile heights in the variants that small grids do not
take: 32- and 64-row tiles over several workgroups with coefficient arrays, A^T
and float32 (IDR: 16-row tiles up to 256 of them, then 32, then 64; Arnoldi steps:
8 to 64), and float32 BiCGStab teams of 33 to 255 workgroups.

A short run is compared with the kernels of one launch per step: in the few
operator applications here an early rounding (2e-16, float32 6e-8) grows less
than 1e4-fold (BiCGStab and IDR: about tenfold in 6 iterations or 12
applications), so the iterates agree to 1e-11 (float32: 1e-3) of their norm."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import gmres as OG, operators as O

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"
AGREE = {"fp64": 1e-11, "fp32_ir": 1e-3}


def tg():
    import paper_2005_03070_amd as m
    return m


def _t(a):
    return torch.tensor(a, device=DEV)


def _operator(kind, dims):
    if kind == "const":
        return O.const_cd(dims, (6.0, 3.0)), tg().Operator.const_cd(dims, (6.0, 3.0), device=DEV)
    kc = W.kfield(dims, 3)
    return O.div_k(dims, kc, (6.0, 3.0)), tg().Operator.div_k(dims, _t(kc), (6.0, 3.0))


def _both(f):
    one = f()
    tg().one_launch(False)
    try:
        return one, f()
    finally:
        tg().one_launch(True)


def _residual(oop, x, b, transpose):
    return np.linalg.norm(b - (O.apply_transpose if transpose else O.apply)(oop, x.cpu().numpy())) / np.linalg.norm(b)


IDR = [((1024, 257), 2), ((1024, 257), 4), ((1024, 257), 8),   # 32 rows
       ((1024, 513), 2), ((1024, 513), 4)]                     # 64 rows


@pytest.mark.parametrize("kind,transpose,precision", [("div_k", False, "fp64"), ("div_k", True, "fp64"),
                                                      ("div_k", True, "fp32_ir"), ("const", False, "fp32_ir"),
                                                      ("const", True, "fp64")])
@pytest.mark.parametrize("dims,s", IDR)
def test_idr_short_run(dims, s, kind, transpose, precision):
    oop, op = _operator(kind, dims)
    b, shadow = W.rhs(op.n, 23), _t(W.shadow_draw(op.n, s, 9))
    start = _t(0.01 * W.rhs(op.n, 24))
    reps = []

    def f():
        x, r = tg().solve_idr(op, _t(b), s=s, shadow=shadow, x0=start, precision=precision, rtol=1e-9, ncyc=1,
                              max_extra=0, maxit_cycle=10, transpose=transpose)
        reps.append(r)
        return x

    one, off = _both(f)
    assert reps[0].mvp_inner == reps[1].mvp_inner and reps[0].cycle_mvps == reps[1].cycle_mvps
    assert torch.linalg.norm(one - off) <= AGREE[precision] * torch.linalg.norm(off)
    assert reps[0].relres_true == pytest.approx(_residual(oop, one, b, transpose), rel=1e-6)


@pytest.mark.parametrize("dims,s,transpose", [((1024, 257), 4, True), ((1024, 513), 4, False),
                                              ((1024, 257), 8, False)])
def test_idr_with_coefficient_arrays_converges(dims, s, transpose):
    oop, op = _operator("div_k", dims)
    b, shadow = W.rhs(op.n, 23), _t(W.shadow_draw(op.n, s, 9))
    x, rep = tg().solve_idr(op, _t(b), s=s, shadow=shadow, rtol=1e-7, max_extra=200, transpose=transpose)
    assert rep.status == 0 and _residual(oop, x, b, transpose) <= 1.01e-7
    assert rep.mvp_inner == sum(rep.cycle_mvps)


@pytest.mark.parametrize("dims", [(65, 130), (257, 500), (257, 1100), (1000, 1000)])  # 8, 16, 32, 64 rows
@pytest.mark.parametrize("transpose", [False, True])
def test_gmres_with_coefficient_arrays(dims, transpose):
    oop, op = _operator("div_k", dims)
    b = W.rhs(op.n, 12)
    x, _ = tg().solve(op, _t(b), method="gmres", m3=12, rtol=1e-13, max_extra=2, transpose=transpose)
    xo, _ = OG.gmres_proj(oop, b, rtol=1e-13, m=12, maxcyc=2, transpose=transpose)
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-10 * np.linalg.norm(xo)  # as test_gpu_arnoldi2d's


@pytest.mark.parametrize("dims", [(600, 500), (1000, 700), (1023, 900)])  # 80, 176, 240 workgroups
@pytest.mark.parametrize("kind,transpose,k", [("const", False, 0), ("const", False, 3), ("div_k", True, 3)])
def test_bicgstab_float32_short_run(dims, kind, transpose, k):
    oop, op = _operator(kind, dims)
    b = W.rhs(op.n, 11)
    space = tg().defl_from_basis(op, _t(W.rng(5).standard_normal((k, op.n))), store=torch.float32,
                                 transpose=transpose) if k else None
    reps = []

    def f():
        x, r = tg().solve(op, _t(b), defl=space, precision="fp32_ir", rtol=1e-10, ncyc=2, max_extra=0, maxit_cycle=4,
                          transpose=transpose)
        reps.append(r[0])
        return x

    one, off = _both(f)
    assert (reps[0].cycles, reps[0].mvp_inner, reps[0].mvp_boundary) == (reps[1].cycles, reps[1].mvp_inner,
                                                                        reps[1].mvp_boundary)
    assert torch.linalg.norm(one - off) <= AGREE["fp32_ir"] * torch.linalg.norm(off)
    assert reps[0].relres_true == pytest.approx(_residual(oop, one, b, transpose), rel=1e-6)


# the vector kernels of IDR past the largest grid that one launch takes
@pytest.mark.parametrize("kind,precision,s", [("const", "fp64", 4), ("div_k", "fp64", 2), ("const", "fp32_ir", 4)])
def test_idr_past_the_chip(kind, precision, s):
    dims = (1024, 1025)
    oop, op = _operator(kind, dims)
    b, shadow = W.rhs(op.n, 23), _t(W.shadow_draw(op.n, s, 9))
    x, r = tg().solve_idr(op, _t(b), s=s, shadow=shadow, precision=precision, rtol=1e-9, ncyc=2, max_extra=0,
                          maxit_cycle=40)
    assert r.mvp_inner == sum(r.cycle_mvps) > 0
    assert r.relres_true == pytest.approx(_residual(oop, x, b, False), rel=1e-6) and r.relres_true < 1.0


# grids one tile past the largest that one launch takes (256 workgroups)
@pytest.mark.parametrize("dims", [(64 * 256, 8), (64 * 256 + 1, 8)])
@pytest.mark.parametrize("k", [0, 4])
def test_bicgstab_at_the_largest_team(dims, k):
    oop, op = O.const_cd(dims, (1.0, 0.5)), tg().Operator.const_cd(dims, (1.0, 0.5), device=DEV)
    b = W.rhs(op.n, 11)
    space = tg().defl_from_basis(op, _t(W.rng(5).standard_normal((k, op.n)))) if k else None
    f = lambda: tg().solve(op, _t(b), defl=space, rtol=1e-10, ncyc=2, max_extra=0, maxit_cycle=6)[0]
    one, off = _both(f)
    assert torch.equal(one, off) == (dims[0] > 64 * 256)
    assert torch.linalg.norm(one - off) <= 1e-11 * torch.linalg.norm(off)
    r = tg().solve(op, _t(b), defl=space, rtol=1e-10, ncyc=2, max_extra=0, maxit_cycle=6)[1][0]
    assert r.relres_true == pytest.approx(_residual(oop, one, b, False), rel=1e-6)
