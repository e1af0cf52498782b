"""Instances of different sizes in one call: each has the bits of its own call,
whatever else is in the call and in whichever order (grids of one tile, of a
few, of a whole chip and past it), and a call costs no more than its parts."""
import time

import pytest
import torch

import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"


def tg():
    import paper_2005_03070_amd as m
    return m


def _instances(dims):
    ops = [tg().Operator.const_cd(d, (min(40.0, 0.5 * min(d)), 1.0), device=DEV) for d in dims]
    return ops, [torch.tensor(W.rhs(o.n, 300 + j), device=DEV) for j, o in enumerate(ops)]


KW = dict(rtol=1e-8, ncyc=10, max_extra=100)


@pytest.mark.parametrize("dims", [
    [(63, 40), (1023, 1000), (64, 64), (130, 70), (33, 65), (500, 300), (20, 9)],   # all fit the chip
    [(63, 40), (1100, 1000), (130, 70), (20, 9)],                                   # one is past 256 tiles
    [(1100, 1000), (40, 30), (1030, 1025)],                                         # two are
])
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
def test_mixed_sizes_equal_solo_bits(dims, precision):
    ops, bs = _instances(dims)
    kw = dict(KW, precision=precision)
    if precision == "fp32_ir":  # (three cycles: float32 cycles alone need not converge on every grid)
        kw.update(ncyc=3, max_extra=0, maxit_cycle=40)
    xs, reps = tg().solve_instances(ops, [None] * len(ops), bs, **kw)
    for o, b, x, r in zip(ops, bs, xs, reps):
        xj, rj = tg().solve(o, b, **kw)
        assert torch.equal(x, xj), o.dims
        assert (r.status, r.cycles, r.mvp_inner, r.relres_true) == (rj[0].status, rj[0].cycles, rj[0].mvp_inner,
                                                                    rj[0].relres_true)
        assert precision == "fp32_ir" or r.status == 0


def test_spaces_of_two_types_are_refused_before_anything_runs():
    ops, bs = _instances([(63, 40), (130, 70)])
    spaces = [tg().defl_from_basis(o, torch.tensor(W.rng(j).standard_normal((3, o.n)), device=DEV), store=t)
              for j, (o, t) in enumerate(zip(ops, (torch.float64, torch.float32)))]
    with pytest.raises(tg()._lib.TgdkError) as e:
        tg().solve_instances(ops, spaces, bs, **KW)
    assert e.value.code == tg()._lib.E_INVALID


def test_a_large_system_does_not_slow_the_small_ones():
    """One 1023^2 system and 96 of 63^2: with teams of the large one's size for
    all, the small ones took turns on 256 workgroups (about 3 times the two
    calls by themselves); in groups the call takes as long as they do."""
    ops, bs = _instances([(1023, 1023)] + [(63, 63)] * 96)

    def best(f):
        f()
        t = []
        for _ in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    whole = best(lambda: tg().solve_instances(ops, [None] * 97, bs, **KW))
    parts = best(lambda: tg().solve(ops[0], bs[0], **KW)) + best(
        lambda: tg().solve_instances(ops[1:], [None] * 96, bs[1:], **KW))
    assert whole <= 1.5 * parts


@pytest.mark.parametrize("store", [torch.float64, torch.float32])
def test_spaces_past_what_one_or_two_tiles_take(store):
    """128 and 129 float64 vectors on one and two tiles (one launch, and the step
    kernel), 129 on three, alone and in one call: each has the bits of its own
    call, and of a launch per step exactly where that is chosen."""
    specs = [((63, 40), 128), ((63, 40), 129), ((64, 64), 129), ((64, 128), 129), ((65, 60), 128), ((64, 129), 129)]
    ops, bs = _instances([d for d, _ in specs])
    spaces = [tg().defl_from_basis(o, torch.tensor(W.rng(j).standard_normal((k, o.n)), device=DEV), store=store)
              for j, (o, (_, k)) in enumerate(zip(ops, specs))]
    # (three iterations, where the two paths differ in the last bits)
    kw = dict(rtol=1e-12, ncyc=3, max_extra=0, maxit_cycle=1)
    xs, reps = tg().solve_instances(ops, spaces, bs, **kw)
    for o, (d, k), b, sp, x in zip(ops, specs, bs, spaces, xs):
        assert torch.equal(tg().solve(o, b, defl=sp, **kw)[0], x), (d, k)
        tg().one_launch(False)
        try:
            off = tg().solve(o, b, defl=sp, **kw)[0]
        finally:
            tg().one_launch(True)
        stepped = store == torch.float64 and k > 128 and d != (64, 129)
        assert torch.equal(off, x) == stepped, (d, k)
        assert torch.linalg.norm(off - x) <= 1e-10 * torch.linalg.norm(off)
