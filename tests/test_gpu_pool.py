"""Memory that contexts keep between calls: bounded, given back, and never
read before it is written (results do not depend on what a block held)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"


def tg():
    import paper_2005_03070_amd as m
    return m


def test_kept_memory_is_bounded_and_given_back():
    """Spaces of many sizes, 12 GB in all, made and dropped: at most the
    pool's 2 GiB stay taken (plus 64 MiB for the driver's own granules), and
    idle blocks leave it: after 200 small requests nothing large is held."""
    small = tg().Operator.const_cd((15, 15), (1.0, 0.0), device=DEV)
    Ws = torch.tensor(W.rng(1).standard_normal((2, small.n)), device=DEV)
    tg().defl_from_basis(small, Ws)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for i in range(12):
        op = tg().Operator.const_cd((1023, 255 + 48 * i), (1.0, 0.0), device=DEV)
        Wt = torch.randn((64, op.n), dtype=torch.float64, device=DEV)
        space = tg().defl_from_basis(op, Wt)
        del space, op, Wt
    torch.cuda.empty_cache()
    assert torch.cuda.mem_get_info()[0] >= free0 - (2 << 30) - (64 << 20)
    for _ in range(200):
        tg().defl_from_basis(small, Ws)
    torch.cuda.synchronize()
    # (solve and partial-sum workspaces of the context stay: a few MB here)
    assert torch.cuda.mem_get_info()[0] >= free0 - (256 << 20)


def test_results_do_not_depend_on_a_blocks_old_contents():
    """The same calls with blocks fresh from the driver, and with blocks full
    of another problem's values (huge and NaN), give the same bits."""
    def calls():
        op = tg().Operator.const_cd((127, 95), (30.0, 5.0), device=DEV)
        b = torch.tensor(W.rhs(op.n, 3), device=DEV)
        s = tg().TwoGridSolver(op, m=24, k=6, maxcyc=4)
        x0 = s.setup(b)
        V, H = s.defl.basis()
        x, _ = tg().solve(op, b, x0=x0, defl=s.defl, method="gmres", m3=20, rtol=1e-12, max_extra=3)
        y, _ = tg().solve_idr(op, b, s=3, x0=x0, defl=s.defl, rtol=1e-8)
        m = s.defl.minres()
        z, rep = s.defl.improve(20, nev=4, tol=1e-12, maxcyc=2)
        return [x0, V, torch.tensor(H), x, y, m.basis()[0], z.basis()[0]]

    first = calls()
    op = tg().Operator.const_cd((127, 95), (30.0, 5.0), device=DEV)
    bad = torch.full((24, op.n), float("nan"), dtype=torch.float64, device=DEV)
    for k in (6, 7, 12, 24):   # blocks of the sizes the calls take, filled with NaN
        with pytest.raises(Exception):
            tg().defl_from_basis(op, bad[:k].contiguous())
    for a, b in zip(first, calls()):
        assert torch.equal(a, b)
