"""Solves from several threads at once, each on its own stream (hence context):
one-launch solves that each want the whole chip, small ones, GMRES cycles and
spaces made and dropped, with the results that the calls give by themselves.
(Where a launch finds the chip held it waits, or after a second takes the
launches per step: then the bits may differ, the tolerance holds.)"""
import threading

import pytest
import torch

import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"


def test_concurrent_solves():
    import paper_2005_03070_amd as tg
    dims = [(1023, 1023), (63, 63), (511, 511), (300, 200)]
    rhs = [torch.tensor(W.rhs(d[0] * d[1], 60 + j), device=DEV) for j, d in enumerate(dims)]
    basis = [torch.tensor(W.rng(j).standard_normal((6, d[0] * d[1])), device=DEV) for j, d in enumerate(dims)]
    torch.cuda.synchronize()

    def work(j, out):
        with torch.cuda.stream(torch.cuda.Stream()):
            op = tg.Operator.const_cd(dims[j], (20.0, 5.0), device=DEV)
            for _ in range(3):
                space = tg.defl_from_basis(op, basis[j])
                x, r = tg.solve(op, rhs[j], defl=space, rtol=1e-8, ncyc=10, max_extra=100)
                y, s = tg.solve_idr(op, rhs[j], s=4, defl=space, rtol=1e-7, ncyc=10, max_extra=100, seed=j)
                z, _ = tg.solve(op, rhs[j], method="gmres", m3=20, rtol=1e-12, max_extra=2)
                out.append((x, r[0], y, s, z))
            torch.cuda.synchronize()

    alone = []
    for j in range(4):
        got = []
        work(j, got)
        alone.append(got[0])
    got = [[] for _ in dims]
    threads = [threading.Thread(target=work, args=(j, got[j])) for j in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
        assert not t.is_alive()
    for j, d in enumerate(dims):
        op = tg.Operator.const_cd(d, (20.0, 5.0), device=DEV)
        norm = torch.linalg.norm(rhs[j])
        assert len(got[j]) == 3
        for x, r, y, s, z in got[j]:
            assert r.status == 0 and s.status == 0
            assert torch.linalg.norm(rhs[j] - op.apply(x)) <= 1.01e-8 * norm
            assert torch.linalg.norm(rhs[j] - op.apply(y)) <= 1.01e-7 * norm
            assert torch.linalg.norm(z - alone[j][4]) <= 1e-9 * torch.linalg.norm(z)
