"""Arnoldi steps in one launch (kernels_arnoldi2d.hip) at the edges of tiles,
teams and column groups: GMRES cycles and coarse GMRES-DR against the oracle.

One cycle's iterate differs between two orders of summation by rounding times
the condition of the small least-squares problem; the existing one-cycle test
holds 1e-10 at 47 x 31, and so do these."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import direct as ODS, gmres as OG, operators as O

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"


def tg():
    import paper_2005_03070_amd as m
    return m


# one workgroup, its edges, thin grids, 8- to 64-row tiles, 32 and 33 workgroups,
# 256 tiles of 64 x 64, and one row more (the launch-per-step path)
@pytest.mark.parametrize("dims,m", [((7, 5), 20), ((64, 8), 9), ((65, 9), 17), ((3, 300), 33), ((300, 3), 8),
                                    ((64, 256), 40), ((64, 264), 40), ((130, 190), 65), ((257, 1100), 12),
                                    ((1024, 1024), 6), ((1024, 1025), 6), ((90, 70), 128), ((90, 70), 140)])
def test_gmres_cycles_match_oracle(dims, m):
    beta = (5.0, 2.0)
    oop = O.const_cd(dims, beta)
    b = W.rhs(oop.n, 12)
    op = tg().Operator.const_cd(dims, beta, device=DEV)
    x, reps = tg().solve(op, torch.tensor(b, device=DEV), method="gmres", m3=m, rtol=1e-13, max_extra=2)
    xo, orep = OG.gmres_proj(oop, b, rtol=1e-13, m=m, maxcyc=2)
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-10 * np.linalg.norm(xo)


@pytest.mark.parametrize("dims", [(63, 66), (140, 90)])
@pytest.mark.parametrize("transpose", [False, True])
def test_gmres_dr_with_coefficient_arrays(dims, transpose):
    """Restarts (the kept column re-orthogonalised in the launch): x_c is the
    solution, and the kept space's H = V^T A V has the harmonic Ritz vectors'
    Rayleigh quotients, all with positive real part."""
    kc = W.kfield(dims, 4)
    oop = O.div_k(dims, kc, (4.0, 1.0))
    op = tg().Operator.div_k(dims, torch.tensor(kc, device=DEV), (4.0, 1.0))
    b = W.rhs(oop.n, 9)
    x, space, rep = tg().coarse_setup(op, torch.tensor(b, device=DEV), 40, 12, nev=8, rtolev=1e-9, rtol=1e-11,
                                      maxcyc=80, transpose=transpose)
    assert rep.status == 0
    xs = ODS.solve(oop, b, transpose=transpose)
    A = O.apply_transpose if transpose else O.apply
    r = np.linalg.norm(b - A(oop, x.cpu().numpy())) / np.linalg.norm(b)
    assert r <= 1e-10 and rep.relres == pytest.approx(r, rel=0.05)
    V, H = space.basis()
    V = V.cpu().numpy()
    np.testing.assert_allclose(V @ V.T, np.eye(len(V)), atol=1e-12)
    # the converged pairs' residuals, formed explicitly
    w, Y = np.linalg.eig(H)
    order = np.argsort(abs(w))[:8]
    norm1 = O.norm1(oop)
    for i in order:
        y = V.T @ Y[:, i]
        Ay = A(oop, y.real) + 1j * A(oop, y.imag)
        assert np.linalg.norm(Ay - w[i] * y) / np.linalg.norm(y) / norm1 <= 1e-6


def test_columns_over_memory_that_held_nans():
    """A kept block that an earlier call left full of NaNs (an IDR workspace
    whose shadow space is refused) becomes V: no point is read before its
    column is written."""
    dims, n = (63, 63), 63 * 63
    op = tg().Operator.const_cd(dims, (5.0, 2.0), device=DEV)
    oop = O.const_cd(dims, (5.0, 2.0))
    b = W.rhs(n, 12)
    bt = torch.tensor(b, device=DEV)
    with pytest.raises(tg()._lib.TgdkError):
        tg().solve_idr(op, bt, s=8, shadow=torch.full((8, n), float("nan"), dtype=torch.float64, device=DEV))
    x, _ = tg().solve(op, bt, method="gmres", m3=23, rtol=1e-13, max_extra=2)
    xo, _ = OG.gmres_proj(oop, b, rtol=1e-13, m=23, maxcyc=2)
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-10 * np.linalg.norm(xo)
