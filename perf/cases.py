"""Performance cases of the two-grid deflated Krylov solvers.

The cases are the work that a program has the library do, through
``paper_2005_03070_amd``'s public functions, from the smallest two-grid solve
(63^2, where latency counts) to the 255^3 one (where HBM bandwidth counts):

========== =============================================================
kind       one pass
========== =============================================================
solve      fine solve of one system with a moved deflation space, to
           convergence
batch      the same for several right-hand sides in one call
adjoint    solve with A^T of the divergence-form operator, then dL/dk
cycles     fine solve with an iteration budget per cycle (a time-boxed
           call on the largest grids, resumable at the cycle boundary)
gmres      GMRES(m)-Proj(k) for a given number of cycles
idr        IDR(s)-Proj(k) to convergence
setup      coarse GMRES-DR(m, k) for a given number of cycles
space      a coarse space moved to the fine grid (prolongation,
           orthonormalisation, H)
multigrid  one application of the multigrid preconditioner
apply      operator application
========== =============================================================

Right-hand sides are N(0, 1), as in the package's workloads, and so are the
coefficient fields' logarithms (times 0.5).  Solves to convergence ask for a
relative residual of 3e-13, so that their result does not depend on the path
of the iteration: it is A^{-1} b to about 1e-10.  ``exact`` computes that
independently with plain torch in float64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2005_03070_amd as tg

RTOL = 3e-13  # of the solves to convergence


def listed():
    return [
        # the small two-grid workload: n = 3969, every launch is latency
        dict(name="solve_63sq", kind="solve", nx=63, ny=63, bx=40.0, k=10, m=30, precision="fp64"),
        # the 1023^2 workload: 80 MB of vectors, between cache and HBM
        dict(name="solve_1023sq", kind="solve", nx=1023, ny=1023, bx=100.0, k=30, m=80, precision="fp64"),
        # 3-D, float32 inner cycles with float64 refinement
        dict(name="solve_127cube_fp32", kind="solve", nx=127, ny=127, nz=127, bx=50.0, k=40, m=90,
             precision="fp32_ir"),
        # 32 right-hand sides that share an operator and a space
        dict(name="batch_32x511sq", kind="batch", nx=511, ny=511, bx=100.0, k=30, m=80, nrhs=32, precision="fp64"),
        # backward pass of a differentiable solve: per-row coefficients, A^T
        dict(name="adjoint_1023sq", kind="adjoint", nx=1023, ny=1023, bx=60.0, k=30, m=80),
        # the largest workload: 16.6 M unknowns, 40 stored vectors
        dict(name="cycles_255cube", kind="cycles", nx=255, ny=255, nz=255, bx=50.0, k=40, its=10, ncyc=4,
             precision="fp64"),
        # the comparison method of the 1023^2 workload
        dict(name="gmres_1023sq", kind="gmres", nx=1023, ny=1023, bx=100.0, k=30, m=50, ncyc=2),
        # IDR(4), the other inner solver
        dict(name="idr4_511sq", kind="idr", nx=511, ny=511, bx=100.0, k=30, m=80, s=4),
        # phase 1 for the 511^2 batch: its coarse grid
        dict(name="setup_255sq", kind="setup", nx=255, ny=255, bx=100.0, m=80, k=30, ncyc=25),
        # moving the 1023^2 workload's vectors
        dict(name="space_1023sq", kind="space", nx=1023, ny=1023, bx=100.0, k=30, store="f64"),
        # the preconditioner of the 511^2 Helmholtz workload
        dict(name="multigrid_511sq", kind="multigrid", nx=511, ny=511, kappa=100.0, cycles=2, nu=2, nrhs=1),
        # one stencil on the largest grid
        dict(name="apply_255cube", kind="apply", nx=255, ny=255, nz=255, bx=50.0, dtype="f64", nrhs=1,
             transpose=False),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def _odd(n):
    return n if n % 2 else n + 1


def draw(rng):
    c = _draw(rng)
    if "bx" in c:  # cell Peclet number below one, on the coarse grid too
        c["bx"] = min(c["bx"], round(0.8 * min(_dims(c)), 1))
    return c


def _draw(rng):
    kind = rng.choice(["solve", "solve", "solve3", "batch", "adjoint", "cycles", "gmres", "idr", "setup", "space",
                       "multigrid", "apply"])
    bx = round(rng.uniform(10.0, 100.0), 1)
    prec = rng.choice(["fp64", "fp32_ir"])
    k = rng.randint(8, 40)
    m = k + rng.randint(20, 50)
    if kind == "solve":
        # any odd side: the coarse grid has (n - 1) / 2 points
        return dict(kind="solve", nx=_odd(_log(rng, 41, 1023)), ny=_odd(_log(rng, 41, 1023)), bx=bx, k=k, m=m,
                    precision=prec)
    if kind == "solve3":
        n = [_odd(_log(rng, 23, 127)) for _ in range(3)]
        return dict(kind="solve", nx=n[0], ny=n[1], nz=n[2], bx=min(bx, 60.0), k=k, m=m, precision=prec)
    if kind == "batch":
        nx, ny = _odd(_log(rng, 63, 511)), _odd(_log(rng, 63, 511))
        return dict(kind="batch", nx=nx, ny=ny, bx=bx, k=k, m=m, nrhs=rng.randint(2, 32), precision=prec)
    if kind == "adjoint":
        return dict(kind="adjoint", nx=_odd(_log(rng, 63, 1023)), ny=_odd(_log(rng, 63, 1023)), bx=min(bx, 60.0),
                    k=k, m=m)
    if kind == "cycles":
        n = [_log(rng, 96, 255) for _ in range(3)]
        return dict(kind="cycles", nx=n[0], ny=n[1], nz=n[2], bx=min(bx, 50.0), k=k, its=rng.randint(5, 10),
                    ncyc=rng.randint(2, 4), precision="fp64")
    if kind == "gmres":
        return dict(kind="gmres", nx=_log(rng, 63, 1023), ny=_log(rng, 63, 1023), bx=bx, k=k,
                    m=rng.randint(20, 60), ncyc=2)
    if kind == "idr":
        return dict(kind="idr", nx=_odd(_log(rng, 63, 511)), ny=_odd(_log(rng, 63, 511)), bx=bx, k=k, m=m,
                    s=rng.choice([1, 2, 4, 4, 5, 8]))
    if kind == "setup":
        return dict(kind="setup", nx=_log(rng, 31, 255), ny=_log(rng, 31, 255), bx=bx, m=60 + k // 2,
                    k=k // 2 + 4, ncyc=25)
    if kind == "space":
        return dict(kind="space", nx=_odd(_log(rng, 127, 1023)), ny=_odd(_log(rng, 127, 1023)), bx=bx, k=k,
                    store=rng.choice(["f64", "f32"]))
    if kind == "multigrid":
        if rng.random() < 0.3:
            n = [rng.choice([31, 47, 63, 95, 127]) for _ in range(3)]
            return dict(kind="multigrid", nx=n[0], ny=n[1], nz=n[2], kappa=round(rng.uniform(10, 100), 1), cycles=2,
                        nu=2, nrhs=rng.choice([1, 2]))
        return dict(kind="multigrid", nx=_odd(_log(rng, 63, 1023)), ny=_odd(_log(rng, 63, 1023)),
                    kappa=round(rng.uniform(10, 100), 1), cycles=2, nu=2, nrhs=rng.choice([1, 1, 4]))
    if rng.random() < 0.5:
        return dict(kind="apply", nx=_log(rng, 63, 1023), ny=_log(rng, 63, 1023), bx=bx,
                    dtype=rng.choice(["f64", "f32"]), nrhs=rng.choice([1, 1, 4]), transpose=rng.random() < 0.5)
    return dict(kind="apply", nx=_log(rng, 31, 255), ny=_log(rng, 31, 255), nz=_log(rng, 31, 255),
                bx=min(bx, 50.0), dtype=rng.choice(["f64", "f32"]), nrhs=1, transpose=rng.random() < 0.5)


# ------------------------------------------------------------------ inputs
def _dims(c):
    return (c["nx"], c["ny"], c["nz"]) if c.get("nz") else (c["nx"], c["ny"])


def _beta(c):
    # the 3-D workload's direction (5, 2, 1); along x in 2-D
    bx = c.get("bx", 0.0)
    return (bx, 0.4 * bx, 0.2 * bx) if c.get("nz") else (bx, 0.0)


def _n(c):
    return math.prod(_dims(c))


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _normal(shape, seed, salt=0, dtype=torch.float64):
    return torch.randn(shape, dtype=dtype, device="cuda", generator=_gen(seed, salt))


def _kcell(c, seed):
    return torch.exp(0.5 * _normal((c["ny"] + 1, c["nx"] + 1), seed, 5))


def _operator(c, seed):
    if c["kind"] == "adjoint":
        return tg.Operator.div_k(_dims(c), _kcell(c, seed), _beta(c))
    if c["kind"] == "multigrid":
        return tg.Operator.const_cd(_dims(c), sigma=c["kappa"] ** 2)
    return tg.Operator.const_cd(_dims(c), _beta(c))


def _modes(c, k, seed):
    """k smooth vectors (products of sines, the Laplacian's lowest modes with
    a little noise): a basis that does not depend on a coarse solve."""
    dims = _dims(c)
    idx = sorted((sum((q + 1) ** 2 for q in np.unravel_index(j, (16,) * len(dims))), j) for j in
                 range(16 ** len(dims)))[:k]
    W = 1e-3 * _normal((k, _n(c)), seed, 7)
    for row, (_, j) in enumerate(idx):
        f = torch.ones((1,) * len(dims), dtype=torch.float64, device="cuda")
        for a, q in enumerate(np.unravel_index(j, (16,) * len(dims))):
            x = torch.arange(1, dims[a] + 1, dtype=torch.float64, device="cuda") * (math.pi * (q + 1) / (dims[a] + 1))
            shape = [1] * len(dims)
            shape[len(dims) - 1 - a] = dims[a]
            f = f * torch.sin(x).reshape(shape)
        W[row] += f.reshape(-1)
    return W


def _two_grid(c, op, b, transpose=False):
    """Phase 1 as a program does it (a bounded number of coarse cycles)."""
    s = tg.TwoGridSolver(op, m=c["m"], k=c["k"], maxcyc=8, rtolev=1e-10, transpose=transpose,
                         store=torch.float32 if c.get("precision") == "fp32_ir" else torch.float64)
    x0 = s.setup(b)
    return s.defl, x0


def prepare(case, seed):
    c = dict(case)
    kind, n = c["kind"], _n(c)
    st = {"c": c, "op": _operator(c, seed)}
    if kind == "apply":
        dt = torch.float64 if c["dtype"] == "f64" else torch.float32
        st["x"] = _normal((n,) if c["nrhs"] == 1 else (c["nrhs"], n), seed, dtype=dt)
        return st
    if kind == "multigrid":
        st["x"] = _normal((n,) if c["nrhs"] == 1 else (c["nrhs"], n), seed)
        st["mg"] = tg.Multigrid(st["op"], cycles=c["cycles"], nu=c["nu"])
        return st
    if kind == "space":
        coarse = st["op"].coarsen()
        cc = dict(c, nx=(c["nx"] - 1) // 2, ny=(c["ny"] - 1) // 2)
        st["coarse"] = coarse
        st["space"] = tg.defl_from_basis(coarse, _modes(cc, c["k"], seed))
        return st
    if kind == "batch":
        st["b"] = _normal((c["nrhs"], n), seed)
        st["defl"], _ = _two_grid(c, st["op"], st["b"][0].contiguous())
        return st
    st["b"] = _normal((n,), seed)
    if kind == "setup":
        return st
    if kind in ("cycles", "gmres"):
        st["defl"] = tg.defl_from_basis(st["op"], _modes(c, c["k"], seed))
        return st
    st["defl"], st["x0"] = _two_grid(c, st["op"], st["b"], transpose=kind == "adjoint")
    if kind == "idr":
        st["shadow"] = _normal((c["s"], n), seed, 9)
    if kind == "adjoint":
        st["u"] = _normal((n,), seed, 6)
    return st


# -------------------------------------------------------------------- pass
def run(st):
    c, op = st["c"], st["op"]
    kind = c["kind"]
    if kind == "solve":
        x, _ = tg.solve(op, st["b"], x0=st["x0"], defl=st["defl"], precision=c["precision"], rtol=RTOL,
                        max_extra=200)
        return {"x": x}
    if kind == "batch":
        x, _ = tg.solve(op, st["b"], defl=st["defl"], precision=c["precision"], rtol=RTOL, max_extra=200)
        return {"x": x}
    if kind == "adjoint":
        lam, _ = tg.solve(op, st["b"], x0=st["x0"], defl=st["defl"], rtol=RTOL, max_extra=200, transpose=True)
        return {"lam": lam, "grad_k": tg.grad_k(op, lam, st["u"])}
    if kind == "cycles":
        x, _ = tg.solve(op, st["b"], defl=st["defl"], precision=c["precision"], rtol=1e-8, ncyc=c["ncyc"],
                        maxit_cycle=c["its"], max_extra=0)
        return {"x": x}
    if kind == "gmres":
        x, _ = tg.solve(op, st["b"], defl=st["defl"], method="gmres", m3=c["m"], rtol=1e-12, max_extra=c["ncyc"])
        return {"x": x}
    if kind == "idr":
        x, _ = tg.solve_idr(op, st["b"], s=c["s"], shadow=st["shadow"], x0=st["x0"], defl=st["defl"], rtol=RTOL,
                            max_extra=200)
        return {"x": x}
    if kind == "setup":
        x, _, _ = tg.coarse_setup(op, st["b"], c["m"], c["k"], rtolev=1e-30, rtol=1e-8, maxcyc=c["ncyc"])
        return {"x": x}
    if kind == "space":
        V, H = tg.defl_prolongate(st["space"], op,
                                  store=torch.float64 if c["store"] == "f64" else torch.float32).basis()
        return {"V": V, "H": H}
    if kind == "multigrid":
        return {"y": st["mg"].apply(st["x"])}
    return {"y": op.apply(st["x"], transpose=c["transpose"])}


def work(case):
    """Bytes and operations a pass cannot do without.  Solves: the operator,
    the right-hand side and the space read once per pass over them that the
    method makes (a BiCGStab iteration's 14 vectors, a projection's two
    passes over V and 10 vectors), for a typical count of iterations."""
    c = case
    n, dim = _n(c), 3 if c.get("nz") else 2
    nnz, k = 2 * dim + 1, c.get("k", 0)
    kind = c["kind"]
    if kind == "apply":
        w = 8 if c["dtype"] == "f64" else 4
        return {"bytes": 2 * w * n * c["nrhs"], "flops": 2 * nnz * n * c["nrhs"]}
    if kind == "multigrid":
        f = 4 / 3 if dim == 2 else 8 / 7
        return {"bytes": 16 * n * c["nrhs"] * c["cycles"], "flops": f * c["cycles"] * c["nrhs"] * n * (
            2 * c["nu"] + 1) * (2 * nnz + 3)}
    if kind == "space":
        nc = n / 2 ** dim
        return {"bytes": 8 * k * (nc + 2 * n), "flops": n * k * (8 * k + 2 * nnz)}
    if kind == "setup":
        steps = c["m"] + (c["ncyc"] - 1) * (c["m"] - c["k"])
        avg = 0.5 * (c["m"] + c["k"])
        return {"bytes": 8 * n * steps * 2 * (avg + 2), "flops": n * steps * (8 * avg + 2 * nnz)}
    if kind == "gmres":
        steps = c["ncyc"] * c["m"]
        avg = 0.5 * c["m"]
        return {"bytes": 8 * n * (steps * 2 * (avg + 2) + c["ncyc"] * 2 * k), "flops": n * steps * (8 * avg + 2 * nnz)}
    w = 4 if c.get("precision") == "fp32_ir" else 8
    if kind == "cycles":
        its, cyc, nrhs = c["ncyc"] * c["its"], c["ncyc"], 1
    else:
        its, cyc, nrhs = (1.6 if dim == 2 else 2.5) * max(_dims(c)), 20, c.get("nrhs", 1)
    if kind == "idr":
        per = 2 * (5 * c["s"] + 10) / 5 * w
    elif kind == "adjoint":
        per = 14 * w + 2 * nnz * w
    else:
        per = 14 * w
    return {"bytes": nrhs * n * (its * per + cyc * (2 * k * w + 80)), "flops": nrhs * n * (
        its * (4 * nnz + 24) + cyc * 4 * k)}


# ------------------------------------------------------------------- exact
def _coef(c, seed, transpose):
    """(axis, shift, coefficient) of the stencil, axis 0 = x: scalars, or
    (n_y, n_x) arrays for the divergence-form operator."""
    dims = _dims(c)
    if c["kind"] == "adjoint":
        kc, (nx, ny), bx = _kcell(c, seed), dims, _beta(c)[0]
        hx, hy = 1.0 / (nx + 1), 1.0 / (ny + 1)
        sw, se, nw, ne = kc[:-1, :-1], kc[:-1, 1:], kc[1:, :-1], kc[1:, 1:]
        W = -0.5 * (sw + nw) / hx ** 2 - bx / (2 * hx)
        E = -0.5 * (se + ne) / hx ** 2 + bx / (2 * hx)
        S, N = -0.5 * (sw + se) / hy ** 2, -0.5 * (nw + ne) / hy ** 2
        C = 0.5 * (sw + nw + se + ne) / hx ** 2 + 0.5 * (sw + se + nw + ne) / hy ** 2
        if not transpose:
            return C, [(0, -1, W), (0, 1, E), (1, -1, S), (1, 1, N)]
        pad = torch.nn.functional.pad
        return C, [(0, -1, pad(E, (1, 0))[:, :-1]), (0, 1, pad(W, (0, 1))[:, 1:]),
                   (1, -1, pad(N, (0, 0, 1, 0))[:-1]), (1, 1, pad(S, (0, 0, 0, 1))[1:])]
    C, off = c["kappa"] ** 2 if c["kind"] == "multigrid" else 0.0, []
    for a, (d, b) in enumerate(zip(dims, _beta(c))):
        h = 1.0 / (d + 1)
        if c["kind"] == "multigrid":
            b = 0.0
        if transpose:
            b = -b
        C += 2.0 / h ** 2
        off += [(a, -1, -1.0 / h ** 2 - b / (2 * h)), (a, 1, -1.0 / h ** 2 + b / (2 * h))]
    return C, off


def _stencil(dims, coef, x):
    C, off = coef
    u = x.reshape((-1,) + tuple(reversed(dims)))
    y = C * u
    for a, s, v in off:
        ax, L = u.dim() - 1 - a, dims[a]
        dst, src = (slice(1, L), slice(0, L - 1)) if s < 0 else (slice(0, L - 1), slice(1, L))
        at = [slice(None)] * u.dim()
        fr = list(at)
        at[ax], fr[ax] = dst, src
        vv = v[tuple(at[1:])] if isinstance(v, torch.Tensor) else v
        y[tuple(at)] += vv * u[tuple(fr)]
    return y.reshape(x.shape)


def _inverse(A, b, passes=60):
    """A^{-1} b by restarted BiCGStab, every restart from the true residual,
    until the residual stops getting smaller."""
    x, r = torch.zeros_like(b), b.clone()
    best, bx, stuck = float(r.norm()), x.clone(), 0
    goal = 2e-15 * best
    for _ in range(passes):
        rh, p, e = r.clone(), r.clone(), torch.zeros_like(b)
        rho = rh @ r
        start = float(r.norm())
        for i in range(4000):
            v = A(p)
            al = rho / (rh @ v)
            s = r - al * v
            t = A(s)
            om = (t @ s) / (t @ t)
            e += al * p + om * s
            r = s - om * t
            new = rh @ r
            p = r + (new / rho) * (al / om) * (p - om * v)
            rho = new
            if i % 20 == 19:
                now = float(r.norm())
                if not now > 1e-4 * start:
                    break
        r = b - A(x + e)
        now = float(r.norm())
        if now < best:
            x = x + e
            stuck = stuck + 1 if now > 0.5 * best else 0
            best, bx = now, x
        else:
            r = b - A(x)
            stuck += 1
        if best <= goal or stuck >= 2:
            break
    return bx


def _project(A, V, LU, r):
    w = torch.linalg.lu_solve(*LU, (V @ r)[:, None])[:, 0] @ V
    return w, r - A(w)


def _orthonormal(W):
    for _ in range(2):
        L = torch.linalg.cholesky(W @ W.T)
        W = torch.linalg.inv(L) @ W
    return W


def _cycles(c, A, b, V, LU):
    """BiCGStab with a projection before every cycle; a cycle ends at its
    share of the remaining reduction or after c["its"] iterations."""
    x = torch.zeros_like(b)
    nu0 = float(b.norm())
    tau = 1e-8 * nu0
    for cyc in range(1, c["ncyc"] + 1):
        w, r = _project(A, V, LU, b - A(x))
        x = x + w
        nu = float(r.norm())
        tol = nu * min((tau / nu) ** (1.0 / (c["ncyc"] - cyc + 1)), (nu0 / nu) * (tau / nu0) ** (cyc / c["ncyc"]))
        rh, p = r.clone(), r.clone()
        rho = rh @ r
        for _ in range(c["its"]):
            v = A(p)
            al = rho / (rh @ v)
            s = r - al * v
            x = x + al * p
            if float(s.norm()) <= tol:
                break
            t = A(s)
            om = (t @ s) / (t @ t)
            x = x + om * s
            r = s - om * t
            if float(r.norm()) <= tol:
                break
            new = rh @ r
            p = r + (new / rho) * (al / om) * (p - om * v)
            rho = new
    return x


def _gmres(c, A, b, V, LU):
    x, m = torch.zeros_like(b), c["m"]
    for _ in range(c["ncyc"]):
        w, r = _project(A, V, LU, b - A(x))
        x = x + w
        Q = torch.zeros((m + 1, b.numel()), dtype=torch.float64, device=b.device)
        H = torch.zeros((m + 1, m), dtype=torch.float64, device=b.device)
        beta = r.norm()
        Q[0] = r / beta
        for j in range(m):
            w = A(Q[j])
            for _ in range(2):
                h = Q[:j + 1] @ w
                w = w - h @ Q[:j + 1]
                H[:j + 1, j] += h
            H[j + 1, j] = w.norm()
            Q[j + 1] = w / H[j + 1, j]
        rhs = torch.zeros((m + 1, 1), dtype=torch.float64)
        rhs[0] = float(beta)
        y = torch.linalg.lstsq(H.cpu(), rhs).solution[:, 0].to(b.device)
        x = x + y @ Q[:m]
    return x


def _prolong(dims, v):
    """Linear interpolation of (rows, n_c) vectors to the grid 2 n_c + 1."""
    u = v.reshape((-1,) + tuple(reversed(dims)))
    for ax in range(1, u.dim()):
        L = u.shape[ax]
        shape = list(u.shape)
        shape[ax] = 2 * L + 1
        f = torch.zeros(shape, dtype=u.dtype, device=u.device)
        at = [slice(None)] * u.dim()
        at[ax] = slice(1, None, 2)  # the points that coincide with coarse ones
        f[tuple(at)] = u
        at[ax] = slice(0, 2 * L, 2)
        f[tuple(at)] += 0.5 * u
        at[ax] = slice(2, None, 2)
        f[tuple(at)] += 0.5 * u
        u = f
    return u.reshape(u.shape[0], -1)


def _restrict(dims, v):
    u = v.reshape((-1,) + tuple(reversed(dims)))
    for ax in range(1, u.dim()):
        L = (u.shape[ax] - 1) // 2
        at = [[slice(None)] * u.dim() for _ in range(3)]
        for q in range(3):
            at[q][ax] = slice(q, q + 2 * L - 1, 2)
        u = 0.25 * u[tuple(at[0])] + 0.5 * u[tuple(at[1])] + 0.25 * u[tuple(at[2])]
    return u.reshape(u.shape[0], -1)


def _vcycle(c, dims, v):
    cc = dict(c, nx=dims[0], ny=dims[1])
    if len(dims) == 3:
        cc["nz"] = dims[2]
    coef = _coef(cc, 0, False)
    sc = (4 / 5 if len(dims) == 2 else 6 / 7) / coef[0]
    z = sc * v
    coarse = all(d >= 3 and d % 2 for d in dims)
    for _ in range((c["nu"] if coarse else 20) - 1):
        z = z + sc * (v - _stencil(dims, coef, z))
    if coarse:
        half = tuple((d - 1) // 2 for d in dims)
        z = z + _prolong(half, _vcycle(c, half, _restrict(dims, v - _stencil(dims, coef, z))))
        for _ in range(c["nu"]):
            z = z + sc * (v - _stencil(dims, coef, z))
    return z


def _grad_k(c, lam, u):
    nx, ny = c["nx"], c["ny"]
    pad = torch.nn.functional.pad
    lam, u = (pad(t.reshape(ny, nx), (1, 1, 1, 1)) for t in (lam, u))
    ex = (lam[:, 1:] - lam[:, :-1]) * (u[:, 1:] - u[:, :-1]) * (nx + 1) ** 2
    ey = (lam[1:] - lam[:-1]) * (u[1:] - u[:-1]) * (ny + 1) ** 2
    return -0.5 * (ex[:-1] + ex[1:] + ey[:, :-1] + ey[:, 1:])


def exact(case, seed):
    c = dict(case)
    kind, n, dims = c["kind"], _n(c), _dims(c)
    if kind == "apply":
        x = _normal((n,) if c["nrhs"] == 1 else (c["nrhs"], n), seed,
                    dtype=torch.float64 if c["dtype"] == "f64" else torch.float32).double()
        return {"y": _stencil(dims, _coef(c, seed, c["transpose"]), x)}
    if kind == "multigrid":
        x = _normal((n,) if c["nrhs"] == 1 else (c["nrhs"], n), seed)
        v = x.reshape(-1, n)
        z, coef = torch.zeros_like(v), _coef(c, seed, False)
        for _ in range(c["cycles"]):
            z = z + _vcycle(c, dims, v - _stencil(dims, coef, z))
        return {"y": z.reshape(x.shape)}
    coef = _coef(c, seed, kind == "adjoint")

    def A(x):
        return _stencil(dims, coef, x)

    if kind == "space":
        half = tuple((d - 1) // 2 for d in dims)
        V = _orthonormal(_prolong(half, _modes(dict(c, nx=half[0], ny=half[1]), c["k"], seed)))
        # the sign of a column is the thin QR's with a positive diagonal,
        # whose coarse factor the library applies before the prolongation;
        # both triangular factors have positive diagonals, so V is unique
        if c["store"] == "f32":
            V = V.float().double()
        return {"V": V, "H": (V @ A(V).T).cpu().numpy()}
    if kind == "batch":
        b = _normal((c["nrhs"], n), seed)
        if c["nrhs"] * max(dims) > 4000:  # about 20 seconds
            return None
        return {"x": torch.stack([_inverse(A, r) for r in b])}
    b = _normal((n,), seed)
    if kind in ("cycles", "gmres"):
        V = _orthonormal(_modes(c, c["k"], seed))
        AV = torch.stack([A(v) for v in V])
        LU = torch.linalg.lu_factor(V @ AV.T)
        del AV
        return {"x": (_cycles if kind == "cycles" else _gmres)(c, A, b, V, LU)}
    if kind in ("solve", "idr", "setup"):
        return {"x": _inverse(A, b)}
    lam = _inverse(A, b)
    return {"lam": lam, "grad_k": _grad_k(c, lam, _normal((n,), seed, 6))}
