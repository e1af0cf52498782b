// IDR(s)(ncyc)-Proj(k) on 2-D grids of up to one tile per compute unit, a
// whole solve in one launch: the rounds of kernels_idr.hip with their vectors
// kept on the chip (see kernels_resident2d.hip for the scheme).
//
// What bounds the vector kernels on such grids is launches: a round of s = 4
// is 24 of them for 5 operator applications (511^2: 55 us per application, 3.7
// of them per one-workgroup epilogue).  Here G, U, r, e and t live in
// registers (2 s + 3 values a point), the shadow columns P in LDS; every
// workgroup carries r, G and U on the ring around its tile by the same
// recurrences, so an operator application needs its neighbours' edge values of
// g_k (or t) alone, in the exchange that also sums its products.  A round has
// 2 s + 1 exchanges: g_k with m = P^T g_k and the last update's ||r||^2; for
// k > 0 P^T g_k again after the orthogonalisation; t with t.t, t.r, r.r; and
// f = P^T r with ||r||^2.  The s x s solves are taken by one thread of every
// workgroup, redundantly.
//
// Tiles are 64 x 16, 32 or 64 (2, 4 or 8 points a thread; P: at most 128 KB of
// LDS): the smallest that leave at most one per compute unit.  More points a
// thread run into spills (float64 with 8 points and s = 4, or 4 points and s = 8:
// 60 registers a step) and instructions issued by too few units; more
// workgroups cost the exchange little.  Microseconds per operator application
// with 64 x 64 and 64 x 16 tiles, float64, s = 4: 63^2 6.7 and 4.9, 127^2 9.0 and 5.6,
// 255^2 10.0 and 6.4, 511^2 10.4 and 6.9; s = 8 with 64 x 32 and 64 x 16: 127^2 11.9 and 8.6,
// 511^2 13.2 and 10.2; s = 1: 255^2 4.8 and 4.4.  A grid that one workgroup's tile
// holds without spills takes one (63^2, s = 1: 2.5, in four 3.2).  Vector kernels
// -> this one, float64, s = 4: 127^2 25.7 -> 5.6, 511^2 30.1 -> 6.9, 1023^2 (64 x 64)
// 50.7 -> 12.8; s = 1, 511^2 25.1 -> 4.8; s = 8, 511^2 46.1 -> 10.2.  Bound now by the
// exchanges (2 to 2.6 us) and, at 1023^2 with s = 4, by the spills.
#include "resident2d.h"

namespace tgdk {

template <class TI, int SM, int RQ>
struct IdrLds : ResLds {
    TI P[SM][RW * RQ * 64];
    double M[SM * SM], f[SM], c[SM], alpha[SM];
    double beta, om;
    int status, mvps;
};

// c = solution of the lower-triangular system M_(k:, k:) c = f_(k:).
template <int SM, class LDS>
__device__ __forceinline__ void idr_coeffs(LDS& S, int s, int k) {
    for (int i = k; i < s; ++i) {
        double v = S.f[i];
        for (int j = k; j < i; ++j) v -= S.M[i * SM + j] * S.c[j - k];
        S.c[i - k] = v / S.M[i * SM + i];
    }
}

// Report of an update of r in the first cycle, and its tests: the cycle's
// end status, or IN_RUNNING.
template <class LDS>
__device__ __forceinline__ int idr_update_tests(LDS& S, SolveState* st, bool report, double rr, double coef, int red,
                                                double target2) {
    if (report && S.hot.icyc == 1 && S.nhist < NHIST) {
        const int h = S.nhist++;
        st->hist[3 * h] = sqrt(rr);
        st->hist[3 * h + 1] = coef;
        st->hist[3 * h + 2] = (double)red;
    }
    if (rr <= target2) return IN_CONVERGED;
    if (!isfinite(rr)) return IN_BREAK_NOUPD;
    return IN_RUNNING;
}

template <bool VAR, class TI, int SM, int RQ>
__global__ __launch_bounds__(RT) void k_resident_idr(ResArgs A, const double* P64, int s, double kappa) {
    __shared__ IdrLds<TI, SM, RQ> S;
    const int t = threadIdx.x, lane = t & 63, wave = uniform((int)(t >> 6));
    ResTeam M;
    res_place(M, A);
    const DevProb& P = A.probs[0];
    SolveState* st = P.st;
    const int k = uniform(P.k), maxit = A.init.maxit;
    ResTile<RQ, VAR> tl;
    tl.set(M, P.op);
    auto ok = [&](int q) { return tl.ok(q); };
    const bool leader = M.w == 0 && t == 0;
    {
        int g[RQ];
        tl.points(g);
        for (int j = 0; j < SM; ++j)
#pragma unroll
            for (int q = 0; q < RQ; ++q)
                S.P[j][(wave * RQ + q) * 64 + lane] = j < s && ok(q) ? (TI)P64[(long long)j * tl.n + g[q]] : TI(0);
    }
    const TI* cf = VAR && tl.var ? uniform(coef_ptr<TI>(P.op)) : nullptr;
    auto stencil = [&](const TI(&u)[RQ], TI ring, TI(&y)[RQ]) {
        if (VAR && tl.var) {
            const int g1 = opaque(tl.g0);
            tile_stencil<TI, VAR>(S, u, ring, tl.full, ok,
                                  [&](int o, int q) { return cf[o * tl.n + (ok(q) ? g1 + q * tl.nx : 0)]; }, y);
        } else {
            // (two points at a time, as with coefficient arrays: G and U leave
            // no registers for the neighbours of all eight)
            tile_stencil<TI, true>(S, u, ring, tl.full, ok, [&](int o, int) { return (TI)tl.cc(o); }, y);
        }
    };
    // P^T y over this thread's points, into a[0 .. SM)
    auto dots = [&](const TI(&y)[RQ], double* a) {
#pragma unroll
        for (int j = 0; j < SM; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            double d = 0.0;
#pragma unroll
            for (int q = 0; q < RQ; ++q) d += (double)S.P[j][(wave * RQ + q) * 64 + lane] * (double)y[q];
            a[j] = d;
        }
    };
    auto norm2 = [&](const TI(&y)[RQ]) {
        double d = 0.0;
#pragma unroll
        for (int q = 0; q < RQ; ++q) d += (double)y[q] * (double)y[q];
        return d;
    };
    if (t == 0) res_begin(S, A.init);
    __syncthreads();
    TI r[RQ], e[RQ], G[SM][RQ], U[SM][RQ];
#pragma unroll
    for (int q = 0; q < RQ; ++q) {
        r[q] = e[q] = TI(0);
#pragma unroll
        for (int j = 0; j < SM; ++j) G[j][q] = U[j][q] = TI(0);
    }
    const TI none[RQ] = {};
    double dummy = 0.0;
    if (!res_enter<false>(M, S, A)) return;
    bool any = false;
    int mvps = 0, inner = IN_CONVERGED;
    for (;;) {
        double r64[RQ], ring;
        const int end = res_boundary<TI>(M, S, A, P, k, tl, leader, [&](int q) { return (double)e[q]; }, any, mvps <= 1,
                                         mvps, inner, r64, r, ring);
        if (end < 0) return;
        if (end) break;
        const double target2 = S.hot.target2;
        TI rr_ = (TI)ring, Gr[SM], Ur[SM];  // ring values of r, G, U
#pragma unroll
        for (int q = 0; q < RQ; ++q) {
            e[q] = TI(0);
#pragma unroll
            for (int j = 0; j < SM; ++j) G[j][q] = U[j][q] = TI(0);
        }
#pragma unroll
        for (int j = 0; j < SM; ++j) Gr[j] = Ur[j] = TI(0);
        // ---- cycle start: f = P^T r
        double a[SM + 1], sum[SM + 1];
        dots(r, a);
        a[SM] = norm2(r);
        if (exchange<SM + 1, false>(M, S, a, none, dummy, sum)) return;
        if (t == 0) {
            for (int i = 0; i < SM * SM; ++i) S.M[i] = 0.0;
            for (int i = 0; i < s; ++i) {
                S.M[i * SM + i] = 1.0;
                S.f[i] = S.c[i] = S.red[i];
            }
            S.om = 1.0;
            S.mvps = 0;
            S.status = S.red[SM] <= target2 ? IN_CONVERGED : IN_RUNNING;
        }
        __syncthreads();
        any = false;
        bool round0 = true;
        while (S.status == IN_RUNNING) {
            for (int kk = 0; kk < s; ++kk) {
                // the update of step kk - 1: r -= beta g, e += beta u
                if (kk > 0) {
                    const double beta = S.beta;
#pragma unroll
                    for (int j = 0; j < SM - 1; ++j)
                        if (j == kk - 1) {
#pragma unroll
                            for (int q = 0; q < RQ; ++q) {
                                r[q] = (TI)((double)r[q] - beta * (double)G[j][q]);
                                e[q] = any ? (TI)((double)e[q] + beta * (double)U[j][q]) : (TI)(beta * (double)U[j][q]);
                            }
                            rr_ = (TI)((double)rr_ - beta * (double)Gr[j]);
                        }
                    any = true;
                }
                // the direction u_kk = U_(kk:) c + omega (r - G_(kk:) c) (first round: r)
                TI u[RQ], ur;
                if (round0) {
#pragma unroll
                    for (int q = 0; q < RQ; ++q) u[q] = r[q];
                    ur = rr_;
                } else {
                    const double om = S.om;
                    double cj[SM];  // c by column, 0 for the others
#pragma unroll
                    for (int j = 0; j < SM; ++j) cj[j] = j >= kk && j < s ? S.c[j >= kk ? j - kk : 0] : 0.0;
                    auto dir = [&](TI rv, auto gj, auto uj) {
                        double gc = 0.0, uc = 0.0;
#pragma unroll
                        for (int j = 0; j < SM; ++j) {
                            gc += (double)gj(j) * cj[j];
                            uc += (double)uj(j) * cj[j];
                        }
                        return (TI)(uc + om * (double)(TI)((double)rv - gc));
                    };
#pragma unroll
                    for (int q = 0; q < RQ; ++q)
                        u[q] = dir(r[q], [&](int j) { return G[j][q]; }, [&](int j) { return U[j][q]; });
                    ur = dir(rr_, [&](int j) { return Gr[j]; }, [&](int j) { return Ur[j]; });
                }
                // g = A u, m = P^T g, and ||r||^2 of the update
                TI g[RQ];
                stencil(u, ur, g);
                dots(g, a);
                a[SM] = norm2(r);
                if (exchange<SM + 1, true>(M, S, a, g, ring, sum)) return;
                TI gr = (TI)ring;
                if (kk > 0) {
                    if (t == 0) {
                        int stt = idr_update_tests(S, st, leader, S.red[SM], S.beta, 0, target2);
                        if (stt == IN_RUNNING && S.mvps >= maxit) stt = IN_MAXIT;
                        S.status = stt;
                        // forward substitution with the leading kk x kk block of M
                        for (int i = 0; i < kk; ++i) {
                            double x = S.red[i];
                            for (int j = 0; j < i; ++j) x -= S.M[i * SM + j] * S.alpha[j];
                            S.alpha[i] = x / S.M[i * SM + i];
                        }
                    }
                    __syncthreads();
                    if (S.status != IN_RUNNING) break;
                    // g -= G_(:kk) alpha, u -= U_(:kk) alpha, and P^T g afresh
                    double al[SM];
#pragma unroll
                    for (int j = 0; j < SM; ++j) al[j] = j < kk ? S.alpha[j] : 0.0;
                    auto orth = [&](TI y, auto yj) {
                        double d = (double)y;
#pragma unroll
                        for (int j = 0; j < SM - 1; ++j) d -= al[j] * (double)yj(j);
                        return (TI)d;
                    };
#pragma unroll
                    for (int q = 0; q < RQ; ++q) {
                        g[q] = orth(g[q], [&](int j) { return G[j][q]; });
                        u[q] = orth(u[q], [&](int j) { return U[j][q]; });
                    }
                    gr = orth(gr, [&](int j) { return Gr[j]; });
                    ur = orth(ur, [&](int j) { return Ur[j]; });
                    dots(g, a);
                    double a2[SM], s2[SM];
#pragma unroll
                    for (int j = 0; j < SM; ++j) a2[j] = a[j];
                    if (exchange<SM, false>(M, S, a2, none, dummy, s2)) return;
                }
#pragma unroll
                for (int j = 0; j < SM; ++j)
                    if (j == kk) {
#pragma unroll
                        for (int q = 0; q < RQ; ++q) {
                            G[j][q] = g[q];
                            U[j][q] = u[q];
                        }
                        Gr[j] = gr;
                        Ur[j] = ur;
                    }
                // M_(kk:, kk), beta, f, and the next step's coefficients
                if (t == 0) {
                    S.mvps += 1;
                    for (int i = kk; i < s; ++i) S.M[i * SM + kk] = S.red[i];
                    const double mkk = S.M[kk * SM + kk];
                    if (mkk == 0.0 || !isfinite(mkk)) {
                        S.status = IN_BREAK_NOUPD;
                    } else {
                        const double beta = S.f[kk] / mkk;
                        S.beta = beta;
                        if (kk + 1 < s) {
                            for (int i = kk + 1; i < s; ++i) S.f[i] -= beta * S.M[i * SM + kk];
                            if (!round0) idr_coeffs<SM>(S, s, kk + 1);
                        }
                    }
                }
                __syncthreads();
                if (S.status != IN_RUNNING) break;
            }
            if (S.status != IN_RUNNING) break;
            // the last step's update, then t = A r with t.t, t.r, r.r
            {
                const double beta = S.beta;
#pragma unroll
                for (int j = 0; j < SM; ++j)
                    if (j == s - 1) {
#pragma unroll
                        for (int q = 0; q < RQ; ++q) {
                            r[q] = (TI)((double)r[q] - beta * (double)G[j][q]);
                            e[q] = any ? (TI)((double)e[q] + beta * (double)U[j][q]) : (TI)(beta * (double)U[j][q]);
                        }
                        rr_ = (TI)((double)rr_ - beta * (double)Gr[j]);
                    }
                any = true;
            }
            TI tv[RQ];
            stencil(r, rr_, tv);
            double a3[3] = {0.0, 0.0, 0.0}, s3[3];
#pragma unroll
            for (int q = 0; q < RQ; ++q) {
                const double td = (double)tv[q], rd = (double)r[q];
                a3[0] += td * td;
                a3[1] += td * rd;
                a3[2] += rd * rd;
            }
            if (exchange<3, true>(M, S, a3, tv, ring, s3)) return;
            if (t == 0) {
                const double tt = S.red[0], ts = S.red[1], rr = S.red[2];
                int stt = idr_update_tests(S, st, leader, rr, S.beta, 0, target2);
                if (stt == IN_RUNNING && S.mvps >= maxit) stt = IN_MAXIT;
                if (stt == IN_RUNNING) {
                    S.mvps += 1;
                    if (tt == 0.0 || ts == 0.0 || !isfinite(ts / tt)) {
                        stt = IN_BREAK_NOUPD;
                    } else {
                        double om = ts / tt;
                        const double rho = fabs(ts) / (sqrt(tt) * sqrt(rr));
                        if (rho < kappa) om = om * kappa / rho;
                        S.om = om;
                    }
                }
                S.status = stt;
            }
            __syncthreads();
            if (S.status != IN_RUNNING) break;
            // e += omega r, r -= omega t, f = P^T r
            const double om = S.om;
#pragma unroll
            for (int q = 0; q < RQ; ++q) {
                const double rv = (double)r[q];
                e[q] = (TI)((double)e[q] + om * rv);
                r[q] = (TI)(rv - om * (double)tv[q]);
            }
            rr_ = (TI)((double)rr_ - om * (double)(TI)ring);
            dots(r, a);
            a[SM] = norm2(r);
            if (exchange<SM + 1, false>(M, S, a, none, dummy, sum)) return;
            round0 = false;
            if (t == 0) {
                int stt = idr_update_tests(S, st, leader, S.red[SM], om, 1, target2);
                for (int i = 0; i < s; ++i) S.f[i] = S.red[i];
                if (stt == IN_RUNNING && S.mvps >= maxit) stt = IN_MAXIT;
                if (stt == IN_RUNNING) idr_coeffs<SM>(S, s, 0);
                S.status = stt;
            }
            __syncthreads();
        }
        mvps = S.mvps;
        inner = S.status;
        __syncthreads();
        if (t == 0) {
            S.mvp_inner += mvps;
            S.iters_total += mvps;
        }
    }
    if (leader) {
        A.ctl[0] = 1;  // the solve ran
        res_end(S, st, mvps, inner);
    }
}

template <bool VAR, class TI, int SM>
static const void* idr_kernel_rows(int rows) {
    if constexpr (SM <= 4)
        if (rows == 64) return (const void*)k_resident_idr<VAR, TI, SM, 8>;
    if (rows == 32) return (const void*)k_resident_idr<VAR, TI, SM, 4>;
    return (const void*)k_resident_idr<VAR, TI, SM, 2>;
}

template <bool VAR, class TI>
static const void* idr_kernel(int s, int rows) {
    if (s <= 1) return idr_kernel_rows<VAR, TI, 1>(rows);
    if (s <= 2) return idr_kernel_rows<VAR, TI, 2>(rows);
    if (s <= 4) return idr_kernel_rows<VAR, TI, 4>(rows);
    return idr_kernel_rows<VAR, TI, 8>(rows);
}

int resident_idr_rows(int s, const DevOp& op, int max_team) {
    if (s > RES_IDR_SMAX) return 0;
    const int one = s <= 2 ? 64 : s <= 4 ? 32 : 16;  // rows of a tile whose vectors don't spill
    for (int rows = 16; rows <= (s <= 4 ? 64 : 32); rows *= 2) {
        const long long tiles = (long long)((op.nx + RTILE - 1) / RTILE) * ((op.ny + rows - 1) / rows);
        const bool fits = op.nx <= RTILE && op.ny <= one;  // one workgroup, no exchange
        if (tiles <= (fits ? 1 : max_team)) return rows;
    }
    return 0;
}

hipError_t launch_resident_idr(int inner_f32, int var, const ResArgs& args, const DevProb* prob, const double* P64,
                               int s, int rows, double kappa, hipStream_t stream) {
    launch_res_setup(args, prob, 1, stream);
    ResArgs a = args;
    void* av[] = {&a, &P64, &s, &kappa};
    const void* f = inner_f32 ? (var ? idr_kernel<true, float>(s, rows) : idr_kernel<false, float>(s, rows))
                              : (var ? idr_kernel<true, double>(s, rows) : idr_kernel<false, double>(s, rows));
    return hipLaunchCooperativeKernel(f, dim3(args.team), dim3(RT), av, 0, stream);
}

}  // namespace tgdk
