// BiCGStab(ncyc)-Proj(k) on 2-D grids of up to one 64 x 64 tile per compute
// unit, whole solves in one launch: the state machine of step_kernel.h with
// its vectors kept on the chip.
//
// What bounds the step kernel on such grids is not bytes but launches: at
// 1023^2 a phase streams 33 to 84 MB from the MALL in 15 to 23 us of which
// about 9 are the launch, the state, the partial sums and the last wave; at
// 63^2 the same 6 us buy 4 k points.  Here a system belongs to a team of
// workgroups, one per 64 x 64 tile (512 threads, 8 points each; 256 tiles
// cover 1023^2), and r, p, v, t, e and the shadow vector live in registers
// (48 of a thread's 128 float64 values).  A phase is the stencil (rows
// exchanged through LDS, x neighbours by lane moves) and one exchange
// (resident.h) of the phase's sums and of the edge values of v or t.  Each
// workgroup also carries r and p on the one-point ring around its tile by the
// same recurrences, from the neighbours' v and t, so an iteration has two
// exchanges and no other global memory access.
//
// What bounds it now: the two exchanges (2.6 us each with 256 workgroups) and
// about 3 us of instructions an iteration (every wave issues the exchange's
// and the decisions' instructions besides its points': 1024 threads of 4
// points took 14 us where 512 of 8 take 3 on one tile).  Microseconds per
// iteration, float64 (step kernel -> this kernel): 63^2 14.9 -> 3.1, 127^2
// 15.7 -> 5.4, 255^2 15.8 -> 6.6, 511^2 16.4 -> 7.0, 1023^2 31.8 -> 7.5; per-row
// coefficients 255^2 17.8 -> 8.3, 1023^2 40.9 -> 9.0.  Their C, W, E and S are
// held in LDS (128 KB in float64), N is loaded ahead of the exchange.
//
// Cycle boundaries (true residual, projection) read x, b and V from memory
// (1023^2 with 30 vectors: c = V^T r in 42 us, V d in 29 us); every workgroup
// sums c over the team in two hops (workgroup w gathers columns w, w + T, ...)
// and forms d = H^{-1} c itself.
//
// The teams take systems from a queue, so a batch of right-hand sides keeps
// 256 / T teams busy (32 of 511^2 to 3e-13: 432 -> 100 ms).  A system's numbers
// do not depend on its team or on the other systems: a team's sums run over
// its workgroups in order, and the ones past a smaller system's tiles add
// zeros.
#include <string.h>

#include "resident2d.h"

namespace tgdk {

constexpr int RQ = 8;  // rows per wave: 64 x 64 tiles

template <bool VAR, class TI>
struct BiLds : ResLds {
    TI coef[VAR ? 4 : 1][VAR ? RTILE * RTILE : 1];  // C, W, E, S of the tile
};

template <bool VAR, class TI>
__global__ __launch_bounds__(RT) void k_resident2d(ResArgs A) {
    __shared__ BiLds<VAR, TI> S;
    const int t = threadIdx.x, lane = t & 63, wave = uniform(t >> 6);
    ResTeam M;
    res_place(M, A);
    if (!res_enter<false>(M, S, A)) return;
    const TI none[RQ] = {};
    double dummy = 0.0;
    for (;;) {
        // the team's next system
        double tick[1] = {0.0};
        if (M.w == 0 && t == 0)
            tick[0] = (double)__hip_atomic_fetch_add(A.ctl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        double got[1];
        if (exchange<1, false>(M, S, tick, none, dummy, got)) return;
        const int sys = (int)got[0];
        if (sys >= A.nprob) return;
        const DevProb& P = A.probs[sys];
        SolveState* st = P.st;
        const int k = uniform(P.k), maxit = A.init.maxit;
        ResTile<RQ, VAR> tl;
        tl.set(M, P.op);
        auto ok = [&](int q) { return tl.ok(q); };
        const bool leader = M.w == 0 && t == 0;
        // VAR kernels hold C, W, E, S of the tile in LDS in the inner type
        // (an operator without coefficient arrays fills in its constants) and
        // N in registers, loaded before the exchange ahead of each stencil
        const TI* cf = nullptr;
        if (VAR) {
            if (tl.var) cf = uniform(coef_ptr<TI>(P.op));
            int g[RQ];
            tl.points(g);
#pragma unroll
            for (int q = 0; q < RQ; ++q)
#pragma unroll
                for (int o = 0; o < 4; ++o)
                    S.coef[VAR ? o : 0][VAR ? (wave * RQ + q) * 64 + lane : 0] =
                        tl.var ? cf[o * tl.n + g[q]] : (TI)tl.cc(o);
        }
        TI nq[VAR ? RQ : 1];
        auto load_n = [&]() {
            if constexpr (VAR) {
                const int g1 = opaque(tl.g0);
                const char* cn = (const char*)(cf + 4 * tl.n);
#pragma unroll
                for (int q = 0; q < RQ; ++q) {
                    nq[q] = (TI)tl.c4;
                    if (tl.var) nq[q] = *(const TI*)(cn + (unsigned)((ok(q) ? g1 + q * tl.nx : 0) * (int)sizeof(TI)));
                }
            }
        };
        auto cin = [&](int o, int q) -> TI {
            if constexpr (VAR) return o < 4 ? S.coef[o < 4 ? o : 0][(wave * RQ + q) * 64 + lane] : nq[q];
            return (TI)tl.cc(o);
        };
        if (t == 0) res_begin(S, A.init);
        __syncthreads();
        TI r[RQ], p[RQ], v[RQ], e[RQ], h[RQ], s[RQ];
#pragma unroll
        for (int q = 0; q < RQ; ++q) r[q] = p[q] = v[q] = e[q] = h[q] = s[q] = TI(0);
        double upd_a = 0.0, upd_w = 0.0;  // pending update e + a p + w s
        bool upd_any = false;
        int iter = 0, inner = IN_CONVERGED;
        for (;;) {
            double r64[RQ], ring;
            const int end = res_boundary<TI>(
                M, S, A, P, k, tl, leader,
                [&](int q) {
                    double u = (double)e[q];
                    if (upd_a != 0.0) u += upd_a * (double)p[q];
                    if (upd_w != 0.0) u += upd_w * (double)s[q];
                    return u;
                },
                upd_any, iter == 0, iter, inner, r64, r, ring);
            if (end < 0) return;
            if (end) break;
            const double target2 = S.hot.target2;
            double rho = S.hot.rho, alpha = 1.0, omega = 1.0;
            TI rr = (TI)ring, rp = rr, rv;  // ring values of r, p, v
#pragma unroll
            for (int q = 0; q < RQ; ++q) {
                h[q] = r[q];
                p[q] = r[q];
                e[q] = TI(0);
            }
            iter = 0;
            load_n();
            for (;;) {
                // v = A p; r^.v, r.r
                tile_stencil<TI, VAR>(S, p, rp, tl.full, ok, cin, v);
                double a2[2] = {0.0, 0.0}, s2[2];
#pragma unroll
                for (int q = 0; q < RQ; ++q) {
                    a2[0] += (double)h[q] * (double)v[q];
                    a2[1] += (double)r[q] * (double)r[q];
                }
                load_n();
                if (exchange<2, true>(M, S, a2, v, ring, s2)) return;
                if (leader) S.mvp_inner += 1;
                const double sig = s2[0];
                if (sig == 0.0 || !isfinite(sig)) {
                    inner = IN_BREAK_NOUPD;
                    upd_a = upd_w = 0.0;
                    upd_any = iter != 0;
                    break;
                }
                alpha = rho / sig;
                // s = r - alpha v; t = A s; s.s, t.s, t.t, r^.s, r^.t
                const TI al = (TI)alpha;
                rv = (TI)ring;
                rr = rr - al * rv;
                TI tv[RQ];
#pragma unroll
                for (int q = 0; q < RQ; ++q) s[q] = r[q] - al * v[q];
                tile_stencil<TI, VAR>(S, s, rr, tl.full, ok, cin, tv);
                double a5[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, s5[5];
#pragma unroll
                for (int q = 0; q < RQ; ++q) {
                    const double sd = (double)s[q], td = (double)tv[q], hd = (double)h[q];
                    a5[0] += sd * sd;
                    a5[1] += td * sd;
                    a5[2] += td * td;
                    a5[3] += hd * sd;
                    a5[4] += hd * td;
                }
                load_n();
                if (exchange<5, true>(M, S, a5, tv, ring, s5)) return;
                ++iter;
                const double ss = s5[0], ts = s5[1], tt = s5[2];
                const bool half = ss <= target2;
                omega = half ? 0.0 : tt != 0.0 ? ts / tt : 0.0;
                if (leader) {
                    S.mvp_inner += 1;
                    S.iters_total += 1;
                    const int hi = S.nhist;
                    if (hi < NHIST) {
                        st->hist[3 * hi] = rho;
                        st->hist[3 * hi + 1] = alpha;
                        st->hist[3 * hi + 2] = half ? __builtin_nan("") : omega;
                        S.nhist = hi + 1;
                    }
                }
                upd_a = alpha;
                upd_w = omega;
                upd_any = 1;
                if (half) {
                    inner = IN_HALF;
                    break;
                }
                if (omega == 0.0 || !isfinite(omega)) {
                    inner = IN_BREAK_FULL;
                    break;
                }
                double rn2 = ss - 2.0 * omega * ts + omega * omega * tt;
                if (rn2 < 0.0) rn2 = 0.0;
                const double rho_new = s5[3] - omega * s5[4];
                if (rn2 <= target2) {
                    inner = IN_CONVERGED;
                    break;
                }
                if (rho_new == 0.0 || !isfinite(rho_new)) {
                    inner = IN_BREAK_FULL;
                    break;
                }
                if (iter >= maxit) {
                    inner = IN_MAXIT;
                    break;
                }
                // e += alpha p + omega s; r = s - omega t; p = r + beta (p - omega v)
                const TI om = (TI)omega, be = (TI)((rho_new / rho) * (alpha / omega));
                rho = rho_new;
#pragma unroll
                for (int q = 0; q < RQ; ++q) {
                    e[q] = e[q] + al * p[q] + om * s[q];
                    r[q] = s[q] - om * tv[q];
                    p[q] = r[q] + be * (p[q] - om * v[q]);
                }
                rr = rr - om * (TI)ring;
                rp = rr + be * (rp - om * rv);
            }
        }
        if (leader) res_end(S, st, iter, inner);
        __syncthreads();
    }
}

// Sets the queue, the abort word and the gates, empties the exchange regions, stores the descriptors that came as
// arguments and writes every system's initial state.
__global__ __launch_bounds__(256) void k_res_setup(ResArgs A, ResProbs Q, long long words, int teams) {
    u64* x = (u64*)A.xch;
    for (long long i = blockIdx.x * 256LL + threadIdx.x; i < words; i += gridDim.x * 256LL) x[i] = RES_EMPTY;
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < 2 + teams; i += 256) A.ctl[i] = i < 2 ? 0 : A.gate0;
    if (A.upload && blockIdx.x == 0) {
        const u64* src = reinterpret_cast<const u64*>(&Q);
        u64* dst = reinterpret_cast<u64*>(A.probs);
        static_assert(sizeof(DevProb) % 8 == 0, "whole words");
        for (int i = threadIdx.x; i < (int)(A.nprob * sizeof(DevProb) / 8); i += 256) dst[i] = src[i];
    }
    for (int j = blockIdx.x; j < A.nprob; j += gridDim.x) {
        SolveState* st = A.states + j;
        u64* w = reinterpret_cast<u64*>(st);
        static_assert(sizeof(SolveState) % 8 == 0, "whole words");
        for (int i = threadIdx.x; i < (int)(sizeof(SolveState) / 8); i += 256) w[i] = 0;
        __syncthreads();
        if (threadIdx.x == 0) {
            st->method = A.init.method;
            st->ncyc = A.init.ncyc;
            st->icyc = st->icyc0 = A.init.icyc0;
            st->maxit = A.init.maxit;
        }
    }
}

void launch_res_setup(const ResArgs& args, const DevProb* probs, int teams, hipStream_t s) {
    const long long words = (long long)args.xstride * teams;
    const long long nb = (words + 1023) / 1024;
    ResProbs q;
    memset(&q, 0, sizeof(q));
    for (int j = 0; args.upload && j < args.nprob; ++j) q.p[j] = probs[j];
    hipLaunchKernelGGL(k_res_setup, dim3((unsigned)(nb < 1024 ? nb : 1024)), dim3(256), 0, s, args, q, words, teams);
}

hipError_t launch_resident2d(int inner_f32, int var, const ResArgs& args, const DevProb* probs, int teams,
                             hipStream_t s) {
    launch_res_setup(args, probs, teams, s);
    ResArgs a = args;
    void* av[] = {&a};
    const void* f = inner_f32 ? (var ? (const void*)k_resident2d<true, float> : (const void*)k_resident2d<false, float>)
                              : (var ? (const void*)k_resident2d<true, double> : (const void*)k_resident2d<false, double>);
    return hipLaunchCooperativeKernel(f, dim3(teams * args.team), dim3(RT), av, 0, s);
}

}  // namespace tgdk
