// Tiles, exchanges and cycle boundaries of the chip-resident 2-D solves
// (kernels_resident2d.hip, kernels_resident_idr.hip): a workgroup of 512
// threads owns a tile of 64 x 8 RQ points (RQ rows of a column per thread).
#pragma once

#include "resident.h"
#include "step_kernel.h"

namespace tgdk {

constexpr int RT = 512;                   // threads
constexpr int RW = RT / 64;               // waves
constexpr int RTILE = 64;                 // tile width (and slots of an edge)
constexpr int RHALO = 4 * RTILE;          // edge slots of a tile
static_assert(RES_TILE == RTILE, "host layout");

// LDS of the shared parts.
struct ResLds {
    double top[RW + 1][64];  // [w + 1]: last row of wave w; [0]: the ring row below the tile
    double bot[RW + 1][64];  // [w]: first row of wave w; [RW]: the ring row above the tile
    double side[2][RTILE];   // ring columns west and east
    double csh[32][4 * RW + 1];  // column partials of the waves' rows
    double sh[RES_NSUM * 4 * RW];
    double red[RES_NSUM];
    double y[MAXK + 1];
    StepHot hot;
    long long mvp_inner, iters_total, mvp_boundary, nproj;
    double nu_final;
    int branch[4];
    int nhist, stop, dead;
};

// This workgroup's place in its team and the team's exchange buffers.
struct ResTeam {
    u64* base;         // sums, totals, tile edges, column partials, column values
    unsigned* abort_word;
    int T, w;          // team size, this workgroup's index
    int ph;            // phase: buffer ph % 3
    int nbr[4];        // neighbours S, N, W, E (-1: none)
};

// Word offsets into the team's region (T: the team size, TP: rounded up to 64).
__device__ __forceinline__ int round64(int T) { return (T + 63) & ~63; }
__device__ __forceinline__ u64* sum_slot(const ResTeam& M, int T, int buf, int v, int w) {
    return M.base + (unsigned)((buf * RES_NSUM + v) * round64(T) + w);
}
__device__ __forceinline__ u64* total_slot(const ResTeam& M, int T, int buf, int v, int copy) {
    return M.base + (unsigned)(3 * RES_NSUM * round64(T) + (buf * RES_COPIES + copy) * RES_TOTALS + v);
}
__device__ __forceinline__ u64* halo_slot(const ResTeam& M, int T, int buf, int w, int side, int i) {
    return M.base + (unsigned)(3 * RES_NSUM * round64(T) + 3 * RES_COPIES * RES_TOTALS + ((buf * T + w) * 4 + side) * RTILE + i);
}
__device__ __forceinline__ u64* cpart_slot(const ResTeam& M, int T, int c, int w) {
    return M.base + (unsigned)(3 * RES_NSUM * round64(T) + 3 * RES_COPIES * RES_TOTALS + 3 * T * RHALO + c * round64(T) + w);
}
__device__ __forceinline__ u64* cval_slot(const ResTeam& M, int T, int kmax, int c) {
    return cpart_slot(M, T, kmax, 0) + c;
}

// One phase's exchange: the team's sums of a[] into tot[], and, with HALO,
// this tile's edge values y published and the ring values (waves 4..7: side
// wave - 4, position lane) returned in ring.  Wave v handles value v.  A team
// of one takes its own sums; up to 32 workgroups every one reads all partial
// sums, beyond (33 to 256) workgroup (v mod 8) (T / 8) gathers value v and all read its
// total; the sums have the same order, hence the same bits, either way.
// True if the grid aborted.
constexpr int RES_DIRECT = 32;
template <int NV, bool HALO, int RQ, class TY>
__device__ __forceinline__ bool exchange(ResTeam& M, ResLds& S, const double (&a)[NV], const TY (&y)[RQ], double& ring,
                                         double (&tot)[NV]) {
    static_assert(NV <= RES_NSUM && RW == 8 && RT == 2 * RHALO, "wave roles");
    const int t = opaque(threadIdx.x), lane = t & 63, wave = uniform(t >> 6);
    const int T = opaque_uniform(M.T);
    const int buf = M.ph % 3;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last phase's emptied slots
    if (HALO) {
        if (wave == 0 && M.nbr[0] >= 0) res_store(halo_slot(M, T, buf, M.w, 0, lane), (double)y[0]);
        if (wave == RW - 1 && M.nbr[1] >= 0) res_store(halo_slot(M, T, buf, M.w, 1, lane), (double)y[RQ - 1]);
        if (lane == 0 && M.nbr[2] >= 0) {
#pragma unroll
            for (int q = 0; q < RQ; ++q) res_store(halo_slot(M, T, buf, M.w, 2, wave * RQ + q), (double)y[q]);
        }
        if (lane == 63 && M.nbr[3] >= 0) {
#pragma unroll
            for (int q = 0; q < RQ; ++q) res_store(halo_slot(M, T, buf, M.w, 3, wave * RQ + q), (double)y[q]);
        }
    }
    {
        const double s = row_sums<NV>(a);
        if ((lane & 15) < NV) S.sh[(lane & 15) * 4 * RW + wave * 4 + (lane >> 4)] = s;
    }
    __syncthreads();
    const int own = T > RES_DIRECT ? wave * (T / 8) : -1;  // the workgroup that gathers wave `wave`'s values
#pragma unroll
    for (int v0 = 0; v0 < NV; v0 += RW) {
        const int v = v0 + wave;
        if (v < NV) {
            const double s = lanes32_sum(S.sh[v * 4 * RW + (lane & 31)]);
            if (lane == 0) {
                if (T == 1)
                    S.red[v] = s;
                else
                    res_store(sum_slot(M, T, buf, v, M.w), s);
            }
            if (T > 1 && (T <= RES_DIRECT || own == M.w)) {
                const u64* ps[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) ps[c] = c * 64 + lane < T ? sum_slot(M, T, buf, v, c * 64 + lane) : nullptr;
                double x[4];
                res_poll<4>(ps, x, M.abort_word, &S.dead);
                const double g = wave_sum_dpp((x[0] + x[1]) + (x[2] + x[3]));
                if (T <= RES_DIRECT) {
                    if (lane == 0) S.red[v] = g;
                } else if (lane < RES_COPIES) {
                    res_store(total_slot(M, T, buf, v, lane), g);
                }
            }
        }
    }
    if (T > 1) {
        if (HALO && wave >= 4) {
            const int side = wave - 4;
            const int nb = side == 0 ? M.nbr[0] : side == 1 ? M.nbr[1] : side == 2 ? M.nbr[2] : M.nbr[3];
            const bool has = nb >= 0 && (side < 2 || lane < RW * RQ);  // a west or east edge has RW RQ values
            ring = has ? res_poll(halo_slot(M, T, buf, nb, side ^ 1, lane), M.abort_word, &S.dead) : 0.0;
        }
        if (T > RES_DIRECT && wave == 0 && lane < NV)
            S.red[lane] = res_poll(total_slot(M, T, buf, lane, M.w % RES_COPIES), M.abort_word, &S.dead);
    } else if (HALO) {
        ring = 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NV; ++v) tot[v] = S.red[v];
    if (T == 1) return false;
    const bool dead = S.dead != 0;
    // empty this workgroup's slots of the buffer that phase ph + 2 uses
    // (every side: the next system's tile may have other neighbours)
    const int old = (M.ph + 2) % 3;
    if (t < RES_NSUM) res_store_bits(sum_slot(M, T, old, t, M.w), RES_EMPTY);
    if (own == M.w && lane < RES_COPIES) {
#pragma unroll
        for (int v0 = 0; v0 < RES_NSUM; v0 += RW)
            if (v0 + wave < RES_NSUM) res_store_bits(total_slot(M, T, old, v0 + wave, lane), RES_EMPTY);
    }
    if (wave < 4) res_store_bits(halo_slot(M, T, old, M.w, wave, lane), RES_EMPTY);
    ++M.ph;
    return dead;
}

// y = A u on the tile: u in registers, ring the ring values (waves 4..7, side
// wave - 4).  coef(o, q): coefficient o (C, W, E, S, N) at point q.  Points
// outside the domain give 0.  Ends without a barrier (the next exchange has
// two).
template <class T, bool VARC, int RQ, class Ok, class F>
__device__ __forceinline__ void tile_stencil(ResLds& S, const T (&u)[RQ], T ring, bool full, Ok ok,
                                             F&& coef, T (&y)[RQ]) {
    const int t = threadIdx.x, lane = t & 63, wave = uniform(t >> 6);
    T* top = reinterpret_cast<T*>(S.top);
    T* bot = reinterpret_cast<T*>(S.bot);
    T* side = reinterpret_cast<T*>(S.side);
    top[(wave + 1) * 64 + lane] = u[RQ - 1];
    bot[wave * 64 + lane] = u[0];
    if (wave >= 4) (wave == 4 ? top : wave == 5 ? bot + RW * 64 : side + (wave - 6) * RTILE)[lane] = ring;
    __syncthreads();
    const T below = top[wave * 64 + lane], above = bot[(wave + 1) * 64 + lane];
    int vz = 0;  // a zero in a vector register: one address for all these loads
    asm volatile("" : "+v"(vz));
    const T* sv = side + (wave * RQ + vz);
#pragma unroll
    for (int q = 0; q < RQ; ++q) {
        // two points' coefficients at a time (all 40 in flight spill)
        if (VARC && q % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        T s = coef(0, q) * u[q];
        s += coef(1, q) * lane_before(u[q], sv[q]);
        s += coef(2, q) * lane_after(u[q], sv[RTILE + q]);
        s += coef(3, q) * (q == 0 ? below : u[q > 0 ? q - 1 : 0]);
        s += coef(4, q) * (q == RQ - 1 ? above : u[q < RQ - 1 ? q + 1 : q]);
        y[q] = s;
    }
    if (!full) {
#pragma unroll
        for (int q = 0; q < RQ; ++q) y[q] = ok(q) ? y[q] : T(0);
    }
}

// Column partials of c = Vl^T r (TV the stored type), into the team's slots.
template <int RQ, class TV>
__device__ __forceinline__ void column_partials(const ResTeam& M, ResLds& S, const DevProb& P, const TV* __restrict__ V,
                                                const int (&g)[RQ], const double (&r)[RQ]) {
    const int t = threadIdx.x, lane = t & 63, wave = uniform(t >> 6), k = P.k;
    const long long ldv = P.ldv;
    for (int j0 = 0; j0 < k; j0 += 32) {
        const int nc = k - j0 < 32 ? k - j0 : 32;
        for (int j = 0; j < nc; j += 4) {
            // 32 loads in flight; columns past k re-read the last one, points
            // outside the domain point 0 (their r is zero).  The next four
            // columns' loads ahead of these sums measured slower.
            TV x[4][RQ];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const TV* Vj = V + (long long)(j0 + (j + i < nc ? j + i : nc - 1)) * ldv;
#pragma unroll
                for (int q = 0; q < RQ; ++q) x[i][q] = Vj[g[q]];
            }
            double cs[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                cs[i] = 0.0;
#pragma unroll
                for (int q = 0; q < RQ; ++q) cs[i] += (double)x[i][q] * r[q];
            }
            const double s = row_sums<4>(cs);
            if ((lane & 15) < 4) S.csh[j + (lane & 15)][wave * 4 + (lane >> 4)] = s;
        }
        __syncthreads();
        // wave w sums columns w, w + 8, ..., two of them a time (32 lanes each)
        for (int c = wave * 2; c < nc; c += 2 * RW) {
            const int cc = c + (lane >> 5);
            const double s = row_sum(S.csh[cc][lane & 31]);
            const double s0 = lane_value<0>(s) + lane_value<16>(s), s1 = lane_value<32>(s) + lane_value<48>(s);
            if ((lane & 31) == 0 && cc < nc) {
                const double v = lane ? s1 : s0;
                if (M.T == 1)
                    S.y[j0 + cc] = v;
                else
                    res_store(cpart_slot(M, M.T, j0 + cc, M.w), v);
            }
        }
        __syncthreads();
    }
}

// w = V d at this thread's points (d in S.y).
template <int RQ, class TV, class Ok>
__device__ __forceinline__ void basis_update(ResLds& S, const DevProb& P, const TV* __restrict__ V, const int (&g)[RQ],
                                             Ok ok, double (&w)[RQ]) {
    const int k = P.k;
    const long long ldv = P.ldv;
#pragma unroll
    for (int q = 0; q < RQ; ++q) w[q] = 0.0;
    for (int j = 0; j < k; j += 4) {
        TV x[4][RQ];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const TV* Vj = V + (long long)(j + i < k ? j + i : k - 1) * ldv;
#pragma unroll
            for (int q = 0; q < RQ; ++q) x[i][q] = Vj[g[q]];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double d = j + i < k ? S.y[j + i] : 0.0;
#pragma unroll
            for (int q = 0; q < RQ; ++q) w[q] += (double)x[i][q] * d;
        }
    }
#pragma unroll
    for (int q = 0; q < RQ; ++q) w[q] = ok(q) ? w[q] : 0.0;
}

// S.y = H^{-1} S.y (column-major, k <= MAXK): 16 lanes a row, 32 rows at a time,
// 8 consecutive entries a lane in flight.  (A thread a row walked its k entries 16 at a
// time, a memory latency for each 16: a boundary at 511^2 with 100 columns
// 138 us, now 135; with 30, 64.7 and 64.0; with 10 at 63^2 24.1 and 24.3.)
__device__ __forceinline__ void hinv_apply(ResLds& S, const double* __restrict__ h, int k) {
    const int t = threadIdx.x, lane = t & 15;
    double* out = S.sh;  // k values, free between exchanges
    for (int row = t >> 4; row < k; row += 32) {
        double d = 0.0;
        for (int j0 = 0; j0 < k; j0 += 128) {
            double hv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = j0 + 8 * lane + i;
                hv[i] = h[(j < k ? j : k - 1) * k + row];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = j0 + 8 * lane + i;
                d += j < k ? hv[i] * S.y[j < k ? j : 0] : 0.0;
            }
        }
        d = row_sum(d);
        if (lane == 0) out[row] = d;
    }
    __syncthreads();
    if (t < k) S.y[t] = out[t];
    __syncthreads();
}

// Start of an inner cycle (all lanes of wave 0): its tolerance, the two powers
// taken side by side by even and odd lanes, and fresh scalars.
__device__ __forceinline__ void start_cycle(ResLds& S, StepHot& N, const ResInit& in, SolveState* st, bool leader,
                                            double nu, double rho0) {
    double rt;
    const int br = cycle_choice(nu, N.nu0, N.tau, N.icyc, in.ncyc, in.precision, in.fp32_floor, rt,
                                [&](double& p1, double& p2) {
                                    const bool odd = threadIdx.x & 1;
                                    const double pw =
                                        pow(N.tau / (odd ? N.nu0 : nu), (odd ? (double)N.icyc : 1.0) /
                                                                            (double)(odd ? in.ncyc : in.ncyc - N.icyc + 1));
                                    p1 = lane_value<0>(pw);
                                    p2 = lane_value<1>(pw);
                                });
    cycle_reset(N, nu, rho0, rt);
    if (leader) {
        S.branch[br] += 1;
        if (N.icyc >= 1 && N.icyc <= NCYCLOG) st->cyc_branch[N.icyc - 1] = br;
    }
}

// A workgroup's tile of a system: points of column gx, rows gy0 + q of this
// thread, the operator's constants.
template <int RQ, bool VAR>
struct ResTile {
    int nx, ny, rows, g0;
    bool full, xin, active, var;
    long long n;
    double c0, c1, c2, c3, c4;
    const double* coef64;

    __device__ __forceinline__ void set(ResTeam& M, const DevOp& op) {
        const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));
        constexpr int H = RW * RQ;  // rows of a tile
        // read once: the exchanges' stores keep the compiler from holding them
        nx = uniform(op.nx);
        ny = uniform(op.ny);
        var = VAR && uniform(op.var);
        n = op.n;
        coef64 = op.coef64;
        c0 = uniform(op.cc[0]);
        c1 = uniform(op.cc[1]);
        c2 = uniform(op.cc[2]);
        c3 = uniform(op.cc[3]);
        c4 = uniform(op.cc[4]);
        const int ntx = (nx + RTILE - 1) / RTILE, nty = (ny + H - 1) / H;
        const int tx = M.w % ntx, ty = M.w / ntx;
        active = M.w < ntx * nty;
        M.nbr[0] = active && ty > 0 ? M.w - ntx : -1;
        M.nbr[1] = active && ty + 1 < nty ? M.w + ntx : -1;
        M.nbr[2] = active && tx > 0 ? M.w - 1 : -1;
        M.nbr[3] = active && tx + 1 < ntx ? M.w + 1 : -1;
        full = active && (tx + 1) * RTILE <= nx && (ty + 1) * H <= ny;
        const int gy0 = ty * H + wave * RQ;
        rows = active ? min(RQ, ny - gy0) : 0;
        xin = tx * RTILE + lane < nx;
        g0 = gy0 * nx + tx * RTILE + lane;
    }
    __device__ __forceinline__ bool ok(int q) const { return xin && q < rows; }
    // indices of this thread's points (0 outside the domain)
    __device__ __forceinline__ void points(int (&g)[RQ]) const {
        const int g1 = opaque(g0);
#pragma unroll
        for (int q = 0; q < RQ; ++q) g[q] = ok(q) ? g1 + q * nx : 0;
    }
    __device__ __forceinline__ double cc(int o) const {
        return o == 0 ? c0 : o == 1 ? c1 : o == 2 ? c2 : o == 3 ? c3 : c4;
    }
    // y = A u in float64
    __device__ __forceinline__ void stencil64(ResLds& S, const double (&u)[RQ], double ring, double (&y)[RQ]) const {
        auto okq = [&](int q) { return ok(q); };
        if (VAR && var) {
            const int g1 = opaque(g0);
            tile_stencil<double, VAR>(S, u, ring, full, okq,
                                      [&](int o, int q) { return coef64[o * n + (ok(q) ? g1 + q * nx : 0)]; }, y);
        } else {
            tile_stencil<double, false>(S, u, ring, full, okq, [&](int o, int) { return cc(o); }, y);
        }
    }
};

// A solve's state at its start (thread 0).
__device__ __forceinline__ void res_begin(ResLds& S, const ResInit& in) {
    S.hot = StepHot{};
    S.hot.first = 1;
    S.hot.icyc = in.icyc0;
    S.hot.solve_state = SV_RUNNING;
    S.mvp_inner = S.iters_total = S.mvp_boundary = S.nproj = 0;
    S.nu_final = 0.0;
    S.nhist = 0;
    S.branch[0] = S.branch[1] = S.branch[2] = S.branch[3] = 0;
}

// The report's part of a finished solve (the leader).
__device__ __forceinline__ void res_end(ResLds& S, SolveState* st, int iter, int inner) {
    const StepHot N = S.hot;
    st->solve_state = N.solve_state;
    st->inner_state = inner;
    st->icyc = N.icyc;
    st->iter = iter;
    st->tau = N.tau;
    st->bnorm = N.bnorm;
    st->nu0 = N.nu0;
    st->nu_final = S.nu_final;
    for (int i = 0; i < 4; ++i) st->branch[i] = S.branch[i];
    st->mvp_inner = S.mvp_inner;
    st->iters_total = S.iters_total;
    st->mvp_boundary = S.mvp_boundary;
    st->nproj = S.nproj;
    st->nhist = S.nhist;
}

// A cycle boundary: x += upd (any: there is an update), the true residual,
// its tests, the projection and the next cycle's tolerance.  iter0: the
// finished cycle made no usable iteration; iter, inner: what is logged of it.
// Returns 0 with the new residual r64 and its ring values (inner type, ring),
// 1 when the solve has ended, -1 when the grid aborts.
template <class TI, int RQ, bool VAR, class Upd>
__device__ __forceinline__ int res_boundary(ResTeam& M, ResLds& S, const ResArgs& A, const DevProb& P, int k,
                                            const ResTile<RQ, VAR>& tl, bool leader, Upd upd, bool any, bool iter0,
                                            int iter, int inner, double (&r64)[RQ], TI (&r)[RQ], double& ring) {
    const int t = threadIdx.x, lane = t & 63, wave = uniform(t >> 6);
    SolveState* st = P.st;
    const bool zero_start = A.init.zero_start != 0;
    const TI none[RQ] = {};
    double dummy = 0.0;
    for (bool last = false;;) {  // last: only the final true residual is left to form
        double xr[RQ], y64[RQ], a1[1] = {0.0}, s1[1];
        int g[RQ];
        tl.points(g);
        ring = 0.0;
#pragma unroll
        for (int q = 0; q < RQ; ++q) {
            xr[q] = tl.ok(q) && !(zero_start && S.hot.first) ? res_quiet(P.x[g[q]]) : 0.0;
            if (any) xr[q] += upd(q);
            if (tl.ok(q) && (any || (zero_start && S.hot.first))) P.x[g[q]] = xr[q];
        }
        if (exchange<1, true>(M, S, a1, xr, ring, s1)) return -1;
        tl.stencil64(S, xr, ring, y64);
        double a3[3] = {0.0, 0.0, 0.0}, s3[3];
#pragma unroll
        for (int q = 0; q < RQ; ++q) {
            const double b = tl.ok(q) ? P.b[g[q]] : 0.0;
            r64[q] = b - y64[q];
            a3[0] += r64[q] * r64[q];
            a3[1] += b * b;
            r[q] = (TI)r64[q];
            a3[2] += (double)r[q] * (double)r[q];
        }
        if (k == 0) {
            if (exchange<3, true>(M, S, a3, r, ring, s3)) return -1;
        } else {
            if (exchange<3, false>(M, S, a3, none, dummy, s3)) return -1;
        }
        if (last) {
            if (t == 0) S.nu_final = sqrt(s3[0]);
            return 1;
        }
        if (wave == 0) {
            StepHot H = S.hot;
            H.iter = iter0 ? 0 : 1;
            H.inner_state = inner;
            StepHot N = H;
            const double nu = sqrt(s3[0]);
            boundary_tests(H, N, &A.init, nu, s3[1]);
            if (leader && !H.first && H.icyc >= 1 && H.icyc <= NCYCLOG) {
                st->cyc_iters[H.icyc - 1] = iter;
                st->cyc_end[H.icyc - 1] = inner;
            }
            if (N.solve_state == SV_RUNNING && k == 0) start_cycle(S, N, A.init, st, leader, nu, s3[2]);
            if (lane == 0) {
                S.mvp_boundary += 1;
                S.nu_final = nu;
                S.stop = N.solve_state != SV_RUNNING;
                S.hot = N;
            }
        }
        __syncthreads();
        if (S.stop) return 1;
        if (k == 0) return 0;
        // projection: c = Vl^T r, d = H^{-1} c, x += V d, r -= A V d
        if (P.vtype)
            column_partials(M, S, P, reinterpret_cast<const float*>(P.Vl), g, r64);
        else
            column_partials(M, S, P, reinterpret_cast<const double*>(P.Vl), g, r64);
        if (M.T > 1) {
            for (int c = M.w + M.T * wave; c < k; c += M.T * RW) {
                const u64* ps[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    ps[i] = i * 64 + lane < M.T ? cpart_slot(M, M.T, c, i * 64 + lane) : nullptr;
                double x[4];
                res_poll<4>(ps, x, M.abort_word, &S.dead);
                const double s = wave_sum_dpp((x[0] + x[1]) + (x[2] + x[3]));
                if (lane == 0) res_store(cval_slot(M, M.T, A.kmax, c), s);
            }
            if (t < k) S.y[t] = res_poll(cval_slot(M, M.T, A.kmax, t), M.abort_word, &S.dead);
            __syncthreads();
            if (S.dead) return -1;
        }
        hinv_apply(S, P.hinv, k);
        double w[RQ];
        auto okq = [&](int q) { return tl.ok(q); };
        if (P.vtype)
            basis_update(S, P, reinterpret_cast<const float*>(P.V), g, okq, w);
        else
            basis_update(S, P, reinterpret_cast<const double*>(P.V), g, okq, w);
        if (exchange<1, true>(M, S, a1, w, ring, s1)) return -1;
        // every workgroup has read the coefficients: empty them
        if (t < k && M.T > 1) {
            res_store_bits(cpart_slot(M, M.T, t, M.w), RES_EMPTY);
            if (t % M.T == M.w) res_store_bits(cval_slot(M, M.T, A.kmax, t), RES_EMPTY);
        }
        tl.stencil64(S, w, ring, y64);
        double a2[2] = {0.0, 0.0}, s2[2];
#pragma unroll
        for (int q = 0; q < RQ; ++q) {
            if (tl.ok(q)) P.x[g[q]] = xr[q] + w[q];
            r64[q] -= y64[q];
            a2[0] += r64[q] * r64[q];
            r[q] = (TI)r64[q];
            a2[1] += (double)r[q] * (double)r[q];
        }
        if (exchange<2, true>(M, S, a2, r, ring, s2)) return -1;
        if (wave == 0) {
            StepHot N = S.hot;
            const double nu = sqrt(s2[0]);
            if (!isfinite(nu))
                N.solve_state = SV_NONFINITE;
            else if (nu <= N.tau)
                N.solve_state = SV_CONVERGED;
            if (N.solve_state == SV_RUNNING) start_cycle(S, N, A.init, st, leader, nu, s2[1]);
            if (lane == 0) {
                S.mvp_boundary += 1;
                S.nproj += 1;
                S.stop = N.solve_state != SV_RUNNING;
                S.hot = N;
            }
        }
        __syncthreads();
        if (!S.stop) return 0;
        last = true;  // the solve ends here: form b - A x afresh
        any = false;
    }
}

// This workgroup's team and place in it.
__device__ __forceinline__ void res_place(ResTeam& M, const ResArgs& A) {
    const int team = blockIdx.x / A.team;
    M.T = A.team;
    M.w = blockIdx.x - team * A.team;
    M.ph = 0;
    M.base = (u64*)A.xch + (size_t)team * A.xstride;
    M.abort_word = A.ctl + 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) M.nbr[i] = -1;
}

static __device__ __attribute__((noinline)) bool res_gate_call(unsigned* word, unsigned team) {
    return res_gate(word, team);
}

// Whether the team begins (its gate is word 2 + team of A.ctl).  Where a kernel
// enters and whether the gate is a CALL is a matter of registers: past the gate's
// atomics the compiler no longer takes what it reads for unchanged.  The IDR kernels
// enter after they have read their descriptor (first, the 64-row ones of coefficient
// arrays spill 186 registers instead of 144), the others first; the Arnoldi kernels
// through a call (64 rows, inlined: 60 instead of 42, 2 % of a cycle at 1023^2),
// BiCGStab's without (with it 1 % of a solve with coefficient arrays).
template <bool CALL>
__device__ __forceinline__ bool res_enter(const ResTeam& M, ResLds& S, const ResArgs& A) {
    if (threadIdx.x == 0) {
        unsigned* word = A.ctl + 2 + blockIdx.x / A.team;
        S.dead = 0;
        S.stop = !(CALL ? res_gate_call(word, (unsigned)M.T) : res_gate(word, (unsigned)M.T));
    }
    __syncthreads();
    return uniform(S.stop) == 0;
}

}  // namespace tgdk
