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

#include "resident.h"
#include "step_kernel.h"

namespace tgdk {

constexpr int RT = 512;                   // threads
constexpr int RW = RT / 64;               // waves
constexpr int RQ = 8;                     // points per thread (rows 8 w .. 8 w + 7 of wave w)
constexpr int RTILE = 64;                 // tile side
constexpr int RHALO = 4 * RTILE;          // edge values of a tile

static_assert(RES_TILE == RTILE && RES_NSUM >= 5, "host layout");

template <bool VAR, class TI>
struct ResLds {
    TI coef[VAR ? 4 : 1][VAR ? RTILE * RTILE : 1];  // C, W, E, S of the tile
    double top[RW + 1][64];  // [w + 1]: last row of wave w; [0]: the ring row below the tile
    double bot[RW + 1][64];  // [w]: first row of wave w; [RW]: the ring row above the tile
    double side[2][RTILE];   // ring columns west and east
    double csh[64][4 * RW + 1];  // column partials of the waves' rows
    double sh[RES_NSUM * 4 * RW];
    double red[RES_NSUM];
    double y[MAXK + 1];
    StepHot hot;
    long long mvp_inner, iters_total;
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
    return M.base + (unsigned)(3 * RES_NSUM * round64(T) + (buf * RES_COPIES + copy) * 8 + v);
}
__device__ __forceinline__ u64* halo_slot(const ResTeam& M, int T, int buf, int w, int side, int i) {
    return M.base + (unsigned)(3 * RES_NSUM * round64(T) + 3 * RES_COPIES * 8 + ((buf * T + w) * 4 + side) * RTILE + i);
}
__device__ __forceinline__ u64* cpart_slot(const ResTeam& M, int T, int c, int w) {
    return M.base + (unsigned)(3 * RES_NSUM * round64(T) + 3 * RES_COPIES * 8 + 3 * T * RHALO + c * round64(T) + w);
}
__device__ __forceinline__ u64* cval_slot(const ResTeam& M, int T, int kmax, int c) {
    return cpart_slot(M, T, kmax, 0) + c;
}

// One phase's exchange: the team's sums of a[] into tot[], and, with HALO,
// this tile's edge values y published and the ring values (waves 4..7: side
// wave - 4, position lane) returned in ring.  Wave v handles value v.  A team
// of one takes its own sums; up to 32 workgroups every one reads all partial
// sums, beyond (33 to 256) workgroup v T / 8 gathers value v and all read its
// total; the sums have the same order, hence the same bits, either way.
// True if the grid aborted.
constexpr int RES_DIRECT = 32;
template <int NV, bool HALO, class LDS, class TY>
__device__ __forceinline__ bool exchange(ResTeam& M, LDS& S, const double (&a)[NV], const TY (&y)[RQ], double& ring,
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
    const int own = T > RES_DIRECT ? wave * (T / 8) : -1;  // the workgroup that gathers value `wave`
    if (wave < NV) {
        const double s = lanes32_sum(S.sh[wave * 4 * RW + (lane & 31)]);
        if (lane == 0) {
            if (T == 1)
                S.red[wave] = s;
            else
                res_store(sum_slot(M, T, buf, wave, M.w), s);
        }
        if (T > 1 && (T <= RES_DIRECT || own == M.w)) {
            const u64* ps[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) ps[c] = c * 64 + lane < T ? sum_slot(M, T, buf, wave, c * 64 + lane) : nullptr;
            double x[4];
            res_poll<4>(ps, x, M.abort_word, &S.dead);
            const double g = wave_sum_dpp((x[0] + x[1]) + (x[2] + x[3]));
            if (T <= RES_DIRECT) {
                if (lane == 0) S.red[wave] = g;
            } else if (lane < RES_COPIES) {
                res_store(total_slot(M, T, buf, wave, lane), g);
            }
        }
    }
    if (T > 1) {
        if (HALO && wave >= 4) {
            const int side = wave - 4;
            const int nb = side == 0 ? M.nbr[0] : side == 1 ? M.nbr[1] : side == 2 ? M.nbr[2] : M.nbr[3];
            ring = nb >= 0 ? res_poll(halo_slot(M, T, buf, nb, side ^ 1, lane), M.abort_word, &S.dead) : 0.0;
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
    if (wave < RES_NSUM && own == M.w && lane < RES_COPIES) res_store_bits(total_slot(M, T, old, wave, lane), RES_EMPTY);
    if (wave < 4) res_store_bits(halo_slot(M, T, old, M.w, wave, lane), RES_EMPTY);
    ++M.ph;
    return dead;
}

// y = A u on the tile: u in registers, ring the ring values (waves 4..7, side
// wave - 4).  coef(o, q): coefficient o (C, W, E, S, N) at point q.  Points
// outside the domain give 0.  Ends without a barrier (the next exchange has
// two).
template <class T, bool VARC, class LDS, class Ok, class F>
__device__ __forceinline__ void tile_stencil(LDS& S, const T (&u)[RQ], T ring, bool full, Ok ok,
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
template <class TV, class LDS>
__device__ __forceinline__ void column_partials(const ResTeam& M, LDS& S, const DevProb& P, const TV* __restrict__ V,
                                                const int (&g)[RQ], const double (&r)[RQ]) {
    const int t = threadIdx.x, lane = t & 63, wave = uniform(t >> 6), k = P.k;
    const long long ldv = P.ldv;
    for (int j0 = 0; j0 < k; j0 += 64) {
        const int nc = k - j0 < 64 ? k - j0 : 64;
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
template <class TV, class LDS, class Ok>
__device__ __forceinline__ void basis_update(LDS& S, const DevProb& P, const TV* __restrict__ V, const int (&g)[RQ],
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

// Start of an inner cycle (all lanes of wave 0): the tolerance of
// cycle_tolerance with its two powers taken side by side by even and odd
// lanes, and fresh scalars.
template <class LDS>
__device__ __forceinline__ void start_cycle(LDS& S, StepHot& N, const ResInit& in, SolveState* st, bool leader,
                                            double nu, double rho0) {
    int br;
    double rt;
    if (N.icyc > in.ncyc) {
        rt = N.tau / nu;
        br = 3;
    } else {
        const bool odd = threadIdx.x & 1;
        const double pw = pow(N.tau / (odd ? N.nu0 : nu),
                              (odd ? (double)N.icyc : 1.0) / (double)(odd ? in.ncyc : in.ncyc - N.icyc + 1));
        const double t1 = lane_value<0>(pw), t2 = (N.nu0 / nu) * lane_value<1>(pw);
        br = t1 <= t2 ? 1 : 2;
        rt = br == 1 ? t1 : t2;
    }
    if (in.precision == 1 && rt < in.fp32_floor) rt = in.fp32_floor;
    cycle_reset(N, nu, rho0, rt);
    if (leader) {
        S.branch[br] += 1;
        if (N.icyc >= 1 && N.icyc <= NCYCLOG) st->cyc_branch[N.icyc - 1] = br;
    }
}

template <bool VAR, class TI>
__global__ __launch_bounds__(RT) void k_resident2d(ResArgs A) {
    __shared__ ResLds<VAR, TI> S;
    static_assert(RT == 64 * RW && RW * RQ == RTILE, "tile rows");
    const int t = threadIdx.x, lane = t & 63, wave = uniform(t >> 6);
    ResTeam M;
    const int team = blockIdx.x / A.team;
    M.T = A.team;
    M.w = blockIdx.x - team * A.team;
    M.ph = 0;
    M.base = (u64*)A.xch + (size_t)team * A.xstride;
    M.abort_word = A.ctl + 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) M.nbr[i] = -1;
    if (t == 0) S.dead = 0;
    __syncthreads();
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
        const DevOp& op = P.op;
        SolveState* st = P.st;
        // read once: the exchanges' stores keep the compiler from holding them
        const int nx = uniform(op.nx), ny = uniform(op.ny), k = uniform(P.k), maxit = A.init.maxit;
        const bool var = VAR && uniform(op.var);
        const long long n = op.n;
        const double c0 = uniform(op.cc[0]), c1 = uniform(op.cc[1]), c2 = uniform(op.cc[2]), c3 = uniform(op.cc[3]),
                     c4 = uniform(op.cc[4]);
        auto cc = [&](int o) { return o == 0 ? c0 : o == 1 ? c1 : o == 2 ? c2 : o == 3 ? c3 : c4; };
        const int ntx = (nx + RTILE - 1) / RTILE, nty = (ny + RTILE - 1) / RTILE;
        const int tx = M.w % ntx, ty = M.w / ntx;
        const bool active = M.w < ntx * nty;
        M.nbr[0] = active && ty > 0 ? M.w - ntx : -1;
        M.nbr[1] = active && ty + 1 < nty ? M.w + ntx : -1;
        M.nbr[2] = active && tx > 0 ? M.w - 1 : -1;
        M.nbr[3] = active && tx + 1 < ntx ? M.w + 1 : -1;
        const bool leader = M.w == 0 && t == 0;
        const bool zero_start = A.init.zero_start != 0;
        // this thread's points: column gx, rows gy0 + q, the first `rows` of them inside
        const bool full = active && (tx + 1) * RTILE <= nx && (ty + 1) * RTILE <= ny;
        const int gy0 = ty * RTILE + wave * RQ;
        const int rows = active ? min(RQ, ny - gy0) : 0;
        const bool xin = tx * RTILE + lane < nx;
        const int g0 = gy0 * nx + tx * RTILE + lane;
        auto ok = [&](int q) { return xin && q < rows; };
        // their indices (0 outside the domain)
        auto points = [&](int (&g)[RQ]) {
            const int g1 = opaque(g0);
#pragma unroll
            for (int q = 0; q < RQ; ++q) g[q] = ok(q) ? g1 + q * nx : 0;
        };
        // VAR kernels hold C, W, E, S of the tile in LDS in the inner type
        // (an operator without coefficient arrays fills in its constants) and
        // N in registers, loaded before the exchange ahead of each stencil
        const TI* cf = nullptr;
        if (VAR) {
            if (var) cf = uniform(coef_ptr<TI>(op));
            int g[RQ];
            points(g);
#pragma unroll
            for (int q = 0; q < RQ; ++q)
#pragma unroll
                for (int o = 0; o < 4; ++o)
                    S.coef[VAR ? o : 0][VAR ? (wave * RQ + q) * 64 + lane : 0] = var ? cf[o * n + g[q]] : (TI)cc(o);
        }
        TI nq[VAR ? RQ : 1];
        auto load_n = [&]() {
            if constexpr (VAR) {
                const int g1 = opaque(g0);
                const char* cn = (const char*)(cf + 4 * n);
#pragma unroll
                for (int q = 0; q < RQ; ++q) {
                    nq[q] = (TI)c4;
                    if (var) nq[q] = *(const TI*)(cn + (unsigned)((ok(q) ? g1 + q * nx : 0) * (int)sizeof(TI)));
                }
            }
        };
        auto cin = [&](int o, int q) -> TI {
            if constexpr (VAR) return o < 4 ? S.coef[o < 4 ? o : 0][(wave * RQ + q) * 64 + lane] : nq[q];
            return (TI)cc(o);
        };
        // y = A u in float64 (the cycle boundary)
        auto stencil64 = [&](const double(&u)[RQ], double ring, double(&y)[RQ]) {
            if (VAR && var) {
                const double* c = op.coef64;
                const int g1 = opaque(g0);
                tile_stencil<double, VAR>(S, u, ring, full, ok,
                                          [&](int o, int q) { return c[o * n + (ok(q) ? g1 + q * nx : 0)]; }, y);
            } else {
                tile_stencil<double, false>(S, u, ring, full, ok, [&](int o, int) { return cc(o); }, y);
            }
        };
        if (t == 0) {
            S.hot = StepHot{};
            S.hot.first = 1;
            S.hot.icyc = A.init.icyc0;
            S.hot.solve_state = SV_RUNNING;
            S.mvp_inner = 0;
            S.iters_total = 0;
            S.nhist = 0;
            S.branch[0] = S.branch[1] = S.branch[2] = S.branch[3] = 0;
        }
        long long mvp_boundary = 0, nproj = 0;
        double nu_final = 0.0;
        bool last = false;  // only the final true residual is left to form
        __syncthreads();
        TI r[RQ], p[RQ], v[RQ], e[RQ], h[RQ], s[RQ];
#pragma unroll
        for (int q = 0; q < RQ; ++q) r[q] = p[q] = v[q] = e[q] = h[q] = s[q] = TI(0);
        double upd_a = 0.0, upd_w = 0.0;  // pending update e + a p + w s
        int upd_any = 0;
        int iter = 0, inner = IN_CONVERGED;
        for (;;) {
            // ---------------------------------------- true residual
            double xr[RQ], r64[RQ], y64[RQ], ring = 0.0, a1[1] = {0.0}, s1[1];
            int g[RQ];
            points(g);
#pragma unroll
            for (int q = 0; q < RQ; ++q) {
                xr[q] = ok(q) && !(zero_start && S.hot.first) ? res_quiet(P.x[g[q]]) : 0.0;
                if (upd_any) {
                    double u = (double)e[q];
                    if (upd_a != 0.0) u += upd_a * (double)p[q];
                    if (upd_w != 0.0) u += upd_w * (double)s[q];
                    xr[q] += u;
                }
                if (ok(q) && (upd_any || (zero_start && S.hot.first))) P.x[g[q]] = xr[q];
            }
            if (exchange<1, true>(M, S, a1, xr, ring, s1)) return;
            stencil64(xr, ring, y64);
            double a3[3] = {0.0, 0.0, 0.0}, s3[3];
#pragma unroll
            for (int q = 0; q < RQ; ++q) {
                const double b = ok(q) ? P.b[g[q]] : 0.0;
                r64[q] = b - y64[q];
                a3[0] += r64[q] * r64[q];
                a3[1] += b * b;
                r[q] = (TI)r64[q];
                a3[2] += (double)r[q] * (double)r[q];
            }
            if (k == 0) {
                if (exchange<3, true>(M, S, a3, r, ring, s3)) return;
            } else {
                if (exchange<3, false>(M, S, a3, r, dummy, s3)) return;
            }
            if (last) {
                nu_final = sqrt(s3[0]);
                break;
            }
            ++mvp_boundary;
            if (wave == 0) {
                StepHot H = S.hot;
                H.iter = iter;
                H.inner_state = inner;
                StepHot N = H;
                const double nu = sqrt(s3[0]);
                nu_final = nu;
                boundary_tests(H, N, &A.init, nu, s3[1]);
                if (leader && !H.first && H.icyc >= 1 && H.icyc <= NCYCLOG) {
                    st->cyc_iters[H.icyc - 1] = H.iter;
                    st->cyc_end[H.icyc - 1] = H.inner_state;
                }
                if (N.solve_state == SV_RUNNING && k == 0) start_cycle(S, N, A.init, st, leader, nu, s3[2]);
                if (lane == 0) {
                    S.stop = N.solve_state != SV_RUNNING;
                    S.hot = N;
                }
            }
            __syncthreads();
            if (S.stop) break;
            // ---------------------------------------- projection
            if (k > 0) {
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
                    if (S.dead) return;
                }
                double d = 0.0;
                if (t < k) {
                    // 16 entries of a row of H^{-1} in flight (past k: the last one again, masked)
                    const double* hi = P.hinv + t;
                    for (int j0 = 0; j0 < k; j0 += 16) {
                        double hv[16];
#pragma unroll
                        for (int j = 0; j < 16; ++j) hv[j] = hi[(j0 + j < k ? j0 + j : k - 1) * k];
#pragma unroll
                        for (int j = 0; j < 16; ++j) d += j0 + j < k ? hv[j] * S.y[j0 + j < k ? j0 + j : 0] : 0.0;
                    }
                }
                __syncthreads();
                if (t < k) S.y[t] = d;
                __syncthreads();
                double w[RQ];
                if (P.vtype)
                    basis_update(S, P, reinterpret_cast<const float*>(P.V), g, ok, w);
                else
                    basis_update(S, P, reinterpret_cast<const double*>(P.V), g, ok, w);
                if (exchange<1, true>(M, S, a1, w, ring, s1)) return;
                // every workgroup has read the coefficients: empty them
                if (t < k && M.T > 1) {
                    res_store_bits(cpart_slot(M, M.T, t, M.w), RES_EMPTY);
                    if (t % M.T == M.w) res_store_bits(cval_slot(M, M.T, A.kmax, t), RES_EMPTY);
                }
                stencil64(w, ring, y64);
                double a2[2] = {0.0, 0.0}, s2[2];
#pragma unroll
                for (int q = 0; q < RQ; ++q) {
                    if (ok(q)) P.x[g[q]] = xr[q] + w[q];
                    r64[q] -= y64[q];
                    a2[0] += r64[q] * r64[q];
                    r[q] = (TI)r64[q];
                    a2[1] += (double)r[q] * (double)r[q];
                }
                if (exchange<2, true>(M, S, a2, r, ring, s2)) return;
                ++mvp_boundary;
                ++nproj;
                if (wave == 0) {
                    StepHot N = S.hot;
                    const double nu = sqrt(s2[0]);
                    if (!isfinite(nu))
                        N.solve_state = SV_NONFINITE;
                    else if (nu <= N.tau)
                        N.solve_state = SV_CONVERGED;
                    if (N.solve_state == SV_RUNNING) start_cycle(S, N, A.init, st, leader, nu, s2[1]);
                    if (lane == 0) {
                        S.stop = N.solve_state != SV_RUNNING;
                        S.hot = N;
                    }
                }
                __syncthreads();
                if (S.stop) {  // the solve ends here: form b - A x afresh
                    last = true;
                    upd_any = 0;
                    continue;
                }
            }
            // ---------------------------------------- inner cycle
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
                tile_stencil<TI, VAR>(S, p, rp, full, ok, cin, v);
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
                tile_stencil<TI, VAR>(S, s, rr, full, ok, cin, tv);
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
        if (leader) {
            const StepHot N = S.hot;
            st->solve_state = N.solve_state;
            st->inner_state = inner;
            st->icyc = N.icyc;
            st->iter = iter;
            st->tau = N.tau;
            st->bnorm = N.bnorm;
            st->nu0 = N.nu0;
            st->nu_final = nu_final;
            for (int i = 0; i < 4; ++i) st->branch[i] = S.branch[i];
            st->mvp_inner = S.mvp_inner;
            st->iters_total = S.iters_total;
            st->mvp_boundary = mvp_boundary;
            st->nproj = nproj;
            st->nhist = S.nhist;
        }
        __syncthreads();
    }
}

// Empties the exchange regions, stores the descriptors that came as
// arguments and writes every system's initial state.
__global__ __launch_bounds__(256) void k_res_setup(ResArgs A, ResProbs Q, long long words) {
    u64* x = (u64*)A.xch;
    for (long long i = blockIdx.x * 256LL + threadIdx.x; i < words; i += gridDim.x * 256LL) x[i] = RES_EMPTY;
    if (blockIdx.x == 0 && threadIdx.x < 2) A.ctl[threadIdx.x] = 0;
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

hipError_t launch_resident2d(int inner_f32, int var, const ResArgs& args, const DevProb* probs, int teams,
                             hipStream_t s) {
    const long long words = (long long)args.xstride * teams;
    const long long nb = (words + 1023) / 1024;
    ResProbs q;
    memset(&q, 0, sizeof(q));
    for (int j = 0; args.upload && j < args.nprob; ++j) q.p[j] = probs[j];
    hipLaunchKernelGGL(k_res_setup, dim3((unsigned)(nb < 1024 ? nb : 1024)), dim3(256), 0, s, args, q, words);
    ResArgs a = args;
    void* av[] = {&a};
    const void* f = inner_f32 ? (var ? (const void*)k_resident2d<true, float> : (const void*)k_resident2d<false, float>)
                              : (var ? (const void*)k_resident2d<true, double> : (const void*)k_resident2d<false, double>);
    return hipLaunchCooperativeKernel(f, dim3(teams * args.team), dim3(RT), av, 0, s);
}

}  // namespace tgdk
