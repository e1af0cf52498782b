// Arnoldi steps of GMRES-Proj and coarse GMRES-DR on 2-D grids of up to one
// tile per compute unit, a whole cycle's steps in one launch: w = A v_j, two
// classical Gram-Schmidt passes (the ones of k_gsc, kernels_dense.hip), the norm
// and v_(j+1).
//
// As launches a step is eight of them (stencil, three passes over V, three
// sums of partials, the scaling), 75 us at 255^2 with 55 columns of which the
// passes' bytes need about 12.  Here a workgroup owns a tile of 64 x 8 RQ
// points: w stays in LDS, v_j in registers with its ring values, V streams from
// memory (a workgroup only ever reads the rows it owns, so its columns' tiles
// sit in its XCD's L2 when they fit).  The columns are split over the eight
// waves as in k_gsc, a pass reads V once.  The sums of a pass go over the team
// in two hops (workgroup w gathers columns w, w + T, ..., all read the totals;
// in one, up to 8 workgroups: 31^2, 30 columns, 17.5 -> 16.3 us a step);
// the norm's exchange carries w's edge values, from which every workgroup scales
// its own ring.  A pass at 1023^2 with 40 columns is bound by V's 340 MB from
// the memory side cache: rows are walked up and down in turn so that the next
// pass begins with the rows the last one left in L2.  Microseconds a step, as
// launches and here: 31^2 32 and 16, 127^2 35 and 23, 511^2 67 and 45,
// 1023^2 171 and 139.
#include "resident2d.h"

namespace tgdk {

constexpr int ARN_PMAX = 128;  // most columns of a step
constexpr int ARN_DIRECT = 8;  // teams up to here read each other's sums directly, in one hop

template <int RQ>
struct ArnLds : ResLds {
    double w[RW * RQ][64];
    double xs[2][RW][8][64];  // the waves' shares of V h for up to 8 rows
    double h[ARN_PMAX];
};

// One pass over the first p columns of V against w: wave `wave` holds columns
// wave, wave + 8, ..., CPW of them, of RB = 32 / CPW (at most 8) of the tile's
// rows at a time, the next rows' loads issued before the current ones are
// used (128 KB in flight a compute unit; with one row at a time a pass at
// 1023^2 was latency bound: 181 us a step).
//   MODE 0: V^T w;  MODE 1: w -= V h, then V^T w;  MODE 2: w -= V h, then w.w
// The update of a row needs all columns: the waves' shares of V h meet in LDS,
// one wave a row sums them in order and stores the row.  Sums of MODE 0 and 1
// go to the team's slots; MODE 2 returns this thread's share of w.w.
template <int MODE, int CPW, int RQ>
__device__ __forceinline__ double gs_tile_pass(ArnLds<RQ>& S, const ResTeam& M, const double* V, long long n, int p,
                                               int nx, int g0, int rows, bool xin, u64* slots, bool rev) {
    constexpr int RB = 32 / CPW < 8 ? 32 / CPW : 8;
    const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));
    double hc[CPW], acc[CPW];
    const double* vc[CPW];
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = wave + RW * i;
        vc[i] = V + (long long)(c < p ? c : 0) * n;  // past p: column 0 again, masked
        hc[i] = MODE >= 1 && c < p ? S.h[c] : 0.0;
        acc[i] = 0.0;
    }
    auto at = [&](int i) { return rev ? rows - 1 - i : i; };  // the i-th row of this pass
    auto load = [&](int r0, double(&d)[RB][CPW]) {
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int row = at(r0 + b < rows ? r0 + b : rows - 1);  // past the tile: its last row again, masked
            const int g = g0 + row * nx;
#pragma unroll
            for (int i = 0; i < CPW; ++i) d[b][i] = vc[i][g];
        }
    };
    double nacc = 0.0, vv[RB][CPW], nv[RB][CPW];
    if (rows > 0) load(0, vv);
    int par = 0;
    for (int r0 = 0; r0 < rows; r0 += RB) {
        if (r0 + RB < rows) load(r0 + RB, nv);
        if (MODE >= 1) {
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                double u = 0.0;
#pragma unroll
                for (int i = 0; i < CPW; ++i) u += vv[b][i] * hc[i];
                S.xs[par][wave][b][lane] = u;
            }
            __syncthreads();
            if (wave < RB && r0 + wave < rows) {
                double s = S.xs[par][0][wave][lane];
#pragma unroll
                for (int q = 1; q < RW; ++q) s += S.xs[par][q][wave][lane];
                const double x = xin ? S.w[at(r0 + wave)][lane] - s : 0.0;
                S.w[at(r0 + wave)][lane] = x;
                if (MODE == 2) nacc += x * x;
            }
            par ^= 1;
            if (MODE == 1) __syncthreads();
        }
        if (MODE <= 1) {
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const double x = r0 + b < rows ? S.w[at(r0 + b < rows ? r0 + b : 0)][lane] : 0.0;
#pragma unroll
                for (int i = 0; i < CPW; ++i) acc[i] += vv[b][i] * x;
            }
        }
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int i = 0; i < CPW; ++i) vv[b][i] = nv[b][i];
    }
    if (MODE <= 1) {
#pragma unroll
        for (int i0 = 0; i0 < CPW; i0 += 4) {
            double s;
            if constexpr (CPW >= 4)
                s = row_sums<4>(acc + i0);
            else
                s = row_sums<CPW>(acc + i0);
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            const int c = wave + RW * (i0 + lane);
            if (lane < (CPW < 4 ? CPW : 4) && c < p) {
                if (M.T == 1)
                    S.h[c] = s;
                else
                    res_store(slots + (unsigned)(c * round64(M.T)) + M.w, s);
            }
        }
    }
    return nacc;
}

template <int MODE, int RQ>
__device__ __forceinline__ double gs_tile(ArnLds<RQ>& S, const ResTeam& M, const double* V, long long n, int p, int nx,
                                          int g0, int rows, bool xin, u64* slots, bool rev) {
    if (p <= RW) return gs_tile_pass<MODE, 1, RQ>(S, M, V, n, p, nx, g0, rows, xin, slots, rev);
    if (p <= 2 * RW) return gs_tile_pass<MODE, 2, RQ>(S, M, V, n, p, nx, g0, rows, xin, slots, rev);
    if (p <= 4 * RW) return gs_tile_pass<MODE, 4, RQ>(S, M, V, n, p, nx, g0, rows, xin, slots, rev);
    if (p <= 8 * RW) return gs_tile_pass<MODE, 8, RQ>(S, M, V, n, p, nx, g0, rows, xin, slots, rev);
    return gs_tile_pass<MODE, 16, RQ>(S, M, V, n, p, nx, g0, rows, xin, slots, rev);
}

template <bool VAR, int RQ>
__global__ __launch_bounds__(RT) void k_arnoldi2d(ArnArgs A) {
    __shared__ ArnLds<RQ> S;
    const int t = threadIdx.x, lane = t & 63, wave = uniform((int)(t >> 6));
    ResTeam M;
    {
        ResArgs ra{};
        ra.team = A.team;
        ra.xstride = 0;
        ra.xch = A.xch;
        ra.ctl = A.ctl;
        res_place(M, ra);
        if (!res_enter<true>(M, S, ra)) return;
        if (M.w == 0 && t == 0) A.ctl[0] = 1;  // begun
    }
    ResTile<RQ, VAR> tl;
    tl.set(M, A.op);
    const int nx = tl.nx;
    const long long n = tl.n;
    // the tile's rows as the passes walk them
    const int ntx = (nx + RTILE - 1) / RTILE, ty = M.w / ntx;
    const int rows = tl.active ? min(RW * RQ, tl.ny - ty * RW * RQ) : 0;
    // (a lane past the grid reads the row's last point, its w is zero: any other
    // workgroup's point may still hold what the memory held before)
    const int gt = ty * RW * RQ * nx + min((M.w % ntx) * RTILE + lane, nx - 1);
    const bool xin = tl.xin && tl.active;
    u64* bank[2] = {cpart_slot(M, M.T, 0, 0), cpart_slot(M, M.T, A.pmax, 0)};
    u64* vals[2] = {cpart_slot(M, M.T, 2 * A.pmax, 0), cpart_slot(M, M.T, 2 * A.pmax, 0) + A.pmax};
    // a pass's sums over the team, into S.h (all have them when it returns)
    auto totals = [&](int b, int p, double* out) -> bool {
        if (M.T > 1 && M.T <= ARN_DIRECT) {
            __syncthreads();  // S.h of the pass before has been read
            if (t < p) {
                const u64* ps[ARN_DIRECT];
                double x[ARN_DIRECT], s = 0.0;
#pragma unroll
                for (int i = 0; i < ARN_DIRECT; ++i) ps[i] = i < M.T ? bank[b] + (unsigned)(t * round64(M.T)) + i : nullptr;
                res_poll<ARN_DIRECT>(ps, x, M.abort_word, &S.dead);
#pragma unroll
                for (int i = 0; i < ARN_DIRECT; ++i) s += x[i];
                S.h[t] = s;
            }
        } else if (M.T > 1) {
            for (int c = M.w + M.T * wave; c < p; c += M.T * RW) {
                const u64* ps[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    ps[i] = i * 64 + lane < M.T ? bank[b] + (unsigned)(c * round64(M.T)) + i * 64 + lane : nullptr;
                double x[4];
                res_poll<4>(ps, x, M.abort_word, &S.dead);
                const double s = wave_sum_dpp((x[0] + x[1]) + (x[2] + x[3]));
                if (lane == 0) res_store(vals[b] + c, s);
            }
            __syncthreads();  // S.h of the pass before has been read
            if (t < p) S.h[t] = res_poll(vals[b] + t, M.abort_word, &S.dead);
        }
        __syncthreads();
        if (out && M.w == 0 && t < p) out[t] = S.h[t];
        return S.dead != 0;
    };
    auto empty = [&](int b, int p) {
        if (M.T > 1 && t < p) {
            res_store_bits(bank[b] + (size_t)t * round64(M.T) + M.w, RES_EMPTY);
            if (t % M.T == M.w) res_store_bits(vals[b] + t, RES_EMPTY);
        }
    };
    // v_j0 (or the column to orthogonalise) at this thread's points and ring
    double v[RQ], vr = 0.0;
    int g[RQ];
    tl.points(g);
    const double* v0 = A.V + (long long)A.j0 * n;
#pragma unroll
    for (int q = 0; q < RQ; ++q) v[q] = tl.ok(q) ? v0[g[q]] : 0.0;
    if (wave >= 4 && !A.reorth) {
        const int side = wave - 4, nb = side == 0 ? M.nbr[0] : side == 1 ? M.nbr[1] : side == 2 ? M.nbr[2] : M.nbr[3];
        if (nb >= 0) {
            const int y0 = ty * RW * RQ, x0 = (M.w % ntx) * RTILE;
            const int gx = side == 0 || side == 1 ? x0 + lane : side == 2 ? x0 - 1 : x0 + RTILE;
            const int gy = side == 0 ? y0 - 1 : side == 1 ? y0 + RW * RQ : y0 + lane;
            if (gx < nx && gy < tl.ny && (side < 2 || lane < RW * RQ)) vr = v0[(long long)gy * nx + gx];
        }
    }
    bool rev = false;  // the passes walk the tile's rows up and down in turn
    for (int j = A.reorth ? A.j0 - 1 : A.j0; j < A.j1; ++j) {
        const bool re = A.reorth && j < A.j0;  // column j0 against the ones before it
        const int p = re ? A.j0 : j + 1;
        double w[RQ];
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // column j and the emptied slots
        if (re) {
#pragma unroll
            for (int q = 0; q < RQ; ++q) w[q] = v[q];
            __syncthreads();
        } else {
            tl.stencil64(S, v, vr, w);
        }
#pragma unroll
        for (int q = 0; q < RQ; ++q) S.w[wave * RQ + q][lane] = w[q];
        __syncthreads();
        double* h1 = re ? nullptr : A.H1 + (size_t)j * A.ldh;
        double* h2 = re ? nullptr : A.H2 + (size_t)j * A.ldh;
        gs_tile<0, RQ>(S, M, A.V, n, p, nx, gt, rows, xin, bank[0], rev);
        rev = !rev;
        if (totals(0, p, h1)) return;
        gs_tile<1, RQ>(S, M, A.V, n, p, nx, gt, rows, xin, bank[1], rev);
        rev = !rev;
        if (M.T == 1) __syncthreads();
        if (totals(1, p, h2)) return;
        empty(0, p);
        double a[1], s[1], ring = 0.0;
        a[0] = gs_tile<2, RQ>(S, M, A.V, n, p, nx, gt, rows, xin, nullptr, rev);
        rev = !rev;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < RQ; ++q) w[q] = S.w[wave * RQ + q][lane];
        if (exchange<1, true>(M, S, a, w, ring, s)) return;
        empty(1, p);
        const double nrm = sqrt(s[0]);
        if (M.w == 0 && t == 0 && !re) A.nrm[j] = nrm;
        double* vn = const_cast<double*>(A.V) + (long long)(re ? A.j0 : j + 1) * n;
#pragma unroll
        for (int q = 0; q < RQ; ++q) {
            v[q] = nrm > 0.0 ? w[q] / nrm : 0.0;
            if (tl.ok(q)) vn[g[q]] = v[q];
        }
        vr = nrm > 0.0 ? ring / nrm : 0.0;
    }
}

template <bool VAR>
static const void* arn_kernel(int rq) {
    switch (rq) {
        case 1: return (const void*)k_arnoldi2d<VAR, 1>;
        case 2: return (const void*)k_arnoldi2d<VAR, 2>;
        case 4: return (const void*)k_arnoldi2d<VAR, 4>;
        default: return (const void*)k_arnoldi2d<VAR, 8>;
    }
}

// The smallest tiles that fit the chip.  64-row tiles only where three quarters of
// their columns are in the grid: a tile's pass takes as long with one column as
// with 64, a pass over V as launches takes the points' time.  us a step as launches
// and in one launch, 40 | 100 columns: 1 x 16384 38 and 69 | 55 and 136, 16 x 16384
// 61 and 71 | 96 and 144, 48 x 16384 107 and 82 | 238 and 211, 130 x 4000 84 and
// 78 | 160 and 184, 200 x 4000 107 and 90 | 233 and 215; 32-row tiles gain at any
// width (1 x 4000 36 and 29 | 54 and 49, 65 x 4000 57 and 48 | 94 and 95).
int arnoldi2d_rows(const DevOp& op, int pmax, int max_team, int* team) {
    if (op.dim != 2 || pmax > ARN_PMAX) return 0;
    for (int rq = 1; rq <= 8; rq *= 2) {
        const int tx = (op.nx + RTILE - 1) / RTILE;
        const long long tiles = (long long)tx * ((op.ny + RW * rq - 1) / (RW * rq));
        if (rq == 8 && 4LL * op.nx < 3LL * RTILE * tx) return 0;
        if (tiles <= max_team) {
            *team = (int)tiles;
            return rq;
        }
    }
    return 0;
}

long long arnoldi2d_words(int team, int pmax) {
    const long long tp = (team + 63) / 64 * 64;
    return 3 * RES_NSUM * tp + 3 * RES_COPIES * RES_TOTALS + 3LL * team * RHALO + 2LL * pmax * (tp + 1);
}

__global__ __launch_bounds__(256) void k_arn_empty(u64* x, long long words, unsigned* ctl, unsigned gate0) {
    for (long long i = blockIdx.x * 256LL + threadIdx.x; i < words; i += gridDim.x * 256LL) x[i] = RES_EMPTY;
    if (blockIdx.x == 0 && threadIdx.x < 3) ctl[threadIdx.x] = threadIdx.x < 2 ? 0 : gate0;
}

hipError_t launch_arnoldi2d(const ArnArgs& args, int rq, hipStream_t s) {
    const long long words = arnoldi2d_words(args.team, args.pmax);
    const long long nb = (words + 1023) / 1024;
    hipLaunchKernelGGL(k_arn_empty, dim3((unsigned)(nb < 1024 ? nb : 1024)), dim3(256), 0, s, (u64*)args.xch, words,
                       args.ctl, args.gate0);
    ArnArgs a = args;
    void* av[] = {&a};
    return hipLaunchCooperativeKernel(args.op.var ? arn_kernel<true>(rq) : arn_kernel<false>(rq), dim3(args.team),
                                      dim3(RT), av, 0, s);
}

}  // namespace tgdk
