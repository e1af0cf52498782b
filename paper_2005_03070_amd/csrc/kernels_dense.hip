// Tall-skinny kernels: Gram products A^T B, V Y products, and the classical
// Gram-Schmidt steps of the Arnoldi process.  All reductions over the long
// dimension are deterministic: per-block partials, then one workgroup per
// value sums them in a fixed order (k_sum_partials).
#include "device_common.h"
#include "launch.h"

namespace tgdk {

constexpr int GS_ROWS_PER_BLOCK = NT;  // rows per block before the cap (grid-strided beyond)
constexpr int GS_MAX_BLOCKS = 1024;  // measured best on 1M rows x 25 columns (4 rows per thread)

int gs_blocks(long long n) {
    long long b = (n + GS_ROWS_PER_BLOCK - 1) / GS_ROWS_PER_BLOCK;
    if (b > GS_MAX_BLOCKS) b = GS_MAX_BLOCKS;
    if (b < 1) b = 1;
    return (int)b;
}

// Sums value i of per-block partials (partial[b * pstride + i], b < nblocks)
// in a fixed order: one workgroup per value, threads take blocks t, t + NT,
// ..., then the block combine.  out[i] = sum (or sqrt(sum) if root).
__global__ __launch_bounds__(NT) void k_sum_partials(const double* __restrict__ partial, int nblocks,
                                                     long long pstride, double* __restrict__ out, int root) {
    __shared__ double sh[NWAVE];
    const int i = blockIdx.x;
    double a = 0.0;
#pragma unroll 8
    for (int b = threadIdx.x; b < nblocks; b += NT) a += partial[(long long)b * pstride + i];
    const double s = block_sum_one(a, sh);
    if (threadIdx.x == 0) out[i] = root ? sqrt(s) : s;
}

// ------------------------------------------------------------- Gram A^T B
// Matrix-core (v_mfma_f64_16x16x4f64) Gram product G = A^T B, K = the long
// dimension n.  Operand layout of the instruction on gfx950 (one wave):
//   A-operand  lane l holds A[l % 16][l / 16]   (16 x 4)
//   B-operand  lane l holds B[l / 16][l % 16]   (4 x 16)
//   result     lane l, register r holds D[l / 16 + 4 r][l % 16]  (16 x 16)
// The rows go in chunks of 32 to nb accumulators (chunk c to accumulator c mod
// nb, four rows at a time), whose partial products k_sum_gram_block sums in a
// fixed order.  An accumulator is a wave: a lane loads its column's rows
// l / 16, 4 + l / 16, ... of the chunk to registers (one line of a column
// serves four loads) while the chunk before is multiplied; A = B loads once
// and forms the upper tiles, which are the lower ones' mirror image.  Lanes
// past the last column repeat it: what they hold enters only rows and columns
// of G that are not stored.
//
// Bound by the loads: 1023^2 x 30, V^T V reads 251 MB in 67 us (chunks
// staged through LDS by four waves that share the tiles, two barriers a chunk
// and B read again where it is A: 160 us), V^T (A V) 502 MB in 124 (180).
// At 31^2 x 8 (eight waves) 134 against 145 us for a whole space.
typedef double d4_t __attribute__((ext_vector_type(4)));

constexpr int GRAM_MAX = 64;   // p, q <= 64
constexpr int GRAM_ROWS = 32;  // rows of a chunk

int gram_blocks(long long n) {
    long long b = (n + 4 * GRAM_ROWS - 1) / (4 * GRAM_ROWS);
    if (b > 1024) b = 1024;
    if (b < 1) b = 1;
    return (int)b;
}

template <int T, bool SAME>
__global__ __launch_bounds__(NT) void k_gram(const double* __restrict__ A, long long lda, int p,
                                                  const double* __restrict__ B, long long ldb, int q, long long n,
                                                  int nacc, double* __restrict__ partial) {
    constexpr int KS = GRAM_ROWS / 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, acci = blockIdx.x * NWAVE + w;
    if (acci >= nacc) return;
    d4_t acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = d4_t{0.0, 0.0, 0.0, 0.0};
    const double* pa[T];
    const double* pb[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int c = i * 16 + (lane & 15);
        pa[i] = A + (long long)(c < p ? c : p - 1) * lda + (lane >> 4);
        pb[i] = B + (long long)(c < q ? c : q - 1) * ldb + (lane >> 4);
    }
    auto load = [&](long long r0, double(&a)[T][KS], double(&b)[T][KS]) {
        if (r0 + GRAM_ROWS <= n) {
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    a[i][s] = pa[i][r0 + 4 * s];
                    if (!SAME) b[i][s] = pb[i][r0 + 4 * s];
                }
        } else {
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const bool in = r0 + 4 * s + (lane >> 4) < n;
                    a[i][s] = in ? pa[i][r0 + 4 * s] : 0.0;
                    if (!SAME) b[i][s] = in ? pb[i][r0 + 4 * s] : 0.0;
                }
        }
    };
    double a[T][KS], na[T][KS];
    double b[T][KS], nb[T][KS];
    const long long step = (long long)nacc * GRAM_ROWS;
    long long r0 = (long long)acci * GRAM_ROWS;
    if (r0 < n) load(r0, a, b);
    for (; r0 < n; r0 += step) {
        if (r0 + step < n) load(r0 + step, na, nb);
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = SAME ? i : 0; j < T; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                        a[i][s], SAME ? a[j][s] : b[j][s], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                a[i][s] = na[i][s];
                if (!SAME) b[i][s] = nb[i][s];
            }
    }
    double* out = partial + (long long)acci * p * q;  // row-major p x q
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = SAME ? i : 0; j < T; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = i * 16 + (lane >> 4) + 4 * r, col = j * 16 + (lane & 15);
                if (row < p && col < q) {
                    out[row * q + col] = acc[i][j][r];
                    if (SAME && j > i) out[col * q + row] = acc[i][j][r];
                }
            }
}

// Entry e = i * qb + j of the summed partials goes to out[i * ldo + j] (a
// GRAM_MAX x GRAM_MAX block of a larger row-major Gram matrix).  A workgroup
// sums four neighbouring entries, its threads partials t, t + NT, ...: one
// entry a workgroup used 8 bytes of every line it read (900 entries of 1024
// partials 11 us, four at a time 8.4).
__global__ __launch_bounds__(NT) void k_sum_gram_block(const double* __restrict__ partial, int nblocks,
                                                       int npair, int qb, double* __restrict__ out, int ldo) {
    __shared__ double sh[4][NWAVE];
    const int e0 = blockIdx.x * 4;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int b = threadIdx.x; b < nblocks; b += NT)
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] += partial[(long long)b * npair + (e0 + i < npair ? e0 + i : npair - 1)];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double v = block_sum_one(a[i], sh[i]);
        const int e = e0 + i;
        if (threadIdx.x == 0 && e < npair) out[(long long)(e / qb) * ldo + e % qb] = v;
    }
}

template <bool SAME>
static void gram_block(const double* A, long long lda, int p, const double* B, long long ldb, int q, long long n,
                      double* partial, int nb, hipStream_t s) {
    const dim3 grid((nb + NWAVE - 1) / NWAVE);
    const int t = ((p > q ? p : q) + 15) / 16;
    if (t == 1)
        hipLaunchKernelGGL((k_gram<1, SAME>), grid, dim3(NT), 0, s, A, lda, p, B, ldb, q, n, nb, partial);
    else if (t == 2)
        hipLaunchKernelGGL((k_gram<2, SAME>), grid, dim3(NT), 0, s, A, lda, p, B, ldb, q, n, nb, partial);
    else if (t == 3)
        hipLaunchKernelGGL((k_gram<3, SAME>), grid, dim3(NT), 0, s, A, lda, p, B, ldb, q, n, nb, partial);
    else
        hipLaunchKernelGGL((k_gram<4, SAME>), grid, dim3(NT), 0, s, A, lda, p, B, ldb, q, n, nb, partial);
}

// G (p x q, row-major) = A^T B in blocks of at most GRAM_MAX x GRAM_MAX (the
// kernel's tile limit), each block's accumulators (a wave's each) summed into its
// place in G; the blocks run one after another on the stream and share the
// partial workspace (gram_blocks(n) * GRAM_MAX^2 doubles suffice).
void launch_gram(const double* A, long long lda, int p, const double* B, long long ldb, int q, long long n, double* G,
                 double* partial, hipStream_t s) {
    const int nb = gram_blocks(n);
    for (int i0 = 0; i0 < p; i0 += GRAM_MAX)
        for (int j0 = 0; j0 < q; j0 += GRAM_MAX) {
            const int pb = p - i0 < GRAM_MAX ? p - i0 : GRAM_MAX, qb = q - j0 < GRAM_MAX ? q - j0 : GRAM_MAX;
            const double *Ab = A + (size_t)i0 * lda, *Bb = B + (size_t)j0 * ldb;
            if (Ab == Bb && lda == ldb && pb == qb)
                gram_block<true>(Ab, lda, pb, Bb, ldb, qb, n, partial, nb, s);
            else
                gram_block<false>(Ab, lda, pb, Bb, ldb, qb, n, partial, nb, s);
            hipLaunchKernelGGL(k_sum_gram_block, dim3((pb * qb + 3) / 4), dim3(NT), 0, s, partial, nb, pb * qb, qb,
                               G + (size_t)i0 * q + j0, q);
        }
}

size_t gram_partial_bytes(long long n, int p, int q) {
    const int pb = p < GRAM_MAX ? p : GRAM_MAX, qb = q < GRAM_MAX ? q : GRAM_MAX;
    return (size_t)gram_blocks(n) * pb * qb * sizeof(double);
}

// ---------------------------------------------------------------- V * Y
// Out (n x q) = V (n x p) Y (p x q) on the matrix cores, computed as
// Out^T = Y^T V^T so that each lane's V load is one of 16 consecutive rows of
// a column (coalesced): B-operand lane l = V[r0 + l % 16][k0 + l / 16],
// A-operand lane l = Y[k0 + l / 16][j0 + l % 16], result lane l, register r =
// Out[r0 + l % 16][j0 + l / 16 + 4 r].
//
// A wave owns R groups of 16 rows and all q <= 16 QT columns, so V is read
// once; the loads of 32 columns are all in flight before the first product
// (16 KB a wave for R = 4), and Y's operands come from LDS, laid out once a
// workgroup where p <= 32, else 32 rows at a time.  Bound by the traffic:
// 1023^2, 30 -> 30 columns, 502 MB in 111 us; with 16 rows a wave, Y from
// global memory and one load in flight it took 300 us.
constexpr int VMUL_MAXQT = 9;

template <int QT, int R>
__global__ __launch_bounds__(NT) void k_vmul(const double* __restrict__ V, long long ldv, int p,
                                             const double* __restrict__ Y, int q, double* __restrict__ Out,
                                             long long ldo, long long n) {
    __shared__ double Ys[8][QT][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    auto stage = [&](int k0) {
        for (int i = threadIdx.x; i < 8 * QT * 64; i += NT) {
            const int l = i & 63, t = (i >> 6) % QT, s = (i >> 6) / QT;
            const int kc = k0 + 4 * s + (l >> 4), jc = t * 16 + (l & 15);
            Ys[s][t][l] = kc < p && jc < q ? Y[(long long)jc * p + kc] : 0.0;
        }
    };
    if (p <= 32) {
        stage(0);
        __syncthreads();
    }
    const long long ngroup = (n + 16 * R * NWAVE - 1) / (16 * R * NWAVE);
    for (long long gr = blockIdx.x; gr < ngroup; gr += gridDim.x) {
        const long long r0 = (gr * NWAVE + w) * 16 * R + (lane & 15);
        d4_t acc[R][QT];
        long long row[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            row[i] = r0 + 16 * i < n ? r0 + 16 * i : n - 1;  // past n: the last row again, not stored
#pragma unroll
            for (int t = 0; t < QT; ++t) acc[i][t] = d4_t{0.0, 0.0, 0.0, 0.0};
        }
        for (int k0 = 0; k0 < p; k0 += 32) {
            double bv[R][8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int kc = k0 + 4 * s + (lane >> 4);
                const double* col = V + (long long)(kc < p ? kc : p - 1) * ldv;  // past p: times a zero of Y
#pragma unroll
                for (int i = 0; i < R; ++i) bv[i][s] = kc < p ? col[row[i]] : 0.0;
            }
            if (p > 32) {
                __syncthreads();
                stage(k0);
                __syncthreads();
            }
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if (k0 + 4 * s >= p) break;
#pragma unroll
                for (int t = 0; t < QT; ++t) {
                    const double av = Ys[s][t][lane];
#pragma unroll
                    for (int i = 0; i < R; ++i)
                        acc[i][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[i][s], acc[i][t], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < QT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int jc = t * 16 + (lane >> 4) + 4 * r;
                if (jc < q) {
#pragma unroll
                    for (int i = 0; i < R; ++i)
                        if (r0 + 16 * i < n) Out[jc * ldo + row[i]] = acc[i][t][r];
                }
            }
    }
}

template <int QT, int R>
static void vmul_block(const double* V, long long ldv, int p, const double* Y, int q, double* Out, long long ldo,
                       long long n, hipStream_t s) {
    long long nb = (n + 16 * R * NWAVE - 1) / (16 * R * NWAVE);
    if (nb > 2048) nb = 2048;
    hipLaunchKernelGGL((k_vmul<QT, R>), dim3((int)nb), dim3(NT), 0, s, V, ldv, p, Y, q, Out, ldo, n);
}

// Out = V Y (not in place) in column blocks of at most 16 * VMUL_MAXQT (the
// kernel's limit): block j0 takes Y's columns j0.. (column-major, leading
// dimension p) and writes Out's.  Fewer columns leave registers for more rows
// in flight; a short V takes 16 rows a wave, so that the chip is not idle.
void launch_vmul(const double* V, long long ldv, int p, const double* Y, int q, double* Out, long long ldo,
                 long long n, hipStream_t s) {
    constexpr int QB = 16 * VMUL_MAXQT;
    for (int j0 = 0; j0 < q; j0 += QB) {
        const int qb = q - j0 < QB ? q - j0 : QB;
        const double* Yb = Y + (size_t)j0 * p;
        double* Ob = Out + (size_t)j0 * ldo;
        const bool tall = n >= 64 * 1024;  // 1024 waves of 64 rows: one a SIMD
        if (qb <= 32 && tall)
            vmul_block<2, 4>(V, ldv, p, Yb, qb, Ob, ldo, n, s);
        else if (qb <= 32)
            vmul_block<2, 1>(V, ldv, p, Yb, qb, Ob, ldo, n, s);
        else if (qb <= 64 && tall)
            vmul_block<4, 2>(V, ldv, p, Yb, qb, Ob, ldo, n, s);
        else if (qb <= 64)
            vmul_block<4, 1>(V, ldv, p, Yb, qb, Ob, ldo, n, s);
        else
            vmul_block<VMUL_MAXQT, 1>(V, ldv, p, Yb, qb, Ob, ldo, n, s);
    }
}

__global__ __launch_bounds__(NT) void k_vmul_add(const double* __restrict__ V, long long ldv, int p,
                                                 const double* __restrict__ y, double* __restrict__ x, long long n) {
    __shared__ double ys[MAXK + 1];
    for (int i = threadIdx.x; i < p; i += NT) ys[i] = y[i];
    __syncthreads();
    for (long long g = blockIdx.x * (long long)NT + threadIdx.x; g < n; g += (long long)gridDim.x * NT) {
        double a = 0.0;
        for (int i = 0; i < p; ++i) a += V[i * ldv + g] * ys[i];
        x[g] += a;
    }
}

void launch_vmul_add(const double* V, long long ldv, int p, const double* y, double* x, long long n,
                     hipStream_t s) {
    long long nb = (n + NT - 1) / NT;
    if (nb > 4096) nb = 4096;
    hipLaunchKernelGGL(k_vmul_add, dim3((int)nb), dim3(NT), 0, s, V, ldv, p, y, x, n);
}

// ------------------------------------------------- Gram-Schmidt (Arnoldi)
// gs_blocks blocks of NT threads, rows grid-strided (4 rows per thread at 1M rows).
// MODE 0: hout = V^T w.  MODE 1: w -= V h, then hout = V^T w, fused per row:
// the row's V values are read for the update and again, from cache, for the
// dot products.  MODE 2: w -= V h, then hout[0] = ||w||.
template <int MODE>
__global__ __launch_bounds__(NT) void k_gs(const double* __restrict__ V, long long ldv, int p, double* w,
                                           const double* __restrict__ h, long long n, double* hout,
                                           double* partial, unsigned* counter) {
    __shared__ double sh[NWAVE * 16];
    __shared__ double hs[MAXK + 1];
    const long long stride = (long long)gridDim.x * NT;
    const long long g0 = blockIdx.x * (long long)NT + threadIdx.x;
    if (MODE >= 1)
        for (int i = threadIdx.x; i < p; i += NT) hs[i] = h[i];
    __syncthreads();
    const int pstride = MAXK + 1;
    if (MODE <= 1) {
        for (int c0 = 0; c0 < p; c0 += 16) {
            const int nc = p - c0 < 16 ? p - c0 : 16;
            double acc[16];
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) acc[jj] = 0.0;
            for (long long g = g0; g < n; g += stride) {
                double wv = w[g];
                if (MODE == 1 && c0 == 0) {
                    // update of this row before its first dot products
#pragma unroll 8
                    for (int i = 0; i < p; ++i) wv -= V[i * ldv + g] * hs[i];
                    w[g] = wv;
                }
                // unconditional loads (columns past p re-read column c0, a
                // cache hit, and are masked), so all 16 are in flight at once
#pragma unroll
                for (int jj = 0; jj < 16; ++jj) {
                    const double v = V[(long long)(jj < nc ? c0 + jj : c0) * ldv + g];
                    acc[jj] += jj < nc ? v * wv : 0.0;
                }
            }
            double tot;
            block_sum<16>(acc, sh, tot);
            if (threadIdx.x < 16 && c0 + threadIdx.x < p)
                partial[(long long)blockIdx.x * pstride + c0 + threadIdx.x] = tot;
        }
    } else {
        double acc[1] = {0.0};
        for (long long g = g0; g < n; g += stride) {
            double a = w[g];
#pragma unroll 8
            for (int i = 0; i < p; ++i) a -= V[i * ldv + g] * hs[i];
            if (p > 0) w[g] = a;
            acc[0] += a * a;
        }
        double tot;
        block_sum<1>(acc, sh, tot);
        if (threadIdx.x == 0) partial[(long long)blockIdx.x * pstride] = tot;
    }
    (void)counter;
    (void)hout;
}

// The same passes with the columns split over the waves, for p <= NW CPW
// (NW waves of 64 threads per workgroup): wave w holds columns w, w + NW, ...,
// w + NW (CPW - 1) of a 64-row block (64 consecutive rows per column load),
// so every pass reads V once and the row loop has no per-chunk reductions.
// The update w -= V h of a row needs all columns: the waves exchange their
// partial sums of V h through LDS (double-buffered, one barrier per row
// block; summed over the waves in order) and every wave forms the same
// updated rows (wave 0 stores them), whose dot products then use the V values
// already in registers.  The next row block's loads are issued before the
// barrier, which does not wait for them.  Columns past p are read at column 0
// (a cache hit) and masked.
template <int MODE, int CPW, int NW>
__global__ __launch_bounds__(64 * NW) void k_gsc(const double* __restrict__ V, long long ldv, int p, double* w,
                                                 const double* __restrict__ h, long long n,
                                                 double* __restrict__ partial) {
    __shared__ double xs[2][NW][64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double* vc[CPW];
    double hc[CPW];
    bool cok[CPW];
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = wv + NW * i;
        cok[i] = c < p;
        vc[i] = V + (long long)(cok[i] ? c : 0) * ldv;
        hc[i] = (MODE >= 1 && cok[i]) ? h[c] : 0.0;
    }
    double acc[CPW];
#pragma unroll
    for (int i = 0; i < CPW; ++i) acc[i] = 0.0;
    double nacc = 0.0;
    const long long nrb = (n + 63) / 64, step = gridDim.x;
    auto load = [&](long long rb, double(&dv)[CPW], double& dw) {
        long long row = rb * 64 + lane;
        if (row >= n) row = n - 1;
#pragma unroll
        for (int i = 0; i < CPW; ++i) dv[i] = vc[i][row];
        dw = w[row];
    };
    double vv[CPW], wr = 0.0;
#pragma unroll
    for (int i = 0; i < CPW; ++i) vv[i] = 0.0;
    long long rb = blockIdx.x;
    if (rb < nrb) load(rb, vv, wr);
    int par = 0;
    for (; rb < nrb; rb += step) {
        double nv[CPW], nw = 0.0;
#pragma unroll
        for (int i = 0; i < CPW; ++i) nv[i] = 0.0;
        if (rb + step < nrb) load(rb + step, nv, nw);
        const long long row = rb * 64 + lane;
        const bool ok = row < n;
        double x = wr;
        if (MODE >= 1) {
            double u = 0.0;
#pragma unroll
            for (int i = 0; i < CPW; ++i) u += cok[i] ? vv[i] * hc[i] : 0.0;
            xs[par][wv][lane] = u;
            __syncthreads();
            double t = xs[par][0][lane];
#pragma unroll
            for (int q = 1; q < NW; ++q) t += xs[par][q][lane];
            x = wr - t;
            if (wv == 0 && ok) w[row] = x;
            par ^= 1;
        }
        if (MODE <= 1) {
#pragma unroll
            for (int i = 0; i < CPW; ++i) acc[i] += (ok && cok[i]) ? vv[i] * x : 0.0;
        } else if (wv == 0) {
            nacc += ok ? x * x : 0.0;
        }
#pragma unroll
        for (int i = 0; i < CPW; ++i) vv[i] = nv[i];
        wr = nw;
    }
    const long long pstride = MAXK + 1;
    if (MODE <= 1) {
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            const double t = wave_sum(acc[i]);
            if (lane == 0 && cok[i]) partial[(long long)blockIdx.x * pstride + wv + NW * i] = t;
        }
    } else if (wv == 0) {
        const double t = wave_sum(nacc);
        if (lane == 0) partial[(long long)blockIdx.x * pstride] = t;
    }
}

// k_gsc for 1 <= p <= 128: 4 waves with 1 ... 16 columns each up to 64
// columns; beyond, 8 waves with 16 each in half as many workgroups (the same
// threads).  Returns the number of workgroups (of partials) launched, or 0 if
// p is out of range.
template <int MODE>
static int launch_gsc(const double* V, long long ldv, int p, double* w, const double* h, long long n,
                      double* partial, int nb, hipStream_t s) {
    if (p < 1 || p > 8 * 16) return 0;
    const dim3 g(nb), b4(256);
    if (p <= 4)
        hipLaunchKernelGGL((k_gsc<MODE, 1, 4>), g, b4, 0, s, V, ldv, p, w, h, n, partial);
    else if (p <= 8)
        hipLaunchKernelGGL((k_gsc<MODE, 2, 4>), g, b4, 0, s, V, ldv, p, w, h, n, partial);
    else if (p <= 16)
        hipLaunchKernelGGL((k_gsc<MODE, 4, 4>), g, b4, 0, s, V, ldv, p, w, h, n, partial);
    else if (p <= 32)
        hipLaunchKernelGGL((k_gsc<MODE, 8, 4>), g, b4, 0, s, V, ldv, p, w, h, n, partial);
    else if (p <= 64)
        hipLaunchKernelGGL((k_gsc<MODE, 16, 4>), g, b4, 0, s, V, ldv, p, w, h, n, partial);
    else {
        nb = nb > 1 ? nb / 2 : 1;
        hipLaunchKernelGGL((k_gsc<MODE, 16, 8>), dim3(nb), dim3(512), 0, s, V, ldv, p, w, h, n, partial);
    }
    return nb;
}

void launch_gs_dot(const double* V, long long ldv, int p, const double* w, long long n, double* hout,
                   double* partial, unsigned* counter, hipStream_t s) {
    int nb = gs_blocks(n);
    if (const int used = launch_gsc<0>(V, ldv, p, const_cast<double*>(w), nullptr, n, partial, nb, s))
        nb = used;
    else
        hipLaunchKernelGGL((k_gs<0>), dim3(nb), dim3(NT), 0, s, V, ldv, p, const_cast<double*>(w),
                           (const double*)nullptr, n, hout, partial, counter);
    if (p > 0) hipLaunchKernelGGL(k_sum_partials, dim3(p), dim3(NT), 0, s, partial, nb, (long long)(MAXK + 1), hout, 0);
}
void launch_gs_update_dot(const double* V, long long ldv, int p, double* w, const double* h, long long n,
                          double* hout, double* partial, unsigned* counter, hipStream_t s) {
    int nb = gs_blocks(n);
    if (const int used = launch_gsc<1>(V, ldv, p, w, h, n, partial, nb, s))
        nb = used;
    else
        hipLaunchKernelGGL((k_gs<1>), dim3(nb), dim3(NT), 0, s, V, ldv, p, w, h, n, hout, partial, counter);
    if (p > 0) hipLaunchKernelGGL(k_sum_partials, dim3(p), dim3(NT), 0, s, partial, nb, (long long)(MAXK + 1), hout, 0);
}
void launch_gs_update_norm(const double* V, long long ldv, int p, double* w, const double* h, long long n,
                           double* nrm, double* partial, unsigned* counter, hipStream_t s) {
    int nb = gs_blocks(n);
    if (const int used = launch_gsc<2>(V, ldv, p, w, h, n, partial, nb, s))
        nb = used;
    else
        hipLaunchKernelGGL((k_gs<2>), dim3(nb), dim3(NT), 0, s, V, ldv, p, w, h, n, nrm, partial, counter);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(NT), 0, s, partial, nb, (long long)(MAXK + 1), nrm, 1);
}
void launch_norm2(const double* w, long long n, double* out, double* partial, unsigned* counter, hipStream_t s) {
    const int nb = gs_blocks(n);
    hipLaunchKernelGGL((k_gs<2>), dim3(nb), dim3(NT), 0, s, (const double*)nullptr, 0LL, 0,
                       const_cast<double*>(w), (const double*)nullptr, n, out, partial, counter);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(NT), 0, s, partial, nb, (long long)(MAXK + 1), out, 1);
}

__global__ void k_scale(const double* w, double* v, const double* __restrict__ nrm,
                        long long n) {
    const double s = *nrm;
    for (long long g = blockIdx.x * (long long)blockDim.x + threadIdx.x; g < n;
         g += (long long)gridDim.x * blockDim.x)
        v[g] = s > 0.0 ? w[g] / s : 0.0;
}
void launch_scale(const double* w, double* v, const double* nrm, long long n, hipStream_t s) {
    long long nb = (n + 255) / 256;
    if (nb > 8192) nb = 8192;
    hipLaunchKernelGGL(k_scale, dim3((int)nb), dim3(256), 0, s, w, v, nrm, n);
}

// c = a - b over n contiguous values (c may be b: each element is read
// before it is written by the same thread)
__global__ __launch_bounds__(NT) void k_sub(const double* __restrict__ a, const double* b, double* c, long long n) {
    for (long long i = blockIdx.x * (long long)NT + threadIdx.x; i < n; i += (long long)gridDim.x * NT)
        c[i] = a[i] - b[i];
}

void launch_sub(const double* a, const double* b, double* c, long long n, hipStream_t s) {
    long long nb = (n + NT - 1) / NT;
    if (nb > 4096) nb = 4096;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_sub, dim3((int)nb), dim3(NT), 0, s, a, b, c, n);
}

// a += b over n values
__global__ __launch_bounds__(NT) void k_add(double* __restrict__ a, const double* __restrict__ b, long long n) {
    for (long long i = blockIdx.x * (long long)NT + threadIdx.x; i < n; i += (long long)gridDim.x * NT) a[i] += b[i];
}

void launch_add(double* a, const double* b, long long n, hipStream_t st) {
    long long nb = (n + NT - 1) / NT;
    if (nb > 4096) nb = 4096;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_add, dim3((int)nb), dim3(NT), 0, st, a, b, n);
}

}  // namespace tgdk
