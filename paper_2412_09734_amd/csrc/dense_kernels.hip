// Dense constraint matrices (row-major, m x n): the r2HPDHG iteration of
// eq. (pdhg-lp) / eq. (hrpdhg) with the two products done as HBM-streaming
// passes over A~ (FP64 GEMV has 0.25 flop per byte, far below the FP64 ridge,
// so the vector units keep up with HBM and matrix cores would not help):
//   rows pass    : a_i = A~_i . v, one wave per four rows (a workgroup per four
//                  rows when there are few), fused with the dual step
//   columns pass : partial sums of A~' w over 256-column tiles (64-column ones
//                  where there are few) and row splits, then a finalize kernel that adds the splits in fixed order
//                  and applies the primal step.
// The epilogues repeat the formulas of the sparse kernels exactly.
#include "device.hpp"

namespace pdhg {

constexpr int kDenseSplits = 16;   // most row splits of the column pass's wide tiles
constexpr int kSplitRows = 256;    // fewest rows per split of the wide tiles
constexpr int kNarrowWgs = 1024;   // workgroups that the narrow tiles aim at, with 64 rows or more per split

enum RowMode : int32_t {
    ROW_DUAL = 0,      // y <- Halpern(prox)
    ROW_DUAL_CHK = 1,  // yhat <- prox
    ROW_CHECK_M = 2,   // check sums over rows
    ROW_STORE_SQ = 3,  // out = a, partial sum of a^2
    ROW_ABSMAX = 4,    // out = max |A_i.|
    ROW_ABSSUM = 5     // out = sum |A_i.|
};

enum ColMode : int32_t {
    COL_PRIMAL = 0,
    COL_PRIMAL_CHK = 1,
    COL_CHECK_N = 2,
    COL_STORE_SQ = 3,
    COL_ABSMAX = 4,
    COL_ABSSUM = 5
};

struct DenseVecs {
    const double *x, *x0, *xhat, *aty, *c, *lv, *uv, *Dc, *c_o, *lv_o, *uv_o;
    double *xw, *xext, *xhat_w, *aty_w;
    const double *y, *y0, *yhat, *lc, *uc, *Dr, *lc_o, *uc_o;
    double *yw, *yhat_w;
    double *out, *partials;
    // checks: the anchor's products, this check's products, ray partials
    const double *p0, *q0;
    double *phat, *qhat, *rays;
    const DevState *st;
    int32_t j;
    double gamma, tau_o, sigma_o;
};

constexpr int kGroupRows = 4;   // rows that a wave, or a workgroup, sums together

// Columns c, c + L, ..., U of them, of R rows: every load is issued
// before the first f(row, k, entry). TAIL: some of the columns are past n;
// their loads are clamped to the last one and come out as 0.
template <int U, bool NT, bool TAIL, int R, class F>
__device__ __forceinline__ void row_columns(const double *const (&Ar)[R], int32_t c, int32_t L, int32_t n, F f) {
    double a[R][U];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int k = 0; k < U; ++k) a[q][k] = load_entry<NT>(Ar[q] + (TAIL ? min(c + k * L, n - 1) : c + k * L));
    __builtin_amdgcn_sched_barrier(0);   // the scheduler would sink loads between the products
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int k = 0; k < U; ++k) f(q, k, TAIL && c + k * L >= n ? 0.0 : a[q][k]);
}

// acc over a lane's columns c, c + L, ... of the rows: products with v, or
// (MODE) maxima and sums of absolute values. U columns x R rows of independent
// loads in flight per lane, each row added in column order; the last columns go
// in one clamped group of 4, 8 or 16 (one at a time they cost a lane of a
// 3,001-column row 15 round trips).
template <int MODE, bool NT, int R>
__device__ __forceinline__ void row_sums(const double *const (&Ar)[R], const double *__restrict__ v, int32_t c,
                                         int32_t L, int32_t n, double (&acc)[R]) {
    constexpr int U = 16;
    constexpr bool NORM = MODE == ROW_ABSMAX || MODE == ROW_ABSSUM;
    double x[U];
    auto take = [&](int q, int k, double a) {
        if constexpr (MODE == ROW_ABSMAX) acc[q] = fmax(acc[q], fabs(a));
        else if constexpr (MODE == ROW_ABSSUM) acc[q] += fabs(a);
        else acc[q] = fma(a, x[k], acc[q]);
    };
    auto load_x = [&](int count, bool tail) {
        if constexpr (!NORM) {
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (k < count) {
                    x[k] = v[tail ? min(c + k * L, n - 1) : c + k * L];
                    if (tail) x[k] = c + k * L < n ? x[k] : 0.0;   // 0 x an infinity is no 0
                }
        }
    };
    for (; c + (U - 1) * L < n; c += U * L) {
        load_x(U, false);
        row_columns<U, NT, false>(Ar, c, L, n, take);
    }
    if (c + 7 * L < n) {
        load_x(U, true);
        row_columns<U, NT, true>(Ar, c, L, n, take);
    } else if (c + 3 * L < n) {
        load_x(8, true);
        row_columns<8, NT, true>(Ar, c, L, n, take);
    } else if (c < n) {
        load_x(4, true);
        row_columns<4, NT, true>(Ar, c, L, n, take);
    }
}

// Row pass: a = sum_c A[i][c] v[c], or |A| norms, for groups of R rows (four; one
// where the matrix has fewer, which a group of four would read again for the
// rows it misses: 1 x 3,000,000 1.72 ms per iteration, so 0.73), each
// v[c] loaded once for the group. W = 1: a wave per group (lanes strided over the
// columns, butterflies), four groups per workgroup; W = 4, 8: a workgroup of W
// waves per group (few rows: enough waves and loads in flight), wave totals
// added in wave order. stream: the matrix is larger than the caches.
template <int MODE, int W, int R>
__global__ __launch_bounds__(W == 1 ? kBlock : 64 * W) void k_dense_rows(
    const double *__restrict__ A, int32_t m, int32_t n, const double *__restrict__ v, DenseVecs d, int32_t stream) {
    if (d.st && d.st->done) return;
    constexpr bool WIDE = W > 1;
    constexpr int BS = WIDE ? 64 * W : kBlock;        // threads per workgroup
    constexpr int L = WIDE ? BS : 64;                 // lanes per row
    const int64_t row0 = WIDE ? (int64_t)blockIdx.x * R
                              : (((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6) * R;
    const int32_t lane = WIDE ? (int32_t)threadIdx.x : (int32_t)(threadIdx.x & 63);
    double acc[R];
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q] = 0.0;
    if (row0 < m) {
        const double *Ar[R];   // rows past the last one repeat it; their sums are dropped
#pragma unroll
        for (int q = 0; q < R; ++q) Ar[q] = A + (size_t)min(row0 + q, (int64_t)m - 1) * n;
        if (stream) row_sums<MODE, true>(Ar, v, lane, L, n, acc);
        else row_sums<MODE, false>(Ar, v, lane, L, n, acc);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q] = MODE == ROW_ABSMAX ? wave_max(acc[q]) : wave_sum(acc[q]);
    double accv = acc[0];
    int64_t row = row0;
    if constexpr (WIDE) {
        // thread q of the workgroup owns row row0 + q
        __shared__ double wt[R][BS / 64];
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int q = 0; q < R; ++q) wt[q][threadIdx.x >> 6] = acc[q];
        }
        __syncthreads();
        const int32_t q = (int32_t)threadIdx.x;
        if (q < R) {
            double t = wt[q][0];
            for (int w = 1; w < BS / 64; ++w) t = MODE == ROW_ABSMAX ? fmax(t, wt[q][w]) : t + wt[q][w];
            accv = t;
        }
        row = row0 + (q < R ? q : 0);
    } else {
        // lane q of the wave owns row row0 + q
#pragma unroll
        for (int q = 1; q < R; ++q)
            if (lane == q) accv = acc[q];
        row = row0 + (lane < R ? lane : 0);
    }
    const double acc_own = accv;
    const bool own = row < m && (WIDE ? (int32_t)threadIdx.x < R : lane < R);
    if (MODE == ROW_CHECK_M || MODE == ROW_STORE_SQ) {
        double vals[4] = {0.0, 0.0, 0.0, 0.0};
        double rsum[1] = {0.0}, rmax[2] = {0.0, 0.0};
        if (own) {
            const int64_t r = row;
            if (MODE == ROW_STORE_SQ) {
                d.out[r] = acc_own;
                vals[0] = acc_own * acc_own;
            } else {
                const double dr = d.Dr[r];
                const double ax = acc_own / dr;
                const double lo = d.lc_o[r], hi = d.uc_o[r];
                const double rpr = ax - clampd(ax, lo, hi);
                vals[0] = rpr * rpr;
                const double yh = d.yhat[r];
                const double yo = dr * yh;
                vals[1] = (isfinite(lo) ? lo * fmax(yo, 0.0) : 0.0) - (isfinite(hi) ? hi * fmax(-yo, 0.0) : 0.0);
                const double dy = yh - d.y[r];
                vals[2] = dy * dy;
                const double d0 = yh - d.y0[r];
                vals[3] = d0 * d0;
                d.phat[r] = acc_own;
                ray_row_terms(acc_own, d.p0[r], dr, d0, lo, hi, rsum, rmax);
            }
        }
        if (MODE == ROW_STORE_SQ) {
            double q[1] = {vals[0]};
            block_sum_store<1, BS>(q, d.partials + blockIdx.x);
        } else {
            block_sum_store<4, BS>(vals, d.partials + (size_t)blockIdx.x * 4);
            block_sum_store<1, BS>(rsum, d.rays + (size_t)blockIdx.x * 3);
            block_max_store<2, BS>(rmax, d.rays + (size_t)blockIdx.x * 3 + 1);
        }
        return;
    }
    if (!own) return;
    const int64_t r = row;
    if (MODE == ROW_ABSMAX || MODE == ROW_ABSSUM) {
        d.out[r] = acc_own;
    } else if (MODE == ROW_DUAL) {
        const double sigma = d.st->sigma;
        const int64_t k = d.st->k_base + (d.j - 1);
        const double yr = d.y[r];
        const double yh = dual_prox(yr, acc_own, sigma, d.lc[r], d.uc[r]);
        const double ak = (double)(k + 1) / (double)(k + 2), bk = 1.0 / (double)(k + 2);
        d.yw[r] = ak * ((1.0 + d.gamma) * yh - d.gamma * yr) + bk * d.y0[r];
    } else if (MODE == ROW_DUAL_CHK) {
        const double sigma = d.sigma_o > 0.0 ? d.sigma_o : d.st->sigma;
        d.yhat_w[r] = dual_prox(d.y[r], acc_own, sigma, d.lc[r], d.uc[r]);
    }
}

// acc over rows [i, r1) of one column (Ac = its first entry): products with w,
// or maxima / sums of absolute values. U rows' loads in flight, added in row
// order; the last rows go in one clamped group.
enum ColSum : int32_t { SUM_DOT = 0, SUM_ABSMAX = 1, SUM_ABS = 2 };
template <int KIND, bool NT>
__device__ __forceinline__ double col_rows(const double *__restrict__ Ac, const double *__restrict__ w, int32_t i,
                                           int32_t r1, int32_t n) {
    double acc = 0.0;
    auto rows = [&](auto width, bool tail) {
        constexpr int U = decltype(width)::value;
        double a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = load_entry<NT>(Ac + (size_t)(tail ? min(i + u, r1 - 1) : i + u) * n);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double e = tail && i + u >= r1 ? 0.0 : a[u];
            if constexpr (KIND == SUM_ABSMAX) acc = fmax(acc, fabs(e));
            else if constexpr (KIND == SUM_ABS) acc += fabs(e);
            else if (!tail || i + u < r1) acc = fma(e, w[i + u], acc);   // 0 x an infinity is no 0
        }
    };
    for (; i + 15 < r1; i += 16) rows(std::integral_constant<int, 16>(), false);
    if (i + 7 < r1) rows(std::integral_constant<int, 16>(), true);
    else if (i + 3 < r1) rows(std::integral_constant<int, 8>(), true);
    else if (i < r1) rows(std::integral_constant<int, 4>(), true);
    return acc;
}

// Partial column sums: partials[split][c] = sum over the split's rows of A[i][c] w[i];
// the splits are gridDim.y equal runs of rows. NARROW = false: 256-column tiles,
// a thread per column. NARROW = true: 64-column tiles whose four waves take a
// quarter of the split's rows each, added in wave order: four times the
// workgroups for the same partials, for matrices with few tiles.
template <int KIND, bool NARROW>
__global__ __launch_bounds__(kBlock) void k_dense_cols_partial(const double *__restrict__ A,
                                                               int32_t m, int32_t n,
                                                               const double *__restrict__ w,
                                                               double *__restrict__ partials,
                                                               const DevState *__restrict__ st,
                                                               int32_t stream) {
    if (st && st->done) return;
    const int32_t split = blockIdx.y, splits = (int32_t)gridDim.y;
    const int32_t per = (m + splits - 1) / splits;
    const int32_t wave = NARROW ? __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6)) : 0;
    const int64_t col = NARROW ? (int64_t)blockIdx.x * 64 + (threadIdx.x & 63) : (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int32_t end = min(m, (split + 1) * per);
    const int32_t part = NARROW ? (per + 3) / 4 : per;
    const int32_t r0 = split * per + wave * part, r1 = NARROW ? min(end, r0 + part) : end;
    double acc = 0.0;
    if (col < n) {
        if (stream) acc = col_rows<KIND, true>(A + col, w, r0, r1, n);
        else acc = col_rows<KIND, false>(A + col, w, r0, r1, n);
    }
    if constexpr (NARROW) {
        __shared__ double sh[4][64];
        sh[wave][threadIdx.x & 63] = acc;
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int q = 1; q < 4; ++q) {
            const double o = sh[q][threadIdx.x];
            acc = KIND == SUM_ABSMAX ? fmax(acc, o) : acc + o;
        }
    }
    if (col < n) partials[(size_t)split * n + col] = acc;
}

// Splits added in order 0..S-1, then the column epilogue.
template <int MODE>
__global__ __launch_bounds__(kBlock) void k_dense_cols_final(int32_t n, int32_t splits,
                                                             const double *__restrict__ part,
                                                             DenseVecs d) {
    if (d.st && d.st->done) return;
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    double s = 0.0;
    if (r < n) {
        // eight splits' loads in flight, added in order
        int32_t q = 0;
        for (; q + 8 <= splits; q += 8) {
            double p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = part[(size_t)(q + u) * n + r];
#pragma unroll
            for (int u = 0; u < 8; ++u) s = MODE == COL_ABSMAX ? fmax(s, p[u]) : s + p[u];
        }
        for (; q < splits; ++q) {
            const double p = part[(size_t)q * n + r];
            s = MODE == COL_ABSMAX ? fmax(s, p) : s + p;
        }
    }
    if (MODE == COL_CHECK_N || MODE == COL_STORE_SQ) {
        double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        double rsum[2] = {0.0, 0.0}, rmax[2] = {0.0, 0.0};
        if (r < n) {
            if (MODE == COL_STORE_SQ) {
                d.out[r] = s;
                v[0] = s * s;
            } else {
                const double q = s;
                const double xh = d.xhat[r];
                const double dx = xh - d.x[r];
                v[0] = dx * dx;
                v[1] = (q - d.aty[r]) * dx;
                const double d0 = xh - d.x0[r];
                v[2] = d0 * d0;
                const double dd = d.Dc[r];
                const double xo = dd * xh;
                const double g = d.c_o[r] - q / dd;
                const double lo = d.lv_o[r], hi = d.uv_o[r];
                const bool lf = isfinite(lo), uf = isfinite(hi);
                const double lam = (!lf && !uf) ? 0.0 : (lf && !uf) ? fmax(g, 0.0) : (!lf && uf) ? fmin(g, 0.0) : g;
                const double rd = g - lam;
                v[3] = rd * rd;
                v[4] = d.c_o[r] * xo;
                v[5] = (lf ? lo * fmax(lam, 0.0) : 0.0) - (uf ? hi * fmax(-lam, 0.0) : 0.0);
                d.qhat[r] = q;
                ray_col_terms(q, d.q0[r], dd, d0, d.c_o[r], lo, hi, rsum, rmax);
            }
        }
        if (MODE == COL_STORE_SQ) {
            double q1[1] = {v[0]};
            block_sum_store<1>(q1, d.partials + blockIdx.x);
        } else {
            block_sum_store<6>(v, d.partials + (size_t)blockIdx.x * 6);
            block_sum_store<2>(rsum, d.rays + (size_t)blockIdx.x * 4);
            block_max_store<2>(rmax, d.rays + (size_t)blockIdx.x * 4 + 2);
        }
        return;
    }
    if (r >= n) return;
    if (MODE == COL_ABSMAX || MODE == COL_ABSSUM) {
        d.out[r] = s;
    } else if (MODE == COL_PRIMAL) {
        const double tau = d.st->tau;
        const int64_t k = d.st->k_base + (d.j - 1);
        const double xr = d.x[r];
        const double xh = clampd(xr - tau * (d.c[r] - s), d.lv[r], d.uv[r]);
        const double ak = (double)(k + 1) / (double)(k + 2), bk = 1.0 / (double)(k + 2);
        d.xext[r] = 2.0 * xh - xr;
        d.xw[r] = ak * ((1.0 + d.gamma) * xh - d.gamma * xr) + bk * d.x0[r];
    } else if (MODE == COL_PRIMAL_CHK) {
        const double tau = d.tau_o > 0.0 ? d.tau_o : d.st->tau;
        const double xr = d.x[r];
        const double xh = clampd(xr - tau * (d.c[r] - s), d.lv[r], d.uv[r]);
        d.xhat_w[r] = xh;
        d.xext[r] = 2.0 * xh - xr;
        d.aty_w[r] = s;
    }
}

// A~_ij <- A~_ij / (r_i s_j) elementwise; also finite check of the input.
__global__ __launch_bounds__(kBlock) void k_dense_scale(double *__restrict__ A, int32_t m, int32_t n,
                                                        const double *__restrict__ rf,
                                                        const double *__restrict__ cf) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t total = (int64_t)m * n;
    for (int64_t e = t; e < total; e += (int64_t)gridDim.x * kBlock) {
        const int64_t i = e / n, j = e - i * n;
        A[e] = A[e] / (rf[i] * cf[j]);
    }
}

__global__ __launch_bounds__(kBlock) void k_dense_finite(const double *__restrict__ A, int64_t total,
                                                         int32_t *__restrict__ flag) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    for (int64_t e = t; e < total; e += (int64_t)gridDim.x * kBlock)
        if (!isfinite(A[e])) atomicOr(flag, 2);
}

__global__ __launch_bounds__(kBlock) void k_iota(int32_t *__restrict__ p, int32_t len) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < len) p[i] = (int32_t)i;
}

// ---------------------------------------------------------------------------
// host side

static unsigned dblk(int64_t len) { return (unsigned)std::max<int64_t>(1, ceil_div(len, kBlock)); }

static DenseVecs dvecs(Handle &h, int32_t j) {
    DenseVecs d;
    memset(&d, 0, sizeof(d));
    d.x = h.x.p;
    d.x0 = h.x0.p;
    d.xhat = h.xhat.p;
    d.aty = h.aty.p;
    d.c = h.c.p;
    d.lv = h.lv.p;
    d.uv = h.uv.p;
    d.Dc = h.Dc.p;
    d.c_o = h.c_o.p;
    d.lv_o = h.lv_o.p;
    d.uv_o = h.uv_o.p;
    d.xw = h.x.p;
    d.xext = h.xext.p;
    d.xhat_w = h.xhat.p;
    d.aty_w = h.aty.p;
    d.y = h.y.p;
    d.y0 = h.y0.p;
    d.yhat = h.yhat.p;
    d.lc = h.lc.p;
    d.uc = h.uc.p;
    d.Dr = h.Dr.p;
    d.lc_o = h.lc_o.p;
    d.uc_o = h.uc_o.p;
    d.yw = h.y.p;
    d.yhat_w = h.yhat.p;
    d.st = h.st.p;
    d.j = j;
    d.gamma = h.opt.gamma;
    d.tau_o = -1.0;
    d.sigma_o = -1.0;
    return d;
}

// Waves per group of four rows: one where the groups alone give the chip enough
// waves, four below 2,048 rows, eight for fewer and long rows. Measured, us per
// iteration with 1 / 4 / 8: 1,537 x 3,001 25.1 / 23.1 / 24.4, 8,000 x 5,000 113 /
// 116 / 131, 700 x 1,500 16.3 / 11.9 / 11.8, 300 x 700 12.1 / 10.7 / 11.2, 300 x 100,003
// 295 / 120 / 109.
static int32_t row_waves(int32_t m, int32_t n) {
    if (m >= 2048) return 1;
    return m < 1024 && n >= 16384 ? 8 : 4;
}
static int32_t group_rows(int32_t m) { return m < kGroupRows ? 1 : kGroupRows; }
static unsigned row_blocks(int32_t m, int32_t n) {
    return row_waves(m, n) > 1 ? (unsigned)std::max<int64_t>(1, ceil_div(m, group_rows(m)))
                            : dblk(ceil_div(m, kGroupRows) * 64);
}

// Whether the passes read the matrix with non-temporal loads. Up to 45 M entries
// (360 MB) enough of it stays in the L2s and the 256 MB memory-side cache
// between the passes to be read with ordinary ones. Measured, us per iteration
// ordinary / non-temporal: 500 x 20,000 36 / 47, 300 x 100,003 120 / 180, 8,000 x
// 5,000 116 / 119, 12,000 x 5,000 179 / 173, 8,000 x 16,000 354 / 326.
static int32_t dense_stream(int32_t m, int32_t n) { return (int64_t)m * n > 45000000 ? 1 : 0; }

template <int MODE>
static void launch_rows(hipStream_t s, const double *A, int32_t m, int32_t n, const double *v,
                        const DenseVecs &d) {
    const int32_t w = row_waves(m, n), stream = dense_stream(m, n);
    const unsigned nb = row_blocks(m, n);
    if (group_rows(m) == 1) {
        if (w == 8) k_dense_rows<MODE, 8, 1><<<nb, 512, 0, s>>>(A, m, n, v, d, stream);
        else k_dense_rows<MODE, 4, 1><<<nb, 256, 0, s>>>(A, m, n, v, d, stream);
        return;
    }
    if (w == 8) k_dense_rows<MODE, 8, kGroupRows><<<nb, 512, 0, s>>>(A, m, n, v, d, stream);
    else if (w == 4) k_dense_rows<MODE, 4, kGroupRows><<<nb, 256, 0, s>>>(A, m, n, v, d, stream);
    else k_dense_rows<MODE, 1, kGroupRows><<<nb, kBlock, 0, s>>>(A, m, n, v, d, stream);
}
static unsigned col_blocks(int32_t n) { return dblk(n); }

// Row splits of the column pass. Wide tiles: up to kDenseSplits, at least
// kSplitRows rows each. Where that leaves fewer than 128 workgroups, narrow
// tiles and enough splits for kNarrowWgs workgroups, with at least 64 rows each.
// Measured, us per iteration wide / narrow: 700 x 1,500 (12 wide workgroups) 22.2 /
// 11.9, 1,537 x 3,001 (72) 29.4 / 23.1, 500 x 20,000 (79) 41.1 / 36.0, 2,500 x 5,500
// (198) 42.2 / 46.0, 300 x 100,003 (391) 115 / 120.
struct ColPlan {
    bool narrow;
    int32_t splits;
};
static ColPlan col_plan(int32_t m, int32_t n) {
    const int32_t wide = (int32_t)std::min<int64_t>(kDenseSplits, std::max<int64_t>(1, m / kSplitRows));
    if ((int64_t)col_blocks(n) * wide >= 128) return {false, wide};
    const int64_t tiles = ceil_div(n, 64);
    const int64_t want = std::min<int64_t>(ceil_div(kNarrowWgs, tiles), ceil_div(m, 64));
    return {true, (int32_t)std::max<int64_t>(1, want)};
}
static int32_t col_splits(const Handle &h) { return col_plan(h.m, h.n).splits; }

template <int KIND>
static void launch_cols(hipStream_t s, const double *A, int32_t m, int32_t n, const double *w, double *part,
                        const DevState *st) {
    const ColPlan p = col_plan(m, n);
    const int32_t stream = dense_stream(m, n);
    if (p.narrow)
        k_dense_cols_partial<KIND, true><<<dim3((unsigned)ceil_div(n, 64), p.splits), kBlock, 0, s>>>(A, m, n, w, part, st, stream);
    else
        k_dense_cols_partial<KIND, false><<<dim3(col_blocks(n), p.splits), kBlock, 0, s>>>(A, m, n, w, part, st, stream);
}

int32_t dense_row_blocks(const Handle &h) { return (int32_t)row_blocks(h.m, h.n); }
int32_t dense_col_blocks(const Handle &h) { return (int32_t)col_blocks(h.n); }

static void cols_partial(Handle &h, const double *w, const DevState *st) {
    launch_cols<SUM_DOT>(h.stream, h.Ad.p, h.m, h.n, w, h.dpart.p, st);
}

void dense_primal(Handle &h, int32_t j) {
    cols_partial(h, h.y.p, h.st.p);
    k_dense_cols_final<COL_PRIMAL><<<col_blocks(h.n), kBlock, 0, h.stream>>>(h.n, col_splits(h), h.dpart.p, dvecs(h, j));
}

void dense_dual(Handle &h, int32_t j) {
    if (h.m == 0) return;
    launch_rows<ROW_DUAL>(h.stream, h.Ad.p, h.m, h.n, h.xext.p, dvecs(h, j));
}

void dense_primal_check(Handle &h, double tau_override) {
    cols_partial(h, h.y.p, h.st.p);
    DenseVecs d = dvecs(h, 0);
    d.tau_o = tau_override;
    k_dense_cols_final<COL_PRIMAL_CHK><<<col_blocks(h.n), kBlock, 0, h.stream>>>(h.n, col_splits(h), h.dpart.p, d);
}

void dense_dual_check(Handle &h, double sigma_override) {
    if (h.m == 0) return;
    DenseVecs d = dvecs(h, 0);
    d.sigma_o = sigma_override;
    launch_rows<ROW_DUAL_CHK>(h.stream, h.Ad.p, h.m, h.n, h.xext.p, d);
}

void dense_check_sums(Handle &h) {
    cols_partial(h, h.yhat.p, h.st.p);
    DenseVecs d = dvecs(h, 0);
    d.partials = h.pn.p;
    d.q0 = h.q0.p;
    d.qhat = h.qhat.p;
    d.rays = h.prn.p;
    k_dense_cols_final<COL_CHECK_N><<<col_blocks(h.n), kBlock, 0, h.stream>>>(h.n, col_splits(h), h.dpart.p, d);
    if (h.m > 0) {
        DenseVecs e = dvecs(h, 0);
        e.partials = h.pm.p;
        e.p0 = h.p0.p;
        e.phat = h.phat.p;
        e.rays = h.prm.p;
        launch_rows<ROW_CHECK_M>(h.stream, h.Ad.p, h.m, h.n, h.xhat.p, e);
    }
}

// out = A~ v with partial sums of out^2 (rows), for the power iteration
void dense_rows_sq(Handle &h, const double *v, double *out, double *partials) {
    DenseVecs d = dvecs(h, 0);
    d.st = nullptr;
    d.out = out;
    d.partials = partials;
    launch_rows<ROW_STORE_SQ>(h.stream, h.Ad.p, h.m, h.n, v, d);
}

// out = A~' w with partial sums of out^2 (columns)
void dense_cols_sq(Handle &h, const double *w, double *out, double *partials) {
    cols_partial(h, w, nullptr);
    DenseVecs d = dvecs(h, 0);
    d.st = nullptr;
    d.out = out;
    d.partials = partials;
    k_dense_cols_final<COL_STORE_SQ><<<col_blocks(h.n), kBlock, 0, h.stream>>>(h.n, col_splits(h), h.dpart.p, d);
}

void dense_build(Handle &h, const pdhg_problem &p) {
    hipStream_t s = h.stream;
    const int64_t total = (int64_t)h.m * h.n;
    h.Ad.alloc((size_t)std::max<int64_t>(1, total));
    if (total > 0)
        PDHG_HIP(hipMemcpyAsync(h.Ad.p, p.a_dense, sizeof(double) * (size_t)total,
                                p.mem == PDHG_MEM_DEVICE ? hipMemcpyDeviceToDevice
                                                         : hipMemcpyHostToDevice,
                                s));
    DBuf<int32_t> flag;
    flag.alloc(1);
    PDHG_HIP(hipMemsetAsync(flag.p, 0, sizeof(int32_t), s));
    if (total > 0) k_dense_finite<<<4096, kBlock, 0, s>>>(h.Ad.p, total, flag.p);
    check_flag(s, flag.p, "non-finite entry in the dense matrix");
    h.perm_r.alloc(h.m);
    h.perm_c.alloc(h.n);
    if (h.m) k_iota<<<dblk(h.m), kBlock, 0, s>>>(h.perm_r.p, h.m);
    k_iota<<<dblk(h.n), kBlock, 0, s>>>(h.perm_c.p, h.n);
    h.dpart.alloc((size_t)col_splits(h) * h.n);
    h.A.rows = h.m;
    h.A.cols = h.n;
    h.A.nnz = total;
    h.AT.rows = h.n;
    h.AT.cols = h.m;
    h.AT.nnz = total;
    PDHG_HIP(hipStreamSynchronize(s));
}

void dense_scale(Handle &h) {
    hipStream_t s = h.stream;
    const int32_t m = h.m, n = h.n;
    DBuf<double> rn, cn;
    rn.alloc(m);
    cn.alloc(n);
    const int passes = h.opt.ruiz_iters + (h.opt.pock_chambolle ? 1 : 0);
    for (int pass = 0; pass < passes && m > 0; ++pass) {
        const bool pc = pass >= h.opt.ruiz_iters;
        DenseVecs d = dvecs(h, 0);
        d.st = nullptr;
        d.out = rn.p;
        if (pc) {
            launch_rows<ROW_ABSSUM>(s, h.Ad.p, m, n, nullptr, d);
            launch_cols<SUM_ABS>(s, h.Ad.p, m, n, nullptr, h.dpart.p, nullptr);
            d.out = cn.p;
            k_dense_cols_final<COL_ABSSUM><<<col_blocks(n), kBlock, 0, s>>>(n, col_splits(h), h.dpart.p, d);
        } else {
            launch_rows<ROW_ABSMAX>(s, h.Ad.p, m, n, nullptr, d);
            launch_cols<SUM_ABSMAX>(s, h.Ad.p, m, n, nullptr, h.dpart.p, nullptr);
            d.out = cn.p;
            k_dense_cols_final<COL_ABSMAX><<<col_blocks(n), kBlock, 0, s>>>(n, col_splits(h), h.dpart.p, d);
        }
        launch_factors(h, rn.p, cn.p);
        k_dense_scale<<<8192, kBlock, 0, s>>>(h.Ad.p, m, n, rn.p, cn.p);
    }
    PDHG_HIP(hipStreamSynchronize(s));
}

}  // namespace pdhg
