// r2HPDHG on one small sparse LP by one workgroup: whole check periods (the
// check iteration, its decisions and the plain iterations after it) run in one
// launch, with the iterate, anchors, cost and bounds in LDS.
//
// What bounds it: a small LP's iteration is a chain of latencies, not bytes. As
// two launches it is about 7 us, of which the kernels' own work is under 2; here
// it is two barriers around two products. The rows of A~' and A~ are the wave
// tasks of the hybrid layout (64 >> lg rows of a segment, or a SELL-64 slice),
// dealt to the 16 waves round robin, at most K per wave and product. The first four
// entries of every lane stay in registers through a period (with at most four
// per lane in rows up to 256 long, that is all of them), so an iteration reads
// no matrix data from memory. With more tasks it is bound by instruction issue:
// some 150 vector instructions per task and product pair.
// Measured: see small_lp_fits.
#include <algorithm>

#include "lp_check.hpp"

namespace pdhg {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallDoubles = 20000;   // LDS doubles for the vectors (6 n + 5 m)
constexpr int kSmallMost = 3;          // wave tasks per wave and product

struct SmallArgs {
    MatView A, AT;
    int32_t m, n;
    double *x, *x0, *y, *y0, *xhat, *yhat, *aty;
    const double *c, *lv, *uv, *lc, *uc;
    const double *Dr, *Dc, *c_o, *lv_o, *uv_o, *lc_o, *uc_o;
    double *p0, *q0, *phat, *qhat;
    DevState *st;
    CtlConst K;
    double gamma;
    int64_t limit;
    int32_t check_every, periods;
    int32_t skip, most;         // skip > 0: plain iterations of a period from the skip-th on; at most `most` of a period
    int32_t tasks_a, tasks_t;   // wave tasks of A~ and A~'
    int32_t force_last;   // not 0: one check that ends the solve with this status
};

// A lane's part of one wave task: its first entry, and its row with the number
// of its entries (5: more than four, in rows longer than 256).
struct SmallTask {
    int32_t e = 0;
    uint32_t w = 0;      // row + (entries << 24)
    __device__ __forceinline__ int32_t row() const { return (int32_t)(w & 0xffffffu); }
    __device__ __forceinline__ int32_t entries() const { return (int32_t)(w >> 24); }
};

// Task `task` of M (wave-uniform; the segments' rows 64 >> lg to a task, then the
// SELL-64 slices): 2^lg lanes per row, entries `stride` apart.
// lead: this lane holds an existing row's sum after the lane group's reduction.
__device__ __forceinline__ SmallTask small_task(const MatView &M, int32_t task, int32_t &lg, int32_t &stride,
                                                bool &lead) {
    SmallTask t;
    lg = 0;
    stride = 64;
    lead = false;
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    int32_t row = -1, e1 = 0, si = 0;
#pragma unroll 1
    for (; si < M.seg.nseg; ++si) {
        const Seg &g = M.seg.s[si];
        const int32_t w = (((g.row_end - g.row_begin) << g.lanes_log2) + 63) >> 6;
        if (task < w) break;
        task -= w;
    }
    if (si < M.seg.nseg) {
        lg = M.seg.s[si].lanes_log2;
        stride = 1 << lg;
        const int32_t r = M.seg.s[si].row_begin + ((task * 64 + lane) >> lg);
        if (r < M.seg.s[si].row_end) {
            row = r;
            t.e = M.rowptr[r] + (lane & (stride - 1));
            e1 = M.rowptr[r + 1];
        }
    } else if (task < M.nslices) {
        const int32_t r = M.R_long + task * 64 + lane;
        if (r < M.rows) {
            row = r;
            t.e = M.slice_ptr[task] + lane;
            e1 = M.slice_ptr[task + 1];
        }
    }
    if (row >= 0) {
        const int32_t left = e1 - t.e;
        const int32_t cnt = left > 0 ? min(5, (left + stride - 1) / stride) : 0;
        if (cnt == 0) t.e = 0;
        t.w = (uint32_t)row | ((uint32_t)cnt << 24);
        lead = (lane & (stride - 1)) == 0 || lg == 0;
    }
    return t;
}

// The first four entries of a lane, unconditional loads at indices clamped to
// its last entry (with predicated loads the compiler waits on each in turn);
// entries past it are zeros.
__device__ __forceinline__ void small_entries(const MatView &M, const SmallTask &t, int32_t stride,
                                              int32_t (&c)[4], double (&a)[4]) {
    const int32_t cnt = t.entries();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int32_t q = t.e + max(0, min(u, cnt - 1)) * stride;
        c[u] = M.colidx[q];
        a[u] = M.val[q];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (u >= cnt) a[u] = 0.0;
}

// acc + the entries from the fifth on of a lane that has more than four.
__device__ __forceinline__ double small_rest(const MatView &M, const SmallTask &t, int32_t stride, const double *v,
                                             double acc) {
    if (t.entries() > 4) {
        const int32_t e1 = M.rowptr[t.row() + 1];
        for (int32_t q = t.e + 4 * stride; q < e1; q += stride) acc = fma(M.val[q], v[M.colidx[q]], acc);
    }
    return acc;
}

__device__ __forceinline__ double small_sum(double acc, int32_t lg) {
    return group_reduce(acc, lg, [](double p, double q) { return p + q; });
}

// f(row, sum) on one lane of every row of M: the check iterations' products,
// a task at a time (little code and few registers beside the long epilogues).
template <class F>
__device__ __forceinline__ void small_each(const MatView &M, int32_t tasks, const double *v, F f) {
#pragma unroll 1
    for (int32_t k = (int32_t)(threadIdx.x >> 6); k < tasks; k += kSmallWaves) {
        int32_t lg, stride;
        bool lead;
        const SmallTask t = small_task(M, __builtin_amdgcn_readfirstlane(k), lg, stride, lead);
        int32_t c[4];
        double a[4], s = 0.0;
        small_entries(M, t, stride, c, a);
#pragma unroll
        for (int u = 0; u < 4; ++u) s = fma(a[u], v[c[u]], s);
        s = small_sum(small_rest(M, t, stride, v, s), __builtin_amdgcn_readfirstlane(lg));
        if (lead) f(t.row(), s);
    }
}

// An opaque copy: what is computed from it (addresses, unpacked indices) is
// computed again in each iteration instead of being kept in registers across
// the loop, which would spill.
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ SmallTask opaque(SmallTask t) {
    t.e = (int32_t)opaque((uint32_t)t.e);
    t.w = opaque(t.w);
    return t;
}

// One product's share of a wave in the plain iterations: its K tasks with the
// first four entries of every lane, column indices two to a register.
template <int K>
struct SmallProduct {
    SmallTask t[K];
    uint32_t ls;              // per task 4 bits: lanes per row (log2); 15: SELL-64 slice
    uint32_t lead;            // bit k: this lane leads a row of task k
    uint32_t c[K][2];
    double a[K][4];

    __device__ __forceinline__ int32_t lg(int k) const {
        const int32_t l = (int32_t)((ls >> (4 * k)) & 15u);
        return l == 15 ? 0 : l;
    }
    __device__ __forceinline__ int32_t stride(int k) const {
        const int32_t l = (int32_t)((ls >> (4 * k)) & 15u);
        return l == 15 ? 64 : 1 << l;
    }
    __device__ __forceinline__ void load(const MatView &M) {
        uint32_t w = 0;
        lead = 0;
        const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
#pragma unroll
        for (int k = 0; k < K; ++k) {
            int32_t l, s, ci[4];
            bool ld;
            t[k] = small_task(M, wave + k * kSmallWaves, l, s, ld);
            w |= (uint32_t)(s == 64 && l == 0 ? 15 : l) << (4 * k);
            lead |= ld ? 1u << k : 0u;
            small_entries(M, t[k], s, ci, a[k]);
            c[k][0] = (uint32_t)ci[0] | ((uint32_t)ci[1] << 16);
            c[k][1] = (uint32_t)ci[2] | ((uint32_t)ci[3] << 16);
        }
        ls = __builtin_amdgcn_readfirstlane(w);
    }
    template <class F>
    __device__ __forceinline__ void each(const MatView &M, const double *v, F f) const {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const SmallTask o = opaque(t[k]);
            const uint32_t c0 = opaque(c[k][0]), c1 = opaque(c[k][1]);
            double s = a[k][0] * v[c0 & 0xffffu];
            s = fma(a[k][1], v[c0 >> 16], s);
            s = fma(a[k][2], v[c1 & 0xffffu], s);
            s = fma(a[k][3], v[c1 >> 16], s);
            s = small_sum(small_rest(M, o, stride(k), v, s), lg(k));
            if ((lead >> k) & 1u) f(o.row(), s);
        }
    }
};

template <int K>
__global__ __launch_bounds__(kSmallThreads) void k_lp_small(SmallArgs a) {
    extern __shared__ double lds[];
    __shared__ DevState st;
    __shared__ double red[15][kSmallWaves];
    const int32_t n = a.n, m = a.m, tid = (int32_t)threadIdx.x;
    double *sx = lds;            // x_ext, at checks xhat
    double *x = sx + n, *x0 = x + n, *c = x0 + n, *lv = c + n, *uv = lv + n;
    double *y = uv + n, *y0 = y + m, *lc = y0 + m, *uc = lc + m, *yh = uc + m;
    if (tid == 0) st = *a.st;
    __syncthreads();
    if (st.done) return;
    for (int32_t r = tid; r < n; r += kSmallThreads) {
        x[r] = a.x[r];
        x0[r] = a.x0[r];
        c[r] = a.c[r];
        lv[r] = a.lv[r];
        uv[r] = a.uv[r];
    }
    for (int32_t r = tid; r < m; r += kSmallThreads) {
        y[r] = a.y[r];
        y0[r] = a.y0[r];
        lc[r] = a.lc[r];
        uc[r] = a.uc[r];
    }
    const double gam = a.gamma;
    const bool detect = a.K.detect != 0;
    __syncthreads();
    for (int32_t period = 0; period < a.periods; ++period) {
        double tau = st.tau, sigma = st.sigma;
        int32_t plain = st.plain_prev;
        if (a.skip == 0) {
            // ---- the check iteration
            const int64_t t = st.t_next;
            const bool is_last = a.force_last != 0 || t >= a.limit - 1;
            plain = is_last ? 0 : (int32_t)min((int64_t)a.check_every - 1, a.limit - 2 - t);
            small_each(a.AT, a.tasks_t, y, [&](int32_t r, double s) {
                const double xr = x[r], xh = clampd(xr - tau * (c[r] - s), lv[r], uv[r]);
                sx[r] = 2.0 * xh - xr;
                a.xhat[r] = xh;
                a.aty[r] = s;
            });
            __syncthreads();
            small_each(a.A, a.tasks_a, sx, [&](int32_t r, double s) {
                const double h = dual_prox(y[r], s, sigma, lc[r], uc[r]);
                yh[r] = h;
                a.yhat[r] = h;
            });
            __syncthreads();
            for (int32_t r = tid; r < n; r += kSmallThreads) sx[r] = a.xhat[r];
            __syncthreads();
            double v[13], mx[2] = {0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 13; ++q) v[q] = 0.0;
            small_each(a.AT, a.tasks_t, yh, [&](int32_t r, double q) {
                double w[6], rsum[2], rmax[2];
                check_n_terms(r, q, sx, x, x0, a.aty, a.Dc, a.c_o, a.lv_o, a.uv_o, a.q0, a.qhat, w, rsum, rmax);
#pragma unroll
                for (int i = 0; i < 6; ++i) v[i] += w[i];
                v[10] += rsum[0];
                v[11] += rsum[1];
                mx[0] = fmax(mx[0], rmax[0]);
                mx[1] = fmax(mx[1], rmax[1]);
            });
            small_each(a.A, a.tasks_a, sx, [&](int32_t r, double p) {
                double w[4], rsum[1], rmax[2];
                check_m_terms(r, p, yh, y, y0, a.Dr, a.lc_o, a.uc_o, a.p0, a.phat, w, rsum, rmax);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[6 + i] += w[i];
                v[12] += rsum[0];
                mx[0] = fmax(mx[0], rmax[0]);
                mx[1] = fmax(mx[1], rmax[1]);
            });
#pragma unroll
            for (int q = 0; q < 13; ++q) {
                const double s = wave_sum(v[q]);
                if ((tid & 63) == 0) red[q][tid >> 6] = s;
            }
            const double m0 = wave_max(mx[0]), m1 = wave_max(mx[1]);
            if ((tid & 63) == 0) {
                red[13][tid >> 6] = m0;
                red[14][tid >> 6] = m1;
            }
            __syncthreads();
            if (tid < 15) {   // the waves in order
                double s = red[tid][0];
                for (int w = 1; w < kSmallWaves; ++w) s = tid < 13 ? s + red[tid][w] : fmax(s, red[tid][w]);
                red[tid][0] = s;
            }
            __syncthreads();
            if (tid == 0) {
                double vn[6], vm[4], rs[3], rx[2];
#pragma unroll
                for (int i = 0; i < 6; ++i) vn[i] = red[i][0];
#pragma unroll
                for (int i = 0; i < 4; ++i) vm[i] = red[6 + i][0];
#pragma unroll
                for (int i = 0; i < 3; ++i) rs[i] = red[10 + i][0];
                rx[0] = red[13][0];
                rx[1] = red[14][0];
                check_decide(&st, vn, vm, rs, rx, detect && st.anchor_valid, a.K, plain, is_last ? 1 : 0,
                             a.force_last ? a.force_last : (int32_t)PDHG_ITERATION_LIMIT);
            }
            __syncthreads();
            if (st.done) break;
            {
                // restart, or the Halpern step of the check iteration
                const bool restart = st.action == 1;
                const int64_t k = st.k_check;
                const double ak = (double)(k + 1) / (double)(k + 2), bk = 1.0 / (double)(k + 2);
                for (int32_t r = tid; r < n; r += kSmallThreads) {
                    const double xh = sx[r];
                    if (restart) {
                        x[r] = xh;
                        x0[r] = xh;
                        a.q0[r] = a.qhat[r];
                    } else {
                        x[r] = ak * ((1.0 + gam) * xh - gam * x[r]) + bk * x0[r];
                    }
                }
                for (int32_t r = tid; r < m; r += kSmallThreads) {
                    const double h = yh[r];
                    if (restart) {
                        y[r] = h;
                        y0[r] = h;
                        a.p0[r] = a.phat[r];
                    } else {
                        y[r] = ak * ((1.0 + gam) * h - gam * y[r]) + bk * y0[r];
                    }
                }
            }
            tau = st.tau;
            sigma = st.sigma;
            __syncthreads();
        }
        int64_t k = st.k_base + a.skip;
        plain = a.skip + min(plain - a.skip, a.most);
        // ---- plain iterations; their matrix registers are loaded once per
        // period, so that the check's epilogues have the registers to themselves
        SmallProduct<K> T, R;   // A~' and A~
        T.load(a.AT);
        R.load(a.A);
        for (int32_t j = a.skip; j < plain; ++j, ++k) {
            const double ak = (double)(k + 1) / (double)(k + 2), bk = 1.0 / (double)(k + 2);
            T.each(a.AT, y, [&](int32_t r, double s) {
                const double xr = x[r], xh = clampd(xr - tau * (c[r] - s), lv[r], uv[r]);
                sx[r] = 2.0 * xh - xr;
                x[r] = ak * ((1.0 + gam) * xh - gam * xr) + bk * x0[r];
            });
            __syncthreads();
            R.each(a.A, sx, [&](int32_t r, double s) {
                const double yr = y[r], h = dual_prox(yr, s, sigma, lc[r], uc[r]);
                y[r] = ak * ((1.0 + gam) * h - gam * yr) + bk * y0[r];
            });
            __syncthreads();
        }
    }
    for (int32_t r = tid; r < n; r += kSmallThreads) {
        a.x[r] = x[r];
        a.x0[r] = x0[r];
    }
    for (int32_t r = tid; r < m; r += kSmallThreads) {
        a.y[r] = y[r];
        a.y0[r] = y0[r];
    }
    if (tid == 0) *a.st = st;
}

// ---------------------------------------------------------------------------
// host side

static int32_t wave_tasks(const HMat &M) {
    int32_t w = M.nslices;
    for (int32_t q = 0; q < M.seg.nseg; ++q) {
        const Seg &g = M.seg.s[q];
        w += (int32_t)ceil_div((int64_t)(g.row_end - g.row_begin) << g.lanes_log2, 64);
    }
    return w;
}

// The wave tasks per wave of the larger product, or 0 where the LP does not
// fit: sparse, no quadratic term, layouts left to the library, vectors within
// LDS and at most kSmallMost tasks a wave.
// Measured, us per iteration (checks included) against 6.9 to 7.1 as launches:
// planted LPs 200 x 400 (1,562 entries, one task a wave) 1.67, 400 x 800 (3,157,
// two) 2.61, 800 x 1,600 (4,920, two) 2.95, 1,150 x 2,300 (7,001, three) 4.18, 400 x 800
// (7,901, three) 4.67; a fourth task would cost another microsecond and spill.
// Streaming the entries of up to eight tasks from L2 instead took 9.7 to 17 us.
int32_t small_lp_fits(const Handle &h) {
    if (h.dense || h.q_kind || h.m < 1 || h.A.nnz == 0 || h.opt.panel_rows >= 0 || h.opt.hot_cols >= 0) return 0;
    if (6 * (int64_t)h.n + 5 * (int64_t)h.m > kSmallDoubles) return 0;
    const int32_t tasks = std::max(wave_tasks(h.A), wave_tasks(h.AT));
    const int32_t per_wave = (int32_t)ceil_div(tasks, kSmallWaves);
    return per_wave <= kSmallMost ? std::max(1, per_wave) : 0;
}

template <int K>
static void launch_small_t(Handle &h, const SmallArgs &a) {
    const size_t lds = sizeof(double) * (6 * (size_t)h.n + 5 * (size_t)h.m);
    PDHG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_lp_small<K>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    k_lp_small<K><<<1, kSmallThreads, lds, h.stream>>>(a);
    PDHG_HIP(hipGetLastError());
}

// Up to `periods` check periods from the handle's state, each with at most `most`
// plain iterations; skip > 0: the plain iterations of the current period from the
// skip-th on; force_last: one check that ends the solve with that status.
void launch_small_lp(Handle &h, int32_t periods, int32_t skip, int32_t most, int32_t force_last) {
    SmallArgs a;
    a.A = view(h.A);
    a.AT = view(h.AT);
    a.m = h.m;
    a.n = h.n;
    a.x = h.x.p;
    a.x0 = h.x0.p;
    a.y = h.y.p;
    a.y0 = h.y0.p;
    a.xhat = h.xhat.p;
    a.yhat = h.yhat.p;
    a.aty = h.aty.p;
    a.c = h.c.p;
    a.lv = h.lv.p;
    a.uv = h.uv.p;
    a.lc = h.lc.p;
    a.uc = h.uc.p;
    a.Dr = h.Dr.p;
    a.Dc = h.Dc.p;
    a.c_o = h.c_o.p;
    a.lv_o = h.lv_o.p;
    a.uv_o = h.uv_o.p;
    a.lc_o = h.lc_o.p;
    a.uc_o = h.uc_o.p;
    a.p0 = h.p0.p;
    a.q0 = h.q0.p;
    a.phat = h.phat.p;
    a.qhat = h.qhat.p;
    a.st = h.st.p;
    a.K = lp_constants(h);
    a.gamma = h.opt.gamma;
    a.limit = h.opt.iteration_limit;
    a.check_every = h.opt.check_every;
    a.periods = force_last ? 1 : periods;
    a.skip = skip;
    a.most = most;
    a.force_last = force_last;
    a.tasks_a = wave_tasks(h.A);
    a.tasks_t = wave_tasks(h.AT);
    switch (small_lp_fits(h)) {
        case 1: launch_small_t<1>(h, a); break;
        case 2: launch_small_t<2>(h, a); break;
        default: launch_small_t<3>(h, a); break;
    }
}

}  // namespace pdhg
