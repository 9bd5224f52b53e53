// Batched rAPDHG (see batch_qp.hip) for QPs with one constraint row, the
// portfolio's budget: every thread keeps its S columns of the instance whole in
// registers - the S rows of F~ (R = the rank rounded up to 8), iterates, bounds
// and its entry of the constraint row - and every thread carries the row's y.
//
// What bounds it: an iteration is two dependent workgroup reductions, t = F~'v
// (R values) and A~ x_ext (one), each a barrier, around some 400 vector
// instructions per wave. The general kernels read F~ from L2 twice per
// iteration (160 KB at n = 500, rank 20) and walk the constraint row with one
// wave; here an iteration reads no matrix and no vector from memory. Measured
// with n = 500, rank 20, 512 instances (two per CU): 1,000 unrolled iterations
// 9.16 -> 2.52 ms, their reverse pass 11.14 -> 2.49 ms, the solve to 1e-4 (769
// iterations the slowest) 6.22 -> 1.43 ms.
//
// t reaches the lanes as scalars: lane p of every wave adds the waves' partial
// sums of value p in wave order, and a lane read makes each a scalar operand of
// the F~ t products, which saves the second barrier and R LDS reads per column.
#include <algorithm>

#include "batch_qp.hpp"

namespace pdhg {

// An instance in registers. Columns j = thread + q BT; those past n hold zeros
// and F~ rows of zeros, so they add nothing to any sum.
template <int BT, int S, int R>
struct RowQP {
    static constexpr int NW = BT / 64;
    double f[S][R], tv[S];
    double c[S], lv[S], uv[S], dd[S];
    double lc, uc;
    double *shr, *sh1;   // LDS: [R + 8][NW] partial sums, [2][NW]
    int32_t n, tid;

    __device__ __forceinline__ int32_t col(int q) const { return tid + q * BT; }

    __device__ __forceinline__ void load_matrix(const QArgs &a) {
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = col(q);
            const bool in = j < n;
#pragma unroll
            for (int p = 0; p < R; ++p) f[q][p] = in ? a.FT[(size_t)p * n + j] : 0.0;
            const int32_t e = in ? a.trp[j] : 0, e1 = in ? a.trp[j + 1] : 0;
            tv[q] = e1 > e ? a.tva[e] : 0.0;
        }
    }

    // Eight sums over the workgroup into scalars (all threads).
    __device__ __forceinline__ void sum8(const double (&v)[8], double (&out)[8]) {
        const int lane = tid & 63, wave = tid >> 6;
        const double ws = wave_sum_x8(v);
        const int u = 4 * ((lane >> 3) & 1) + 2 * ((lane >> 4) & 1) + ((lane >> 5) & 1);
        __syncthreads();
        if ((lane & 7) == 0) shr[u * NW + wave] = ws;
        __syncthreads();
        const double s = waves_total(lane & 7);
#pragma unroll
        for (int q = 0; q < 8; ++q) out[q] = lane_value(s, q);
    }
    __device__ __forceinline__ double waves_total(int p) const {
        double s = shr[p * NW];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += shr[p * NW + w];
        return s;
    }

    // The partial sums of F~'w, written for the barrier that the caller places.
    __device__ __forceinline__ void factor_partials(const double (&w)[S]) {
        const int lane = tid & 63, wave = tid >> 6;
        const int u = 4 * ((lane >> 3) & 1) + 2 * ((lane >> 4) & 1) + ((lane >> 5) & 1);
#pragma unroll
        for (int p0 = 0; p0 < R; p0 += 8) {
            double s[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                s[i] = f[0][p0 + i] * w[0];
#pragma unroll
                for (int q = 1; q < S; ++q) s[i] = fma(f[q][p0 + i], w[q], s[i]);
            }
            const double ws = wave_sum_x8(s);
            if ((lane & 7) == 0) shr[(p0 + u) * NW + wave] = ws;
        }
    }
    // out = Q~ w = F~ t + d~ w, t from the partial sums.
    __device__ __forceinline__ void factor_apply(const double (&w)[S], double (&out)[S]) {
        const int lane = tid & 63;
        const double tp = waves_total(lane < R ? lane : 0);
#pragma unroll
        for (int q = 0; q < S; ++q) out[q] = 0.0;
#pragma unroll
        for (int p = 0; p < R; ++p) {
            const double t = lane_value(tp, p);
#pragma unroll
            for (int q = 0; q < S; ++q) out[q] = fma(f[q][p], t, out[q]);
        }
#pragma unroll
        for (int q = 0; q < S; ++q) out[q] = out[q] + dd[q] * w[q];
    }
    __device__ __forceinline__ void quad(const double (&w)[S], double (&out)[S]) {
        __syncthreads();
        factor_partials(w);
        __syncthreads();
        factor_apply(w, out);
    }
    // A~ w, the same value in every thread. sh1 may be written again once a
    // barrier has followed.
    __device__ __forceinline__ double row_partial(const double (&w)[S]) const {
        double s = tv[0] * w[0];
#pragma unroll
        for (int q = 1; q < S; ++q) s = fma(tv[q], w[q], s);
        return s;
    }
    __device__ __forceinline__ double row_total(double part) {
        const double s = wave_sum(part);
        if ((tid & 63) == 0) sh1[tid >> 6] = s;
        __syncthreads();
        double t = sh1[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += sh1[w];
        return t;
    }

    // Scaled data of instance b, and the norms |c~|, |b~|, |c|, |b|.
    __device__ __forceinline__ void prepare(const QArgs &a, int32_t b, double &cn, double &bn, double &cnorm,
                                            double &bnorm) {
        double nrm[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = col(q);
            c[q] = lv[q] = uv[q] = dd[q] = 0.0;
            if (j < n) {
                const double d = a.Dc[j], co = a.c_o[(size_t)b * n + j];
                c[q] = d * co;
                lv[q] = a.lv_o[(size_t)b * n + j] / d;
                uv[q] = a.uv_o[(size_t)b * n + j] / d;
                dd[q] = (d * d) * a.d_o[(size_t)b * n + j];
                nrm[0] += c[q] * c[q];
                nrm[2] += co * co;
            }
        }
        const double d = a.Dr[0], lo = a.lc_o[b], uo = a.uc_o[b];
        lc = d * lo;
        uc = d * uo;
        double bb = 0.0, bo = 0.0;
        if (isfinite(lc)) bb = fmax(bb, fabs(lc));
        if (isfinite(uc)) bb = fmax(bb, fabs(uc));
        if (isfinite(lo)) bo = fmax(bo, fabs(lo));
        if (isfinite(uo)) bo = fmax(bo, fabs(uo));
        double tot[8];
        sum8(nrm, tot);
        cn = sqrt(tot[0]);
        bn = sqrt(bb * bb);
        cnorm = sqrt(tot[2]);
        bnorm = sqrt(bo * bo);
    }
};

// The iterate of one instance: columns in registers, the row's y everywhere.
template <int S>
struct RowState {
    double x[S], xb[S], y, yb;
};

// One iteration (Algorithm 2); v and the projection states come back for the
// unrolled forward. oe = omega / eta and sigma = eta omega change at restarts
// only.
template <int BT, int S, int R>
__device__ __forceinline__ void row_step(RowQP<BT, S, R> &Q, RowState<S> &z, int64_t k, double oe, double sigma,
                                         double normq, double (&v)[S], bool (&inside)[S], bool &at_u, bool &at_l) {
    const double beta = 2.0 / (double)(k + 2), theta = beta;
    const double tau = 1.0 / (oe + 2.0 * normq / (double)(k + 1));
    double qv[S], xe[S];
#pragma unroll
    for (int q = 0; q < S; ++q) v[q] = (1.0 - beta) * z.xb[q] + beta * z.x[q];
    Q.factor_partials(v);
    __syncthreads();
    Q.factor_apply(v, qv);
#pragma unroll
    for (int q = 0; q < S; ++q) {
        const double u = z.x[q] - tau * (qv[q] + Q.c[q] - Q.tv[q] * z.y);
        inside[q] = u > Q.lv[q] && u < Q.uv[q];
        const double xp = clampd(u, Q.lv[q], Q.uv[q]);
        xe[q] = 2.0 * xp - z.x[q];
        z.x[q] = xp;
        z.xb[q] = (1.0 - theta) * z.xb[q] + theta * xp;
    }
    const double av = Q.row_total(Q.row_partial(xe));
    const double w = z.y / sigma - av;
    at_u = w < -Q.uc;
    at_l = w > -Q.lc;
    z.y = sigma * (w - clampd(w, -Q.uc, -Q.lc));
    z.yb = (1.0 - theta) * z.yb + theta * z.y;
}

// KKT terms of the averages in the original space (qcheck of batch_qp.hip).
template <int BT, int S, int R>
__device__ __forceinline__ void row_check(const QArgs &a, RowQP<BT, S, R> &Q, const RowState<S> &z,
                                          const double (&x0)[S], double y0, int32_t b, double (&out)[8]) {
    double qv[S];
    Q.quad(z.xb, qv);
    double v[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) v[p] = 0.0;
#pragma unroll
    for (int q = 0; q < S; ++q) {
        const int32_t j = Q.col(q);
        if (j >= Q.n) continue;
        const size_t o = (size_t)b * Q.n + j;
        const double xb = z.xb[q], d0 = xb - x0[q], d = a.Dc[j], co = a.c_o[o];
        v[0] += d0 * d0;
        const double qx = qv[q] / d, xo = d * xb;
        const double g = qx + co - Q.tv[q] * z.yb / d;
        const double lo = a.lv_o[o], hi = a.uv_o[o];
        const bool lf = isfinite(lo), uf = isfinite(hi);
        const double lam = (!lf && !uf) ? 0.0 : (lf && !uf) ? fmax(g, 0.0) : (!lf && uf) ? fmin(g, 0.0) : g;
        const double rd = g - lam;
        v[1] += rd * rd;
        v[2] += xo * qx;
        v[3] += co * xo;
        v[4] += (lf ? lo * fmax(lam, 0.0) : 0.0) - (uf ? hi * fmax(-lam, 0.0) : 0.0);
    }
    v[5] = Q.row_partial(z.xb);
    Q.sum8(v, out);
    const double d = a.Dr[0], ax = out[5] / d, lo = a.lc_o[b], hi = a.uc_o[b];
    const double rpr = ax - clampd(ax, lo, hi), yo = d * z.yb, e0 = z.yb - y0;
    out[5] = rpr * rpr;
    out[6] = (isfinite(lo) ? lo * fmax(yo, 0.0) : 0.0) - (isfinite(hi) ? hi * fmax(-yo, 0.0) : 0.0);
    out[7] = e0 * e0;
}

// Ray terms of the averages against the restart anchor (qray of batch_qp.hip).
template <int BT, int S, int R>
__device__ __forceinline__ void row_rays(const QArgs &a, RowQP<BT, S, R> &Q, const RowState<S> &z,
                                         const double (&x0)[S], double y0, int32_t b, double (&rs)[3],
                                         double (&rm)[2]) {
    double dx[S], qv[S];
#pragma unroll
    for (int q = 0; q < S; ++q) dx[q] = z.xb[q] - x0[q];
    Q.quad(dx, qv);
    double v[8], t[8], m0 = 0.0, m1 = 0.0;
#pragma unroll
    for (int p = 0; p < 8; ++p) v[p] = 0.0;
#pragma unroll
    for (int q = 0; q < S; ++q) {
        const int32_t j = Q.col(q);
        if (j >= Q.n) continue;
        const size_t o = (size_t)b * Q.n + j;
        const double d = a.Dc[j];
        m1 = fmax(m1, fabs(qv[q] / d));
        double s[2], mx[2];
        ray_col_terms(Q.tv[q] * z.yb, Q.tv[q] * y0, d, dx[q], a.c_o[o], a.lv_o[o], a.uv_o[o], s, mx);
        v[0] += s[0];
        v[1] += s[1];
        m0 = fmax(m0, mx[0]);
        m1 = fmax(m1, mx[1]);
    }
    v[2] = Q.row_partial(dx);
    Q.sum8(v, t);
    double s[1], mx[2];
    ray_row_terms(t[2], 0.0, a.Dr[0], z.yb - y0, a.lc_o[b], a.uc_o[b], s, mx);
    rs[0] = t[0];
    rs[1] = t[1];
    rs[2] = s[0];
    const double w0 = wave_max(fmax(m0, mx[0])), w1 = wave_max(fmax(m1, mx[1]));
    constexpr int NW = BT / 64;
    __syncthreads();
    if ((Q.tid & 63) == 0) {
        Q.shr[Q.tid >> 6] = w0;
        Q.shr[NW + (Q.tid >> 6)] = w1;
    }
    __syncthreads();
    rm[0] = Q.shr[0];
    rm[1] = Q.shr[NW];
    for (int w = 1; w < NW; ++w) {
        rm[0] = fmax(rm[0], Q.shr[w]);
        rm[1] = fmax(rm[1], Q.shr[NW + w]);
    }
}

// Point x = proj_X(x_init / D_c), y = proj_Y(y_init / D_r), averages equal to it.
template <int BT, int S, int R>
__device__ __forceinline__ void row_start(const QArgs &a, const RowQP<BT, S, R> &Q, RowState<S> &z, const double *xi,
                                          const double *yi) {
#pragma unroll
    for (int q = 0; q < S; ++q) {
        const int32_t j = Q.col(q);
        const double v0 = xi && j < Q.n ? xi[j] / a.Dc[j] : 0.0;
        z.x[q] = z.xb[q] = j < Q.n ? clampd(v0, Q.lv[q], Q.uv[q]) : 0.0;
    }
    const double v0 = yi ? yi[0] / a.Dr[0] : 0.0;
    z.y = z.yb = clampd(v0, isfinite(Q.uc) ? -INFINITY : 0.0, isfinite(Q.lc) ? INFINITY : 0.0);
}

// The restart test of Algorithm 2 on the weighted KKT norm.
struct RowRestart {
    double start = 0.0, prev = 0.0;
    __device__ __forceinline__ bool due(const QOpts &o, double r, int64_t t, int64_t k) {
        bool re = false;
        if (t == 0) start = prev = r;
        else if (r <= o.beta_suff * start || (r <= o.beta_nec * start && r > prev) || (double)k >= o.beta_art * (double)t)
            re = true;
        else prev = r;
        if (re) start = prev = r;
        return re;
    }
};

#define ROW_KERNEL __global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(2)))

template <int BT, int S, int R>
ROW_KERNEL void k_bqp_row_solve(QArgs a, QOpts o) {
    __shared__ double shr[R * (BT / 64)], sh1[BT / 64];
    RowQP<BT, S, R> Q;
    Q.n = a.n;
    Q.tid = (int32_t)threadIdx.x;
    Q.shr = shr;
    Q.sh1 = sh1;
    Q.load_matrix(a);
    for (;;) {
        const int32_t b = __builtin_amdgcn_readfirstlane(qnext<BT>(a.queue));
        if (b >= a.B) return;
        double cn, bn, cnorm, bnorm;
        Q.prepare(a, b, cn, bn, cnorm, bnorm);
        RowState<S> z;
        row_start(a, Q, z, a.x_init ? a.x_init + (size_t)b * a.n : nullptr, a.y_init ? a.y_init + b : nullptr);
        double x0[S], y0 = z.y;
#pragma unroll
        for (int q = 0; q < S; ++q) x0[q] = z.x[q];
        const double normq = a.normq[b];
        double omega = (cn > 1e-10 && bn > 1e-10) ? cn / bn : 1.0;
        double oe = omega / a.eta, sigma = a.eta * omega;
        int64_t t = 0, k = 0, restarts = 0;
        int32_t tc = 0;   // t modulo check_every
        RowRestart rr;
        double P = 0.0, D = 0.0, kkt = 0.0, rp = 0.0, rd = 0.0, rg = 0.0, ray_scale = 0.0;
        int32_t status = 0;
        __syncthreads();
        for (;;) {
            double v[S];
            bool in[S], au, al;
            row_step(Q, z, k, oe, sigma, normq, v, in, au, al);
            const bool last = t + 1 >= o.limit;
            bool restart = false;
            if (tc == 0 || last) {
                double w[8];
                row_check(a, Q, z, x0, y0, b, w);
                P = 0.5 * w[2] + w[3];
                D = -0.5 * w[2] + w[6] + w[4];
                const double ap = sqrt(w[5]), ad = sqrt(w[1]), ag = fabs(P - D);
                rp = ap / (1.0 + bnorm);
                rd = ad / (1.0 + cnorm);
                rg = ag / (1.0 + fabs(P) + fabs(D));
                kkt = rp;
                if (rd > kkt || isnan(rd)) kkt = rd;
                if (rg > kkt || isnan(rg)) kkt = rg;
                if (isnan(kkt)) { status = PDHG_NUMERICAL_ERROR; break; }
                if (kkt <= o.eps) { status = PDHG_OPTIMAL; break; }
                if (o.detect && restarts > 0) {
                    double rs[3], rm[2];
                    row_rays(a, Q, z, x0, y0, b, rs, rm);
                    const double obj_d = rs[0] + rs[2], obj_p = rs[1];
                    if (o.eps_pinf > 0.0 && obj_d > 0.0 && rm[0] <= o.eps_pinf * obj_d) {
                        status = PDHG_PRIMAL_INFEASIBLE;
                        ray_scale = 1.0 / obj_d;
                        break;
                    }
                    if (o.eps_dinf > 0.0 && obj_p < 0.0 && rm[1] <= o.eps_dinf * (-obj_p)) {
                        status = PDHG_DUAL_INFEASIBLE;
                        ray_scale = -1.0 / obj_p;
                        break;
                    }
                }
                if (last) { status = PDHG_ITERATION_LIMIT; break; }
                restart = rr.due(o, sqrt(omega * ap * ap + ad * ad / omega + ag * ag), t, k);
                if (restart) {
                    omega = batch_new_omega(omega, sqrt(w[0]), sqrt(w[7]));
                    oe = omega / a.eta;
                    sigma = a.eta * omega;
#pragma unroll
                    for (int q = 0; q < S; ++q) z.x[q] = x0[q] = z.xb[q];
                    z.y = y0 = z.yb;
                    ++restarts;
                }
                __syncthreads();
            }
            k = restart ? 0 : k + 1;
            ++t;
            tc = tc + 1 == o.check_every ? 0 : tc + 1;
        }
        const bool xray = status == PDHG_DUAL_INFEASIBLE, yray = status == PDHG_PRIMAL_INFEASIBLE;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = Q.col(q);
            if (j < a.n) a.x_out[(size_t)b * a.n + j] = a.Dc[j] * (xray ? (z.xb[q] - x0[q]) * ray_scale : z.xb[q]);
        }
        if (threadIdx.x == 0) {
            a.y_out[b] = a.Dr[0] * (yray ? (z.yb - y0) * ray_scale : z.yb);
            double *r = a.res + (size_t)b * 12;
            r[0] = P; r[1] = D; r[2] = rp; r[3] = rd; r[4] = rg; r[5] = kkt; r[6] = omega;
            r[7] = normq; r[8] = (double)(t + 1); r[9] = (double)restarts; r[10] = status; r[11] = 0.0;
        }
        __syncthreads();
    }
}

// Unrolled rAPDHG (k_bqp_unrolled): exactly T iterations from zero.
template <int BT, int S, int R>
ROW_KERNEL void k_bqp_row_unrolled(QArgs a, QOpts o) {
    __shared__ double shr[R * (BT / 64)], sh1[BT / 64];
    RowQP<BT, S, R> Q;
    Q.n = a.n;
    Q.tid = (int32_t)threadIdx.x;
    Q.shr = shr;
    Q.sh1 = sh1;
    Q.load_matrix(a);
    const int32_t n = a.n, xw = (n + 63) >> 6, wave = Q.tid >> 6;
    const int64_t nck = (a.T + kCkpt - 1) / kCkpt;
    const size_t cks = 2 * (size_t)n + 2;
    for (;;) {
        const int32_t b = __builtin_amdgcn_readfirstlane(qnext<BT>(a.queue));
        if (b >= a.B) return;
        double cn, bn, cnorm, bnorm;
        Q.prepare(a, b, cn, bn, cnorm, bnorm);
        RowState<S> z;
        row_start<BT, S, R>(a, Q, z, nullptr, nullptr);
        double x0[S], y0 = z.y;
#pragma unroll
        for (int q = 0; q < S; ++q) x0[q] = z.x[q];
        const double normq = a.normq[b];
        double omega = (cn > 1e-10 && bn > 1e-10) ? cn / bn : 1.0;
        double oe = omega / a.eta, sigma = a.eta * omega;
        uint8_t *rs_ = a.restart + (size_t)b * a.T;
        double *om_ = a.omega + (size_t)b * a.T;
        int32_t *kk_ = a.kk + (size_t)b * a.T;
        RowRestart rr;
        int64_t k = 0;
        int32_t tc = 0, tk = 0;   // t modulo check_every and kCkpt
        __syncthreads();
        for (int64_t t = 0; t < a.T; ++t) {
            if (a.replay) {
                omega = om_[t];
                oe = omega / a.eta;
                sigma = a.eta * omega;
            }
            if (tk == 0 && !a.vall) {   // a reverse pass that recomputes starts here
                double *ck = a.ckpt + ((size_t)b * nck + t / kCkpt) * cks;
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const int32_t j = Q.col(q);
                    if (j < n) {
                        ck[j] = z.x[q];
                        ck[n + j] = z.xb[q];
                    }
                }
                if (Q.tid == 0) {
                    ck[2 * (size_t)n] = z.y;
                    ck[2 * (size_t)n + 1] = z.yb;
                }
            }
            double v[S];
            bool in[S], au, al;
            row_step(Q, z, k, oe, sigma, normq, v, in, au, al);
            uint64_t *xmt = a.xmask + ((size_t)b * a.T + t) * xw;
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t j = Q.col(q);
                const uint64_t bits = __ballot(j < n && in[q]);
                if ((Q.tid & 63) == 0 && j < n) xmt[q * (BT / 64) + wave] = bits;
                if (a.vall && j < n) a.vall[((size_t)b * a.T + t) * n + j] = v[q];
            }
            if (Q.tid == 0) {
                uint64_t *ymt = a.ymask + ((size_t)b * a.T + t) * 2;
                ymt[0] = au ? 1 : 0;
                ymt[1] = al ? 1 : 0;
                om_[t] = omega;
                kk_[t] = (int32_t)k;
            }
            if (t + 1 >= a.T) break;
            bool restart = a.replay ? rs_[t] != 0 : false;
            if (!a.replay && tc == 0) {
                double w[8];
                row_check(a, Q, z, x0, y0, b, w);
                const double P = 0.5 * w[2] + w[3];
                const double D = -0.5 * w[2] + w[6] + w[4];
                const double ap = sqrt(w[5]), ad = sqrt(w[1]), ag = fabs(P - D);
                restart = rr.due(o, sqrt(omega * ap * ap + ad * ad / omega + ag * ag), t, k);
                if (restart) {
                    omega = batch_new_omega(omega, sqrt(w[0]), sqrt(w[7]));
                    oe = omega / a.eta;
                    sigma = a.eta * omega;
                }
                __syncthreads();
            }
            if (Q.tid == 0 && !a.replay) rs_[t] = restart ? 1 : 0;
            if (restart) {
#pragma unroll
                for (int q = 0; q < S; ++q) z.x[q] = x0[q] = z.xb[q];
                z.y = y0 = z.yb;
            }
            k = restart ? 0 : k + 1;
            tc = tc + 1 == o.check_every ? 0 : tc + 1;
            tk = tk + 1 == kCkpt ? 0 : tk + 1;
        }
        if (Q.tid == 0 && !a.replay) rs_[a.T - 1] = 0;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = Q.col(q);
            if (j < n) a.x_out[(size_t)b * n + j] = a.Dc[j] * z.xb[q];
        }
        if (Q.tid == 0) a.y_out[b] = a.Dr[0] * z.yb;
        __syncthreads();
    }
}

// Reverse pass of the unrolled iterations (k_bqp_backward), every momentum
// point kept by the forward. The row's sum is only needed by the next reversed
// iteration, so it shares the factor product's barrier: with two sets of
// partial sums used in turn, an iteration has one.
template <int BT, int S, int R>
ROW_KERNEL void k_bqp_row_backward(QArgs a, QOpts) {
    constexpr int NW = BT / 64;
    __shared__ double sh[2][(R + 1) * NW];
    RowQP<BT, S, R> Q;
    Q.n = a.n;
    Q.tid = (int32_t)threadIdx.x;
    Q.sh1 = nullptr;
    Q.load_matrix(a);
    const int32_t n = a.n, xw = (n + 63) >> 6, wave = Q.tid >> 6, lane = Q.tid & 63;
    for (;;) {
        const int32_t b = __builtin_amdgcn_readfirstlane(qnext<BT>(a.queue));
        if (b >= a.B) return;
        const double normq = a.normq[b];
        const uint8_t *rs_ = a.restart + (size_t)b * a.T;
        const double *om_ = a.omega + (size_t)b * a.T;
        const int32_t *kk_ = a.kk + (size_t)b * a.T;
        double bx[S], bxb[S], gc[S], gd[S];
        double by = 0.0, byb = a.Dr[0] * (a.gy ? a.gy[b] : 0.0), glc = 0.0, guc = 0.0;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = Q.col(q);
            bx[q] = gc[q] = gd[q] = bxb[q] = Q.dd[q] = 0.0;
            if (j < n) {
                const double d = a.Dc[j];
                bxb[q] = d * a.gx[(size_t)b * n + j];
                Q.dd[q] = (d * d) * a.d_o[(size_t)b * n + j];
            }
        }
        // what the recorded iteration t left, loaded one iteration ahead
        struct Rec {
            double vt[S], omega;
            uint64_t xm[S], yu, yl;
            int32_t k;
            bool re;
        };
        auto load = [&](int64_t t) {
            Rec r;
            const size_t o = (size_t)b * a.T + t;
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t j = Q.col(q);
                r.vt[q] = j < n ? a.vall[o * n + j] : 0.0;
                r.xm[q] = j < n ? a.xmask[o * xw + q * NW + wave] : 0;
            }
            r.yu = a.ymask[o * 2];
            r.yl = a.ymask[o * 2 + 1];
            r.omega = om_[t];
            r.k = kk_[t];
            r.re = t < a.T - 1 && rs_[t] != 0;
            return r;
        };
        Rec nx = load(a.T - 1);
        double omega_at = -1.0, oe = 0.0, sigma = 1.0;
        int32_t buf = 0;
        for (int64_t t = a.T - 1; t >= 0; --t) {
            const Rec r = nx;
            if (t > 0) nx = load(t - 1);
            if (r.re) {
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    bxb[q] += bx[q];
                    bx[q] = 0.0;
                }
                byb += by;
                by = 0.0;
            }
            if (r.omega != omega_at) {
                omega_at = r.omega;
                oe = r.omega / a.eta;
                sigma = a.eta * r.omega;
            }
            const double beta = 2.0 / (double)((int64_t)r.k + 2), theta = beta;
            const double tau = 1.0 / (oe + 2.0 * normq / (double)((int64_t)r.k + 1));
            // averages and the dual step
            const double byp = by + theta * byb;
            byb = (1.0 - theta) * byb;
            const bool at_u = (r.yu & 1) != 0, at_l = (r.yl & 1) != 0;
            const double w = (at_u || at_l) ? sigma * byp : 0.0;
            if (at_u) guc += sigma * byp;
            if (at_l) glc += sigma * byp;
            by = w / sigma;
            // x_ext = 2x+ - x and the primal step
            double bqv[S], xe[S];
#pragma unroll
            for (int q = 0; q < S; ++q) {
                bx[q] = bx[q] + theta * bxb[q];
                bxb[q] = (1.0 - theta) * bxb[q];
                const double bxe = Q.tv[q] * -w;
                const double bxp = bx[q] + 2.0 * bxe;
                const double bu = ((r.xm[q] >> lane) & 1) ? bxp : 0.0;
                bx[q] = -bxe + bu;
                bqv[q] = -tau * bu;
                gc[q] += -tau * bu;
                xe[q] = tau * bu;
            }
            // F~'bqv and A~ xe; Q~ bqv and the gradient in d~
            Q.shr = sh[buf];
            buf ^= 1;
            Q.factor_partials(bqv);
            const double rowp = wave_sum(Q.row_partial(xe));
            if (lane == 0) Q.shr[R * NW + wave] = rowp;
            __syncthreads();
            double bv[S];
            Q.factor_apply(bqv, bv);
            by += Q.waves_total(R);
#pragma unroll
            for (int q = 0; q < S; ++q) {
                gd[q] += bqv[q] * r.vt[q];
                bxb[q] += (1.0 - beta) * bv[q];
                bx[q] += beta * bv[q];
            }
        }
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = Q.col(q);
            if (j < n) {
                const double d = a.Dc[j];
                a.gc[(size_t)b * n + j] = d * gc[q];
                a.gd[(size_t)b * n + j] = (d * d) * gd[q];
            }
        }
        if (Q.tid == 0) {
            a.glc[b] = isfinite(a.lc_o[b]) ? a.Dr[0] * glc : 0.0;
            a.guc[b] = isfinite(a.uc_o[b]) ? a.Dr[0] * guc : 0.0;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// host side

// Two columns per thread hold 2 R doubles of F~ in the 256 registers of a
// two-waves-per-SIMD kernel (R <= 32: 128 of them); the forms of rank 25 to 32 then
// keep up to 58 others in scratch memory, across checks. Up to 256 columns take one
// per thread, and 512 threads carry up to 1,024 columns.
int32_t qrow_fits(const BatchHandle &h) {
    if (h.m != 1 || h.q_rank < 1 || h.q_rank > kRmax || h.n > 1024) return 0;
    return h.n <= 512 ? 256 : 512;
}

template <int BT, int S, int R>
static void qrow_launch_t(BatchHandle &h, QK which, const QArgs &a, const QOpts &o) {
    auto go = [&](void (*kernel)(QArgs, QOpts)) {
        int per_cu = 0;
        PDHG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kernel), BT, 0));
        int32_t wg = std::min(h.B, std::max(1, per_cu) * h.q_cus);
        if (h.workgroups > 0) wg = std::min(wg, h.workgroups);
        kernel<<<wg, BT, 0, h.stream>>>(a, o);
    };
    if (which == QK::solve) go(k_bqp_row_solve<BT, S, R>);
    else if (which == QK::unrolled) go(k_bqp_row_unrolled<BT, S, R>);
    else go(k_bqp_row_backward<BT, S, R>);
}

template <int BT, int S>
static void qrow_launch_r(BatchHandle &h, QK which, const QArgs &a, const QOpts &o) {
    switch ((a.r + 7) >> 3) {
        case 1: qrow_launch_t<BT, S, 8>(h, which, a, o); break;
        case 2: qrow_launch_t<BT, S, 16>(h, which, a, o); break;
        case 3: qrow_launch_t<BT, S, 24>(h, which, a, o); break;
        default: qrow_launch_t<BT, S, 32>(h, which, a, o); break;
    }
}

void qrow_launch(BatchHandle &h, QK which, const QArgs &a, const QOpts &o) {
    PDHG_HIP(hipMemsetAsync(h.queue.p, 0, sizeof(int32_t), h.stream));
    if (a.n <= 256) qrow_launch_r<256, 1>(h, which, a, o);
    else if (a.n <= 512) qrow_launch_r<256, 2>(h, which, a, o);
    else qrow_launch_r<512, 2>(h, which, a, o);
    PDHG_HIP(hipGetLastError());
    PDHG_HIP(hipStreamSynchronize(h.stream));
}

}  // namespace pdhg
