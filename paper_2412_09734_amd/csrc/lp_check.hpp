// The terms of an LP check and the decisions taken on their totals, shared by
// the multi-kernel iteration (lp_kernels.hip) and the one-workgroup solve
// (lp_small.hip).
#pragma once

#include "device.hpp"

namespace pdhg {

// Column side of a check for row r of A~' given q = (A~'yhat)_r (see k_check_n).
__device__ __forceinline__ void check_n_terms(
    int32_t r, double q, const double *__restrict__ xhat, const double *__restrict__ x,
    const double *__restrict__ x0, const double *__restrict__ aty, const double *__restrict__ Dc,
    const double *__restrict__ c_o, const double *__restrict__ lv_o, const double *__restrict__ uv_o,
    const double *__restrict__ q0, double *__restrict__ qhat, double (&v)[6], double (&rsum)[2],
    double (&rmax)[2]) {
    const double xh = xhat[r];
    const double dx = xh - x[r];
    v[0] = dx * dx;
    v[1] = (q - aty[r]) * dx;
    const double d0 = xh - x0[r];
    v[2] = d0 * d0;
    const double d = Dc[r];
    const double xo = d * xh;
    const double g = c_o[r] - q / d;
    const double lo = lv_o[r], hi = uv_o[r];
    const bool lf = isfinite(lo), uf = isfinite(hi);
    const double lam = (!lf && !uf) ? 0.0 : (lf && !uf) ? fmax(g, 0.0) : (!lf && uf) ? fmin(g, 0.0) : g;
    const double rd = g - lam;
    v[3] = rd * rd;
    v[4] = c_o[r] * xo;
    v[5] = (lf ? lo * fmax(lam, 0.0) : 0.0) - (uf ? hi * fmax(-lam, 0.0) : 0.0);
    qhat[r] = q;
    ray_col_terms(q, q0[r], d, d0, c_o[r], lo, hi, rsum, rmax);
}

// Row side of a check for row r given p = (A~xhat)_r (see k_check_m).
__device__ __forceinline__ void check_m_terms(
    int32_t r, double p, const double *__restrict__ yhat, const double *__restrict__ y,
    const double *__restrict__ y0, const double *__restrict__ Dr, const double *__restrict__ lc_o,
    const double *__restrict__ uc_o, const double *__restrict__ p0, double *__restrict__ phat,
    double (&v)[4], double (&rsum)[1], double (&rmax)[2]) {
    const double d = Dr[r];
    const double ax = p / d;
    const double lo = lc_o[r], hi = uc_o[r];
    const double rpr = ax - clampd(ax, lo, hi);
    v[0] = rpr * rpr;
    const double yh = yhat[r];
    const double yo = d * yh;
    v[1] = (isfinite(lo) ? lo * fmax(yo, 0.0) : 0.0) - (isfinite(hi) ? hi * fmax(-yo, 0.0) : 0.0);
    const double dy = yh - y[r];
    v[2] = dy * dy;
    const double d0 = yh - y0[r];
    v[3] = d0 * d0;
    phat[r] = p;
    ray_row_terms(p, p0[r], d, d0, lo, hi, rsum, rmax);
}

// One thread: relative KKT error and fixed-point residual in the PDHG norm
// from the totals of a check, termination and restart decisions, primal-weight
// update. vn / vm: the column and row sums; rays: rs and rx hold the ray
// totals (0 dual-ray objective (columns), 1 c'dx, 2 dual-ray objective (rows);
// maxima: 0 dual-ray violation, 1 primal-ray violation).
__device__ __forceinline__ void check_decide(DevState *st, const double (&vn)[6], const double (&vm)[4],
                                             const double (&rs)[3], const double (&rx)[2], bool rays,
                                             const CtlConst &K, int32_t chunk_plain, int32_t is_last,
                                             int32_t last_status) {
    const int64_t t = st->t_next;
    const int64_t k = st->first ? 0 : st->k_base + st->plain_prev;
    const double P = vn[4];
    const double D = vm[1] + vn[5];
    const double abs_p = sqrt(vm[0]), abs_d = sqrt(vn[3]), abs_g = fabs(P - D);
    const double rel_p = abs_p / (1.0 + K.bnorm);
    const double rel_d = abs_d / (1.0 + K.cnorm);
    const double rel_g = abs_g / (1.0 + fabs(P) + fabs(D));
    double kkt = rel_p;
    if (rel_d > kkt || isnan(rel_d)) kkt = rel_d;
    if (rel_g > kkt || isnan(rel_g)) kkt = rel_g;
    st->kkt = kkt;
    st->rel_p = rel_p;
    st->rel_d = rel_d;
    st->rel_g = rel_g;
    st->pobj = P;
    st->dobj = D;
    st->abs_p = abs_p;
    st->abs_d = abs_d;
    st->abs_g = abs_g;
    st->k_check = k;
    st->t_done = t;
    st->first = 0;
    st->plain_prev = chunk_plain;
    st->t_next = t + 1 + chunk_plain;
    if (isnan(kkt)) {
        st->done = 1;
        st->status = PDHG_NUMERICAL_ERROR;
        st->action = 2;
        return;
    }
    // a polishing phase stops on its own residual alone
    const double term_val = K.term == 1 ? rel_p : K.term == 2 ? rel_d : kkt;
    if (term_val <= K.eps) {
        st->done = 1;
        st->status = PDHG_OPTIMAL;
        st->action = 2;
        return;
    }
    if (rays) {
        const double obj_d = rs[0] + rs[2], obj_p = rs[1];
        if (K.eps_pinf > 0.0 && obj_d > 0.0 && rx[0] <= K.eps_pinf * obj_d) {
            st->done = 1;
            st->status = PDHG_PRIMAL_INFEASIBLE;
            st->ray_scale = 1.0 / obj_d;
            st->action = 2;
            return;
        }
        if (K.eps_dinf > 0.0 && obj_p < 0.0 && rx[1] <= K.eps_dinf * (-obj_p)) {
            st->done = 1;
            st->status = PDHG_DUAL_INFEASIBLE;
            st->ray_scale = -1.0 / obj_p;
            st->action = 2;
            return;
        }
    }
    if (is_last) {
        st->done = 1;
        st->status = last_status;
        st->action = 2;
        return;
    }
    const double tau = st->tau, sigma = st->sigma;
    double r2 = vn[0] / tau + vm[2] / sigma + 2.0 * vn[1];
    const double r = r2 > 0.0 ? sqrt(r2) : 0.0;
    st->last_r = r;
    int restart = 0;
    if (t == 0) {
        st->r_start = r;
        st->r_prev = r;
    } else if (r <= K.beta_suff * st->r_start ||
               (r <= K.beta_nec * st->r_start && r > st->r_prev) ||
               (double)k >= K.beta_art * (double)t) {
        restart = 1;
    } else {
        st->r_prev = r;
    }
    if (restart) {
        const double dxr = sqrt(vn[2]), dyr = sqrt(vm[3]);
        double omega = st->omega;
        if (dxr > 1e-10 && dyr > 1e-10) omega = exp(0.5 * log(dyr / dxr) + 0.5 * log(omega));
        st->omega = omega;
        st->tau = K.eta / omega;
        st->sigma = K.eta * omega;
        st->r_start = r;
        st->r_prev = r;
        st->restarts += 1;
        st->k_base = 0;
        st->action = 1;
        st->anchor_valid = 1;   // k_apply stores the new anchor's products
    } else {
        st->k_base = k + 1;
        st->action = 0;
    }
}

}  // namespace pdhg
