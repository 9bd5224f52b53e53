// Shared pieces of the batched rAPDHG kernels (batch_qp.hip, batch_qp_row.hip).
#pragma once

#include "batch_internal.hpp"
#include "device.hpp"

namespace pdhg {

constexpr int kRmax = 32;   // largest supported rank of F
constexpr int kCkpt = 50;   // checkpoint spacing of the unrolled QP
constexpr int kWaveRowsMax = 256;   // row limit of the wave-per-row mode

struct QArgs {
    int32_t B, m, n, r;
    int32_t wave_rows;      // 1: each constraint row is reduced by one wave (few, long rows)
    const int32_t *arp, *aci, *trp, *tci;
    const double *ava, *tva, *Dr, *Dc;
    double eta;
    const double *FT;       // F~' [r_pad][n], r_pad = r rounded up to 8, zero rows past r
    const double *d_o;      // original d [B][n]
    double *normq;          // [B]
    const double *c_o, *lc_o, *uc_o, *lv_o, *uv_o;
    double *c, *lc, *uc, *lv, *uv, *dd;   // scaled, per instance
    double *x, *y, *xb, *yb, *x0, *y0, *xe, *v;
    const double *x_init, *y_init;
    double *x_out, *y_out;
    double *res;            // [B][12]
    int32_t *queue;
    // unrolled
    int64_t T;
    int32_t replay;
    uint8_t *restart;
    double *omega;
    int32_t *kk;
    uint64_t *xmask, *ymask;   // [B][T][words]
    double *ckpt;              // [B][nck][2n + 2m]
    double *vseg;              // [B][kCkpt][n]
    double *vall;              // [B][T][n] every momentum point, or null (recompute from checkpoints)
    const double *gx, *gy;
    double *gc, *glc, *guc, *gd;
    double *bxb, *byb, *bw, *bqv;   // reverse scratch
};

struct QOpts {
    double eps, gamma, beta_suff, beta_nec, beta_art, power_tol;
    double eps_pinf, eps_dinf;   // infeasibility certificate tolerances
    int64_t limit;
    int32_t check_every, power_max_iters;
    int32_t detect, pad;         // 1: test the rays at checks
};

template <int BT>
__device__ __forceinline__ int32_t qnext(int32_t *queue) {
    __shared__ int32_t id;
    if (threadIdx.x == 0) id = atomicAdd(queue, 1);
    __syncthreads();
    const int32_t r = id;
    __syncthreads();
    return r;
}

enum class QK { norm, solve, unrolled, backward };

// The kernels for batches with one constraint row (batch_qp_row.hip).
// qrow_fits: threads per instance they would take, or 0 where they do not apply.
int32_t qrow_fits(const BatchHandle &h);
void qrow_launch(BatchHandle &h, QK which, const QArgs &a, const QOpts &o);

}  // namespace pdhg
