// Batched r2HPDHG (MPAX paper, Section 3 "Batched solving"; Algorithm 1).
//
// One workgroup owns one LP instance at a time and runs its whole solve:
// scaling and power iteration (setup kernel), then the iteration loop with
// checks, restarts and early exit (solve kernel). Workgroups take instances
// from a queue (an integer counter) until the batch is exhausted, so a launch
// of as many workgroups as the GPU holds covers any batch size. Every
// reduction is a fixed-order workgroup tree, so an instance's result does not
// depend on which workgroup ran it.
//
// Matrices are plain CSR (rows in original order) with instance-local column
// indices; row pointers hold global entry offsets. The setup and the
// memory-resident kernels walk it, their vectors staying in L2 while the
// instance runs; the on-chip kernels read SELL-64 copies (see BArgs), keep an
// instance's vectors in registers and LDS and its entries as far as that pays
// (k_batch_solve_res: all, _lds: the first of every row, _stream: none).
#include <algorithm>
#include <climits>
#include <memory>
#include <vector>

#include "device.hpp"
#include "batch_internal.hpp"

namespace pdhg {

struct BOpts {
    double eps, gamma, step_safety, beta_suff, beta_nec, beta_art, power_tol;
    int64_t limit;
    int32_t check_every, ruiz_iters, pock_chambolle, power_max_iters;
    double eps_pinf, eps_dinf;   // infeasibility certificate tolerances
    int32_t detect, pad;         // 1: test the rays at checks
};

struct BArgs {
    int32_t B, shared, m, n;
    const int32_t *row_off, *col_off;
    const int32_t *arp, *aci;
    double *ava;
    const int32_t *trp, *tci;
    double *tva;
    double *Dr, *Dc, *eta;
    int32_t *power_iters;
    const double *c_o, *lc_o, *uc_o, *lv_o, *uv_o;
    double *c, *lc, *uc, *lv, *uv;
    double *x, *x0, *xh, *xe, *aty, *y, *y0, *yh;
    const double *x_init, *y_init;
    double *x_out, *y_out;
    BatchRes *res;
    int32_t *queue;
    // SELL-64 copies of A~ and A~' over positions: position i of an instance
    // is its row perm[i] (ragged batches: rows by falling length, so that a
    // slice's rows fill its width; null: position = row). Pair k of position
    // i, its entries 2k and 2k + 1, is at 64 (sp[sfirst + i/64] + k) + i%64:
    // the two positions gathered, as byte offsets 8 j in the halves of sci,
    // and the two values; past a row's end they are (0, 0.0).
    const int32_t *asp, *asfirst, *aperm, *tsp, *tsfirst, *tperm;
    const uint32_t *asci, *tsci;
    const double2 *asva, *tsva;
    double *lhist;    // Lanczos alpha / beta per instance, stride 2 (power_max_iters + 1)
    // infeasibility rays: the anchor's products A~x0 (like y), A~'y0 (like x)
    // and this check's A~xhat, A~'yhat
    double *p0, *q0, *ph, *qh;
};

// Geometry of instance b: matrix rows start at r0 (A) / c0 (A'); vectors at
// vr / vc; scaling vectors at dr / dc.
struct Geo {
    int32_t m, n, r0, c0, vr, vc, dr, dc, sidx;
};

__device__ __forceinline__ Geo geometry(const BArgs &a, int32_t b) {
    Geo g;
    if (a.shared) {
        g.m = a.m;
        g.n = a.n;
        g.r0 = 0;
        g.c0 = 0;
        g.vr = b * a.m;
        g.vc = b * a.n;
        g.dr = 0;
        g.dc = 0;
        g.sidx = 0;
    } else {
        g.r0 = a.row_off[b];
        g.c0 = a.col_off[b];
        g.m = a.row_off[b + 1] - g.r0;
        g.n = a.col_off[b + 1] - g.c0;
        g.vr = g.r0;
        g.vc = g.c0;
        g.dr = g.r0;
        g.dc = g.c0;
        g.sidx = b;
    }
    return g;
}

// Deterministic workgroup sum of K values per thread, result in every thread:
// wave butterflies, then thread q adds the wave totals of value q in wave
// order (one value per thread keeps the register footprint independent of
// the workgroup size).
template <int BT, int K>
__device__ __forceinline__ void wg_sum(double (&v)[K]) {
    constexpr int NW = BT / 64;
    __shared__ double sh[K][NW];
    __shared__ double tot[K];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const double s = wave_sum(v[q]);
        if (lane == 0) sh[q][wave] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < K) {
        double s = 0.0;
        for (int w = 0; w < NW; ++w) s += sh[threadIdx.x][w];
        tot[threadIdx.x] = s;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K; ++q) v[q] = tot[q];
    __syncthreads();
}

// Workgroup maxima of K values (order-free), result in every thread.
template <int BT, int K>
__device__ __forceinline__ void wg_max(double (&v)[K]) {
    constexpr int NW = BT / 64;
    __shared__ double sh[K][NW];
    __shared__ double tot[K];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const double s = wave_max(v[q]);
        if (lane == 0) sh[q][wave] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < K) {
        double s = sh[threadIdx.x][0];
        for (int w = 1; w < NW; ++w) s = fmax(s, sh[threadIdx.x][w]);
        tot[threadIdx.x] = s;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K; ++q) v[q] = tot[q];
    __syncthreads();
}

template <int BT>
__device__ __forceinline__ int32_t next_instance(int32_t *queue) {
    __shared__ int32_t id;
    if (threadIdx.x == 0) id = atomicAdd(queue, 1);
    __syncthreads();
    // the same value in every lane: a scalar, so the instance's pointers and
    // sizes live in scalar registers
    const int32_t r = __builtin_amdgcn_readfirstlane(id);
    __syncthreads();
    return r;
}

// CSR row dot product, entries added in row order; four entries' loads (and
// then their gathers) are issued before their products, so a thread's walk
// over the row waits on a quarter as many round trips.
__device__ __forceinline__ double csr_dot(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                          const double *__restrict__ va, int32_t row,
                                          const double *__restrict__ v) {
    double acc = 0.0;
    int32_t e = rp[row];
    const int32_t e1 = rp[row + 1];
    for (; e + 4 <= e1; e += 4) {
        int32_t c[4];
        double a[4], x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = ci[e + q];
            a[q] = va[e + q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = v[c[q]];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = fma(a[q], x[q], acc);
    }
    for (; e < e1; ++e) acc = fma(va[e], v[ci[e]], acc);
    return acc;
}

// Ruiz / Pock-Chambolle factor of one CSR row: max |a| (pc = false) or the sum
// of |a| (pc = true) over the row in entry order, loads four at a time.
__device__ __forceinline__ double csr_absnorm(const int32_t *__restrict__ rp, const double *__restrict__ va,
                                              int32_t row, bool pc) {
    double acc = 0.0;
    int32_t e = rp[row];
    const int32_t e1 = rp[row + 1];
    for (; e + 4 <= e1; e += 4) {
        double a[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = fabs(va[e + q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = pc ? acc + a[q] : fmax(acc, a[q]);
    }
    for (; e < e1; ++e) acc = pc ? acc + fabs(va[e]) : fmax(acc, fabs(va[e]));
    return acc;
}

// va[e] /= (r * f[ci[e]]) over CSR row `row`, four entries at a time.
__device__ __forceinline__ void csr_rescale(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                            double *__restrict__ va, int32_t row, double r,
                                            const double *__restrict__ f) {
    int32_t e = rp[row];
    const int32_t e1 = rp[row + 1];
    for (; e + 4 <= e1; e += 4) {
        int32_t c[4];
        double a[4], x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = ci[e + q];
            a[q] = va[e + q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = f[c[q]];
#pragma unroll
        for (int q = 0; q < 4; ++q) va[e + q] = a[q] / (r * x[q]);
    }
    for (; e < e1; ++e) va[e] = va[e] / (r * f[ci[e]]);
}

// The two gathers of one pair of SELL-64 entries, added in row order.
template <class V>
__device__ __forceinline__ double sell_pair(uint32_t c, double2 a, const V *v, double acc) {
    acc = fma(a.x, v[(c & 0xffffu) >> 3], acc);
    return fma(a.y, v[c >> 19], acc);
}

// Row sum of a SELL-64 slice row: lane `lane` of slice `sl`; entries walked in
// row order, two pairs' loads in flight.
__device__ __forceinline__ double sell_dot(const int32_t *__restrict__ sp, const uint32_t *__restrict__ ci,
                                           const double2 *__restrict__ va, int32_t sl, int32_t lane,
                                           const double *__restrict__ v) {
    const int32_t k1 = sp[sl + 1];
    int32_t k = sp[sl];
    double acc = 0.0;
    for (; k + 2 <= k1; k += 2) {
        const int32_t e = 64 * k + lane;
        const uint32_t c0 = ci[e], c1 = ci[e + 64];
        const double2 a0 = va[e], a1 = va[e + 64];
        acc = sell_pair(c0, a0, v, acc);
        acc = sell_pair(c1, a1, v, acc);
    }
    if (k < k1) acc = sell_pair(ci[64 * k + lane], va[64 * k + lane], v, acc);
    return acc;
}

// The same with four pairs' loads in flight, the last ones in groups of two and
// one, for the reverse pass: 256 instances of 60 x 120 4.68 -> 4.46 us an iteration,
// 256 of up to 250 x 500 9.1 -> 7.8. In the forward pass it fills the 128 registers of
// 1,024 threads and costs 12%.
__device__ __forceinline__ double sell_dot4(const int32_t *__restrict__ sp, const uint32_t *__restrict__ ci,
                                            const double2 *__restrict__ va, int32_t sl, int32_t lane,
                                            const double *__restrict__ v) {
    const int32_t k0 = sp[sl];
    int32_t w = sp[sl + 1] - k0, e = 64 * k0 + lane;
    double acc = 0.0;
    auto pairs = [&](auto width) {
        constexpr int U = decltype(width)::value;
        uint32_t c[U];
        double2 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = ci[e + 64 * u];
            a[u] = va[e + 64 * u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc = sell_pair(c[u], a[u], v, acc);
        e += 64 * U;
    };
    for (; w >= 4; w -= 4) pairs(std::integral_constant<int, 4>());
    if (w & 2) pairs(std::integral_constant<int, 2>());
    if (w & 1) pairs(std::integral_constant<int, 1>());
    return acc;
}

// The row (column) at position i of an instance whose permutation starts at p.
__device__ __forceinline__ int32_t row_at(const int32_t *p, int32_t off, int32_t i) { return p ? p[off + i] : i; }

__device__ __forceinline__ uint64_t splitmix64_b(uint64_t x) {
    uint64_t z = x + 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// ---------------------------------------------------------------------------
// setup: Ruiz + Pock-Chambolle scaling and the power iteration, per instance
// (once for a shared matrix).

// T = B'B for the Golub-Kahan bidiagonal B (alpha on the diagonal, beta above
// it): diagonal d_i = alpha_i^2 + beta_{i-1}^2, squared off-diagonal e_i =
// (alpha_i beta_i)^2. The first kTriLds of them are kept in LDS.
constexpr int kTriLds = 256;
struct Tridiag {
    const double *alpha, *beta;   // all of them (memory)
    const double *d, *e;          // the first kTriLds (LDS)
    __device__ __forceinline__ double diag(int32_t i) const {
        if (i < kTriLds) return d[i];
        return alpha[i] * alpha[i] + beta[i - 1] * beta[i - 1];
    }
    __device__ __forceinline__ double off2(int32_t i) const {
        if (i < kTriLds) return e[i];
        const double o = alpha[i] * beta[i];
        return o * o;
    }
};

// Whether every eigenvalue of the leading k x k block lies below x: the leading
// minors s_i of x I - T are positive, s_i = (x - d_i) s_{i-1} - e_{i-1} s_{i-2}.
// Scaled by a power of two (sc, with sc T of norm about 1), and rescaled every
// eight steps, so that nothing overflows; two dependent operations a step where
// the ratio recurrence has a division.
__device__ __forceinline__ bool tridiag_below(const Tridiag &T, int32_t k, double x, double sc) {
    const double xs = x * sc, sc2 = sc * sc;
    double sp = 0.0, s = 1.0, e = 0.0;
    for (int32_t i0 = 0; i0 < k; i0 += 8) {
        const int32_t i1 = min(k, i0 + 8);
        for (int32_t i = i0; i < i1; ++i) {
            const double a = xs - T.diag(i) * sc;
            const double t = fma(a, s, -(e * sp));
            sp = s;
            s = t;
            e = T.off2(i) * sc2;
            if (!(s > 0.0)) return false;
        }
        const int ex = -__builtin_amdgcn_frexp_exp(s);
        s = ldexp(s, ex);
        sp = ldexp(sp, ex);
    }
    return true;
}

// Largest eigenvalue of the leading k x k block by one wave: the smallest
// double above all eigenvalues, found by 64 tests at a time. lower: a value not
// above it (the eigenvalue of a smaller block, or 0). The first tests are spaced
// by powers of two from lower on: close to convergence the eigenvalue moves by
// 1e-7 of itself, which leaves some 30 bits to find instead of 52.
__device__ double tridiag_lambda_max(const Tridiag &T, int32_t k, double lower) {
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    double g = 0.0;   // Gershgorin bound
    for (int32_t i = lane; i < k; i += 64) {
        const double el = i > 0 ? sqrt(T.off2(i - 1)) : 0.0;
        const double er = i + 1 < k ? sqrt(T.off2(i)) : 0.0;
        g = fmax(g, T.diag(i) + el + er);
    }
    g = wave_max(g);
    if (!(g > 0.0)) return 0.0;
    const double sc = ldexp(1.0, -__builtin_amdgcn_frexp_exp(g));
    double lo = lower * (1.0 - 1e-12), hi = g * (1.0 + 1e-14);
    // spaced tests, the first at lo itself
    double x = lane == 0 ? lo : fmin(hi, lo + lo * ldexp(1.0, lane - 60));
    uint64_t below = __ballot(x > 0.0 && tridiag_below(T, k, x, sc));
    if (below & 1ull) {
        lo = 0.0;
    } else if (below) {
        const int f = __ffsll((unsigned long long)below) - 1;
        hi = lane_value(x, f);
        lo = lane_value(x, f - 1);
    } else if (lo > 0.0) {
        lo = lane_value(x, 63);
    }
    for (int round = 0; round < 40; ++round) {
        const double mid = 0.5 * (lo + hi);
        if (!(mid > lo && mid < hi)) break;
        x = fmax(lo, fmin(hi, lo + (hi - lo) * ((double)(lane + 1) * (1.0 / 64.0))));
        if (lane == 63) x = hi;
        if (lane == 31) x = mid;   // strictly inside, so the interval always shrinks
        below = __ballot(x >= hi || (x > lo && tridiag_below(T, k, x, sc)));
        const int f = __ffsll((unsigned long long)below) - 1;   // lane 63 is always set
        const double nlo = f > 0 ? lane_value(x, f - 1) : lo;
        hi = lane_value(x, f);
        lo = fmax(lo, nlo);
    }
    return hi;
}

// ONCHIP: the power iteration's gathered vectors v (n) and w (m) live in LDS.
// The eigenvalue searches of the norm estimate were 50 of the 75 us of each of
// its steps on a 32 x 32 grid (a workgroup-wide bisection with a division per
// pivot, six rounds a step); as eight waves' searches of eight steps at a time
// the setup of that batch takes 1.26 instead of 5.58 ms.
template <int BT, bool ONCHIP>
__global__ __launch_bounds__(BT) void k_batch_setup(BArgs a, BOpts o, int32_t count, int32_t nmax) {
    extern __shared__ double lds[];
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= count) return;
        const Geo g = geometry(a, b);
        const int32_t *arp = a.arp + g.r0, *trp = a.trp + g.c0;
        double *Dr = a.Dr + g.dr, *Dc = a.Dc + g.dc;
        double *rs = a.yh + g.vr, *cs = a.xh + g.vc;   // factor scratch
        for (int32_t i = threadIdx.x; i < g.m; i += BT) Dr[i] = 1.0;
        for (int32_t j = threadIdx.x; j < g.n; j += BT) Dc[j] = 1.0;
        const int passes = o.ruiz_iters + (o.pock_chambolle ? 1 : 0);
        for (int pass = 0; pass < passes; ++pass) {
            const bool pc = pass >= o.ruiz_iters;
            __syncthreads();
            for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                const double acc = csr_absnorm(arp, a.ava, i, pc);
                rs[i] = acc > 0.0 ? sqrt(acc) : 1.0;
            }
            for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                const double acc = csr_absnorm(trp, a.tva, j, pc);
                cs[j] = acc > 0.0 ? sqrt(acc) : 1.0;
            }
            __syncthreads();
            for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                Dr[i] = Dr[i] / rs[i];
                csr_rescale(arp, a.aci, a.ava, i, rs[i], cs);
            }
            for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                Dc[j] = Dc[j] / cs[j];
                csr_rescale(trp, a.tci, a.tva, j, cs[j], rs);
            }
        }
        __syncthreads();
        // ||A~||_2 by Golub-Kahan-Lanczos bidiagonalisation from the SplitMix64
        // start vector (see estimate_steps for the recurrences)
        int64_t nnz = (int64_t)arp[g.m] - arp[0];
        double lam = 0.0;
        int32_t it = 0;
        if (g.m > 0 && nnz > 0) {
            double *v = ONCHIP ? lds : a.xh + g.vc;          // gathered by rows
            double *u = ONCHIP ? lds + nmax : a.yh + g.vr;   // gathered by columns
            double *pr = a.y + g.vr, *qc = a.xe + g.vc;      // owner-only scratch
            double *al = a.lhist + (size_t)g.sidx * 2 * (o.power_max_iters + 1);
            double *be = al + (o.power_max_iters + 1);
            // eigenvalues are wanted at every step, but only to find the step to
            // stop at: each wave finds the one of a step of its own, kLag steps
            // at a time, and what the steps past the stop computed is dropped
            constexpr int kLag = BT / 64 < 8 ? BT / 64 : 8;
            __shared__ double tri_d[kTriLds], tri_e[kTriLds];
            __shared__ double lam_sh[kLag];
            const Tridiag T{al, be, tri_d, tri_e};
            double q0[1] = {0.0};
            for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                const double val = 0.5 + (double)(splitmix64_b((uint64_t)j) >> 11) * 0x1.0p-53;
                v[j] = val;
                q0[0] += val * val;
            }
            for (int32_t i = threadIdx.x; i < g.m; i += BT) u[i] = 0.0;
            wg_sum<BT, 1>(q0);
            const double nv = sqrt(q0[0]);
            for (int32_t j = threadIdx.x; j < g.n; j += BT) v[j] = v[j] / nv;
            __syncthreads();
            double lam_prev = 0.0, bprev = 0.0;
            int32_t done = 0;       // steps whose eigenvalue is known
            // eigenvalues of steps done + 1 .. last; the step that stops, or 0
            auto settle = [&](int32_t last, bool beta_zero) -> int32_t {
                const int32_t wave = (int32_t)(threadIdx.x >> 6), k = done + 1 + wave;
                __syncthreads();
                if (wave < kLag && k <= last) {
                    const double l = tridiag_lambda_max(T, k, lam_prev);
                    if ((threadIdx.x & 63) == 0) lam_sh[wave] = l;
                }
                __syncthreads();
                int32_t at = 0;
                for (int32_t k2 = done + 1; k2 <= last && !at; ++k2) {
                    lam = lam_sh[k2 - done - 1];
                    if ((k2 == last && beta_zero) || (k2 > 1 && fabs(lam - lam_prev) <= o.power_tol * lam)) at = k2;
                    else lam_prev = lam;
                }
                done = last;
                __syncthreads();
                return at;
            };
            for (it = 1; it <= o.power_max_iters; ++it) {
                double sp[1] = {0.0};
                for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                    const double pv = csr_dot(arp, a.aci, a.ava, i, v) - bprev * u[i];
                    pr[i] = pv;
                    sp[0] += pv * pv;
                }
                wg_sum<BT, 1>(sp);
                const double al_k = sqrt(sp[0]);
                if (!(al_k > 0.0)) {
                    // the Krylov space closes; the block still gains the row of the
                    // last beta, the whole norm where A~ has one row
                    if (it == 1) break;
                    if (threadIdx.x == 0) {
                        al[it - 1] = be[it - 1] = 0.0;
                        if (it <= kTriLds) {
                            tri_d[it - 1] = bprev * bprev;
                            tri_e[it - 1] = 0.0;
                        }
                    }
                    it = settle(it, true);
                    break;
                }
                for (int32_t i = threadIdx.x; i < g.m; i += BT) u[i] = pr[i] / al_k;
                __syncthreads();
                double sq[1] = {0.0};
                for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                    const double qv = csr_dot(trp, a.tci, a.tva, j, u) - al_k * v[j];
                    qc[j] = qv;
                    sq[0] += qv * qv;
                }
                wg_sum<BT, 1>(sq);
                const double be_k = sqrt(sq[0]);
                if (threadIdx.x == 0) {
                    al[it - 1] = al_k;
                    be[it - 1] = be_k;
                    if (it <= kTriLds) {
                        tri_d[it - 1] = al_k * al_k + bprev * bprev;
                        const double off = al_k * be_k;
                        tri_e[it - 1] = off * off;
                    }
                }
                const bool beta_zero = !(be_k > 0.0);
                if (beta_zero || it - done == kLag || it == o.power_max_iters) {
                    const int32_t at = settle(it, beta_zero);
                    if (at) {
                        it = at;
                        break;
                    }
                }
                for (int32_t j = threadIdx.x; j < g.n; j += BT) v[j] = qc[j] / be_k;
                bprev = be_k;
                __syncthreads();
            }
            if (it > o.power_max_iters) it = o.power_max_iters;
        }
        if (threadIdx.x == 0) {
            const double na = sqrt(lam);
            a.eta[g.sidx] = na > 0.0 ? o.step_safety / na : 1.0;
            a.power_iters[g.sidx] = it;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// solve

// Infeasibility rays of instance g at a check (after its products were kept
// in qh / ph): sums rs = (dual-ray bound terms over the columns, c'dx,
// dual-ray bound terms over the rows) and maxima rm = (dual-ray violation,
// primal-ray violation), every thread receiving the totals, for the
// memory-resident k_batch_solve (a pass of its own there; x0 is read from
// memory). The on-chip kernels sum the same terms inside their check loops.
template <int BT>
__device__ __forceinline__ void batch_ray_pass(const BArgs &a, const Geo &g,
                                            const double *__restrict__ xh, const double *__restrict__ yh,
                                            const double *__restrict__ y0, double (&rs)[3], double (&rm)[2]) {
    const double *Dr = a.Dr + g.dr, *Dc = a.Dc + g.dc;
    const double *x0 = a.x0 + g.vc;
    double s[3] = {0.0, 0.0, 0.0}, mx[2] = {0.0, 0.0};
    // opaque thread index: the addresses below are formed here, not kept
    // live across the iteration loop the pass sits in
    int32_t t0 = (int32_t)threadIdx.x;
    asm volatile("" : "+v"(t0));
#pragma unroll 1
    for (int32_t j = t0; j < g.n; j += BT) {
        double s2[2], m2[2];
        ray_col_terms(a.qh[g.vc + j], a.q0[g.vc + j], Dc[j], xh[j] - x0[j], a.c_o[g.vc + j],
                      a.lv_o[g.vc + j], a.uv_o[g.vc + j], s2, m2);
        s[0] += s2[0];
        s[1] += s2[1];
        mx[0] = fmax(mx[0], m2[0]);
        mx[1] = fmax(mx[1], m2[1]);
    }
#pragma unroll 1
    for (int32_t i = t0; i < g.m; i += BT) {
        double s1[1], m2[2];
        ray_row_terms(a.ph[g.vr + i], a.p0[g.vr + i], Dr[i], yh[i] - y0[i], a.lc_o[g.vr + i],
                      a.uc_o[g.vr + i], s1, m2);
        s[2] += s1[0];
        mx[0] = fmax(mx[0], m2[0]);
        mx[1] = fmax(mx[1], m2[1]);
    }
    wg_sum<BT, 3>(s);
    wg_max<BT, 2>(mx);
    for (int q = 0; q < 3; ++q) rs[q] = s[q];
    rm[0] = mx[0];
    rm[1] = mx[1];
}

// RAYS: the checks also test infeasibility rays (a separate instantiation,
// so that solves without the test keep the leaner register budget).
template <int BT, bool RAYS>
__global__ __launch_bounds__(BT) void k_batch_solve(BArgs a, BOpts o) {
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= a.B) return;
        const Geo g = geometry(a, b);
        const int32_t *arp = a.arp + g.r0, *trp = a.trp + g.c0;
        const int32_t *aci = a.aci, *tci = a.tci;
        const double *ava = a.ava, *tva = a.tva;
        const double *Dr = a.Dr + g.dr, *Dc = a.Dc + g.dc;
        const double *c_o = a.c_o + g.vc, *lv_o = a.lv_o + g.vc, *uv_o = a.uv_o + g.vc;
        const double *lc_o = a.lc_o + g.vr, *uc_o = a.uc_o + g.vr;
        double *c = a.c + g.vc, *lv = a.lv + g.vc, *uv = a.uv + g.vc;
        double *lc = a.lc + g.vr, *uc = a.uc + g.vr;
        double *x = a.x + g.vc, *x0 = a.x0 + g.vc, *xh = a.xh + g.vc, *xe = a.xe + g.vc;
        double *aty = a.aty + g.vc;
        double *y = a.y + g.vr, *y0 = a.y0 + g.vr, *yh = a.yh + g.vr;
        const double eta = a.eta[g.sidx];
        const double gam = o.gamma;

        // scaled data, norms, initial point
        double nrm[4] = {0.0, 0.0, 0.0, 0.0};
        for (int32_t j = threadIdx.x; j < g.n; j += BT) {
            const double d = Dc[j];
            const double cj = d * c_o[j];
            c[j] = cj;
            lv[j] = lv_o[j] / d;
            uv[j] = uv_o[j] / d;
            nrm[0] += cj * cj;
            nrm[2] += c_o[j] * c_o[j];
        }
        for (int32_t i = threadIdx.x; i < g.m; i += BT) {
            const double d = Dr[i];
            const double l = d * lc_o[i], u = d * uc_o[i];
            lc[i] = l;
            uc[i] = u;
            double bb = 0.0, bo = 0.0;
            if (isfinite(l)) bb = fmax(bb, fabs(l));
            if (isfinite(u)) bb = fmax(bb, fabs(u));
            if (isfinite(lc_o[i])) bo = fmax(bo, fabs(lc_o[i]));
            if (isfinite(uc_o[i])) bo = fmax(bo, fabs(uc_o[i]));
            nrm[1] += bb * bb;
            nrm[3] += bo * bo;
        }
        wg_sum<BT, 4>(nrm);
        const double cn = sqrt(nrm[0]), bn = sqrt(nrm[1]);
        const double cnorm = sqrt(nrm[2]), bnorm = sqrt(nrm[3]);
        double omega = (cn > 1e-10 && bn > 1e-10) ? cn / bn : 1.0;
        double tau = eta / omega, sigma = eta * omega;
        for (int32_t j = threadIdx.x; j < g.n; j += BT) {
            const double v0 = a.x_init ? a.x_init[g.vc + j] / Dc[j] : 0.0;
            const double xv = clampd(v0, lv[j], uv[j]);
            x[j] = xv;
            x0[j] = xv;
        }
        for (int32_t i = threadIdx.x; i < g.m; i += BT) {
            const double v0 = a.y_init ? a.y_init[g.vr + i] / Dr[i] : 0.0;
            const double lo = isfinite(uc[i]) ? -INFINITY : 0.0;
            const double hi = isfinite(lc[i]) ? INFINITY : 0.0;
            const double yv = clampd(v0, lo, hi);
            y[i] = yv;
            y0[i] = yv;
        }
        __syncthreads();

        int64_t t = 0, k = 0, restarts = 0;
        double r_start = 0.0, r_prev = 0.0;
        int32_t status = 0;
        bool anchor_valid = false;   // the anchor's products are stored (after a restart)
        double ray_scale = 0.0;
        double kkt = 0.0, rel_p = 0.0, rel_d = 0.0, rel_g = 0.0, P = 0.0, D = 0.0;
        for (;;) {
            const bool check = (t % o.check_every) == 0;
            const bool last = t + 1 >= o.limit;
            const bool keep = check || last;
            const double ak = (double)(k + 1) / (double)(k + 2), bk = 1.0 / (double)(k + 2);
            // primal step over the rows of A'
            for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                const double s = csr_dot(trp, tci, tva, j, y);
                const double xr = x[j];
                const double xhat = clampd(xr - tau * (c[j] - s), lv[j], uv[j]);
                xe[j] = 2.0 * xhat - xr;
                if (keep) {
                    xh[j] = xhat;
                    aty[j] = s;
                } else {
                    x[j] = ak * ((1.0 + gam) * xhat - gam * xr) + bk * x0[j];
                }
            }
            __syncthreads();
            // dual step over the rows of A
            for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                const double av = csr_dot(arp, aci, ava, i, xe);
                const double yr = y[i];
                const double yhat = dual_prox(yr, av, sigma, lc[i], uc[i]);
                if (keep)
                    yh[i] = yhat;
                else
                    y[i] = ak * ((1.0 + gam) * yhat - gam * yr) + bk * y0[i];
            }
            __syncthreads();
            if (!keep) {
                ++k;
                ++t;
                continue;
            }
            // check: KKT in the original space and the fixed-point residual
            double v[10];
#pragma unroll
            for (int q = 0; q < 10; ++q) v[q] = 0.0;
            for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                const double q = csr_dot(trp, tci, tva, j, yh);
                const double xhv = xh[j];
                const double dx = xhv - x[j];
                v[0] += dx * dx;
                v[1] += (q - aty[j]) * dx;
                const double d0 = xhv - x0[j];
                v[2] += d0 * d0;
                const double d = Dc[j];
                const double gr = c_o[j] - q / d;
                const double lo = lv_o[j], hi = uv_o[j];
                const bool lf = isfinite(lo), uf = isfinite(hi);
                const double lam = (!lf && !uf) ? 0.0 : (lf && !uf) ? fmax(gr, 0.0) : (!lf && uf) ? fmin(gr, 0.0) : gr;
                const double rd = gr - lam;
                v[3] += rd * rd;
                v[4] += c_o[j] * (d * xhv);
                v[5] += (lf ? lo * fmax(lam, 0.0) : 0.0) - (uf ? hi * fmax(-lam, 0.0) : 0.0);
                if (RAYS) a.qh[g.vc + j] = q;
            }
            for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                const double p = csr_dot(arp, aci, ava, i, xh);
                const double d = Dr[i];
                const double ax = p / d;
                const double lo = lc_o[i], hi = uc_o[i];
                const double rpr = ax - clampd(ax, lo, hi);
                v[6] += rpr * rpr;
                const double yhv = yh[i];
                const double yo = d * yhv;
                v[7] += (isfinite(lo) ? lo * fmax(yo, 0.0) : 0.0) - (isfinite(hi) ? hi * fmax(-yo, 0.0) : 0.0);
                const double dy = yhv - y[i];
                v[8] += dy * dy;
                const double d0 = yhv - y0[i];
                v[9] += d0 * d0;
                if (RAYS) a.ph[g.vr + i] = p;
            }
            wg_sum<BT, 10>(v);
            P = v[4];
            D = v[7] + v[5];
            rel_p = sqrt(v[6]) / (1.0 + bnorm);
            rel_d = sqrt(v[3]) / (1.0 + cnorm);
            rel_g = fabs(P - D) / (1.0 + fabs(P) + fabs(D));
            kkt = rel_p;
            if (rel_d > kkt || isnan(rel_d)) kkt = rel_d;
            if (rel_g > kkt || isnan(rel_g)) kkt = rel_g;
            if (isnan(kkt)) {
                status = PDHG_NUMERICAL_ERROR;
                break;
            }
            if (kkt <= o.eps) {
                status = PDHG_OPTIMAL;
                break;
            }
            if (RAYS && anchor_valid) {
                double rs[3], rm[2];
                batch_ray_pass<BT>(a, g, xh, yh, y0, rs, rm);
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
            if (last) {
                status = PDHG_ITERATION_LIMIT;
                break;
            }
            const double r2 = v[0] / tau + v[8] / sigma + 2.0 * v[1];
            const double r = r2 > 0.0 ? sqrt(r2) : 0.0;
            bool restart = false;
            if (t == 0) {
                r_start = r;
                r_prev = r;
            } else if (r <= o.beta_suff * r_start || (r <= o.beta_nec * r_start && r > r_prev) ||
                       (double)k >= o.beta_art * (double)t) {
                restart = true;
            } else {
                r_prev = r;
            }
            if (restart) {
                const double dxr = sqrt(v[2]), dyr = sqrt(v[9]);
                omega = batch_new_omega(omega, dxr, dyr);
                tau = eta / omega;
                sigma = eta * omega;
                for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                    x[j] = xh[j];
                    x0[j] = xh[j];
                }
                for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                    y[i] = yh[i];
                    y0[i] = yh[i];
                }
                if (RAYS) {   // the new anchor's products, from this check
                    int32_t t0 = (int32_t)threadIdx.x;
                    asm volatile("" : "+v"(t0));
                    for (int32_t j = t0; j < g.n; j += BT) a.q0[g.vc + j] = a.qh[g.vc + j];
                    for (int32_t i = t0; i < g.m; i += BT) a.p0[g.vr + i] = a.ph[g.vr + i];
                    anchor_valid = true;
                }
                k = 0;
                r_start = r;
                r_prev = r;
                ++restarts;
            } else {
                for (int32_t j = threadIdx.x; j < g.n; j += BT)
                    x[j] = ak * ((1.0 + gam) * xh[j] - gam * x[j]) + bk * x0[j];
                for (int32_t i = threadIdx.x; i < g.m; i += BT)
                    y[i] = ak * ((1.0 + gam) * yh[i] - gam * y[i]) + bk * y0[i];
                ++k;
            }
            ++t;
            __syncthreads();
        }
        // original-space output of the last PDHG point, or the certifying ray
        const bool xray = status == PDHG_DUAL_INFEASIBLE, yray = status == PDHG_PRIMAL_INFEASIBLE;
        for (int32_t j = threadIdx.x; j < g.n; j += BT)
            a.x_out[g.vc + j] = Dc[j] * (xray ? (xh[j] - x0[j]) * ray_scale : xh[j]);
        for (int32_t i = threadIdx.x; i < g.m; i += BT)
            a.y_out[g.vr + i] = Dr[i] * (yray ? (yh[i] - y0[i]) * ray_scale : yh[i]);
        if (threadIdx.x == 0) {
            BatchRes r;
            r.pobj = P;
            r.dobj = D;
            r.rel_p = rel_p;
            r.rel_d = rel_d;
            r.rel_g = rel_g;
            r.kkt = kkt;
            r.omega = omega;
            r.eta = eta;
            r.iterations = t + 1;
            r.restarts = restarts;
            r.status = status;
            r.power_iters = a.power_iters[g.sidx];
            a.res[b] = r;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// solve with a register-resident matrix

// Entries per column slice and per row slice of the register-resident matrix
// (node-arc incidence matrices: two entries per column, node degree <= 8).
constexpr int kResCol = 2, kResRow = 8;


// LDS of k_batch_solve_res, in doubles: y and y0 of the owned rows and x_ext
// and x0 of the owned columns (whole slots, so slots past the end need no
// test; one pad double after every 32 columns, see res_pos), and the momentum
// factors of kResSteps iterations.
constexpr int kResSteps = 64;

// An element of the LDS: kept as the 32-bit address itself, a gather is one
// instruction without address arithmetic.
typedef __attribute__((address_space(3))) double LdsDouble;

// clampd without the two instructions that fmin / fmax spend on quieting a
// signalling NaN among loaded bounds (none reaches here: bounds are results
// of products and quotients).
__device__ __forceinline__ double clamp_quiet(double v, double lo, double hi) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(v), "v"(lo));
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(r), "v"(hi));
    return r;
}

// LDS element of column j. A row's entries are often a fixed stride apart
// from the next row's (4 for the out-arcs of grid nodes), which would put a
// wave's gathers on a few banks; the pad shifts every 32 columns by one.
__host__ __device__ constexpr int32_t res_pos(int32_t j) { return j + (j >> 5); }

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ double uniform_value(double v) { return lane_value(v, 0); }

template <int BT, int S>
struct ResLds {
    static constexpr int SR = S >= 4 ? S / 4 : 1;   // row slots per thread
    static constexpr int32_t y0 = SR * BT;
    static constexpr int32_t x = 2 * SR * BT;
    static constexpr int32_t x0 = x + S * res_pos(BT);
    static constexpr int32_t aty = x0 + S * res_pos(BT);   // A~'y of the iteration before a check
    static constexpr int32_t step = aty + S * BT;
    static constexpr size_t bytes = ((size_t)step + 4 * kResSteps) * sizeof(double);
};

// Entries of the columns and rows that a thread owns, each index turned into
// the LDS address of what it gathers.
template <int BT, int S>
struct ResEntries {
    static constexpr int SR = ResLds<BT, S>::SR;
    const LdsDouble *tci[S][kResCol], *rci[SR][kResRow];
    double tva[S][kResCol], rva[SR][kResRow];

    __device__ __forceinline__ void load_col(const BArgs &a, const Geo &g, const LdsDouble *sy, int q, int32_t j) {
        int32_t e0 = 0, w = 0;
        if (j < g.n) {
            e0 = a.tsp[j >> 6];
            w = a.tsp[(j >> 6) + 1] - e0;
        }
#pragma unroll
        for (int u = 0; u < kResCol / 2; ++u) {
            const bool in = u < w;
            const int32_t e = 64 * (e0 + u) + (j & 63);
            const uint32_t c = in ? a.tsci[e] : 0;
            const double2 v = in ? a.tsva[e] : double2{0.0, 0.0};
            tci[q][2 * u] = sy + ((c & 0xffffu) >> 3);
            tci[q][2 * u + 1] = sy + (c >> 19);
            tva[q][2 * u] = v.x;
            tva[q][2 * u + 1] = v.y;
        }
    }
    __device__ __forceinline__ void load_rows(const BArgs &a, const Geo &g, const LdsDouble *sx) {
        int32_t t0 = (int32_t)threadIdx.x;
        asm volatile("" : "+v"(t0));   // addresses are formed here, not kept over a loop
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = t0 + q * BT;
            int32_t e0 = 0, w = 0;
            if (i < g.m) {
                e0 = a.asp[i >> 6];
                w = a.asp[(i >> 6) + 1] - e0;
            }
#pragma unroll
            for (int u = 0; u < kResRow / 2; ++u) {
                const bool in = u < w;
                const int32_t e = 64 * (e0 + u) + (i & 63);
                const uint32_t c = in ? a.asci[e] : 0;
                const double2 v = in ? a.asva[e] : double2{0.0, 0.0};
                rci[q][2 * u] = sx + res_pos((c & 0xffffu) >> 3);
                rci[q][2 * u + 1] = sx + res_pos(c >> 19);
                rva[q][2 * u] = v.x;
                rva[q][2 * u + 1] = v.y;
            }
        }
    }
    // one product with the vector `off` elements after the gathered one
    __device__ __forceinline__ double col(int q, int off) const {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < kResCol; ++u) s = fma(tva[q][u], tci[q][u][off], s);
        return s;
    }
    __device__ __forceinline__ double row(int q, int off) const {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < kResRow; ++u) s = fma(rva[q][u], rci[q][u][off], s);
        return s;
    }
    // all products of a phase, every gather in flight before the first product
    __device__ __forceinline__ void cols(double (&s)[S]) const {
        double v[S][kResCol];
#pragma unroll
        for (int q = 0; q < S; ++q)
#pragma unroll
            for (int u = 0; u < kResCol; ++u) v[q][u] = *tci[q][u];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < S; ++q) {
            s[q] = 0.0;
#pragma unroll
            for (int u = 0; u < kResCol; ++u) s[q] = fma(tva[q][u], v[q][u], s[q]);
        }
    }
    __device__ __forceinline__ void rows(double (&s)[SR]) const {
        double v[SR][kResRow];
#pragma unroll
        for (int q = 0; q < SR; ++q)
#pragma unroll
            for (int u = 0; u < kResRow; ++u) v[q][u] = *rci[q][u];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            s[q] = 0.0;
#pragma unroll
            for (int u = 0; u < kResRow; ++u) s[q] = fma(rva[q][u], v[q][u], s[q]);
        }
    }
};

// Factors of x <- A x^ - G x + B x0 at restart length k.
__device__ __forceinline__ void momentum_factors(double k, double gam, double &A, double &G, double &B) {
    const double ak = (k + 1.0) / (k + 2.0);
    A = ak * (1.0 + gam);
    G = ak * gam;
    B = 1.0 / (k + 2.0);
}

// The iteration of k_batch_solve for a shared matrix whose column slices hold
// at most kResCol entries and row slices at most kResRow (node-arc incidence
// matrices: two entries per column, node degree <= 8); S columns and SR rows
// per thread. Everything an instance needs stays in registers for its whole
// solve - the entries of the owned columns and rows, each index turned into
// the LDS address of what it gathers, and x, x0, c~, l~, u~, y, y0 and the
// clamp bounds of the dual step - except the gathered vectors in LDS. The
// loop has no branch per slot (slots past the end work on zeros and write
// into LDS nobody gathers), so all gathers of a phase are in flight at once;
// the momentum factors come from a table that the first wave's lanes fill for
// kResSteps iterations at a time, and the dual step is w = y - sigma a,
// y^ = w - clamp(w, -sigma u_c, -sigma l_c): no division is left in the loop.
// Checks work on the same registers: c_j x_j and l_j lambda_j are the same
// products in scaled space, the products of the anchor that the rays compare
// with are gathered again from x0 and y0 in LDS, and only D_c, D_r, the row
// bounds and (afterwards) the row entries are read from memory.
//
// What bounds it: at 32x32 grids (3,968 columns, 1,024 rows; 512 threads, 8
// columns and 2 rows each) an iteration issues 960 wave instructions and keeps
// the LDS busy for 1,400 cycles, which the two barriers put one after the
// other: 0.99 us, and 1.23 us with a check every 64 iterations. Streaming the
// row bounds, cost and anchor from LDS with a branch per slot and four
// divisions took 2.82 us (2,650 wave instructions, 2,350 LDS cycles, 1,000 of
// them bank conflicts). Checks in rolled loops from memory cost 58 us each,
// at 1,024 threads 146 us of spills: hence 512 threads at most.
template <int BT, int S>
__global__ __launch_bounds__(BT) void k_batch_solve_res(BArgs a, BOpts o) {
    using L = ResLds<BT, S>;
    constexpr int SR = L::SR;
    constexpr int PX = res_pos(BT);   // LDS elements per column slot
    extern __shared__ double lds[];
    LdsDouble *const sy = (LdsDouble *)lds, *const sx = sy + L::x, *const stp = sy + L::step;
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= a.B) return;
        const Geo g = geometry(a, b);
        const double *Dr = a.Dr, *Dc = a.Dc;
        const double eta = a.eta[0];
        const double gam = o.gamma;
        ResEntries<BT, S> M;
        double xr[S], x0r[S], cr[S], lr[S], ur[S];
        double yr[SR], y0r[SR], lo[SR], hi[SR];   // lo, hi: -sigma u_c, -sigma l_c
        LdsDouble *const myx = sx + res_pos((int32_t)threadIdx.x), *const myy = sy + (int32_t)threadIdx.x;
        LdsDouble *const myx0 = myx + (L::x0 - L::x), *const myaty = myy + L::aty;

        // entries, scaled data, norms, initial point
        double nrm[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = (int32_t)threadIdx.x + q * BT;
            xr[q] = x0r[q] = cr[q] = lr[q] = ur[q] = 0.0;
            if (j < g.n) {
                const double d = Dc[j], co = a.c_o[g.vc + j];
                cr[q] = d * co;
                lr[q] = a.lv_o[g.vc + j] / d;
                ur[q] = a.uv_o[g.vc + j] / d;
                nrm[0] += cr[q] * cr[q];
                nrm[2] += co * co;
                xr[q] = clampd(a.x_init ? a.x_init[g.vc + j] / d : 0.0, lr[q], ur[q]);
                x0r[q] = xr[q];
            }
            M.load_col(a, g, sy, q, j);
            myx0[q * PX] = x0r[q];
        }
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = (int32_t)threadIdx.x + q * BT;
            yr[q] = y0r[q] = lo[q] = hi[q] = 0.0;
            if (i < g.m) {
                const double d = Dr[i], loo = a.lc_o[g.vr + i], hio = a.uc_o[g.vr + i];
                const double l = d * loo, u = d * hio;
                double bb = 0.0, bo = 0.0;
                if (isfinite(l)) bb = fmax(bb, fabs(l));
                if (isfinite(u)) bb = fmax(bb, fabs(u));
                if (isfinite(loo)) bo = fmax(bo, fabs(loo));
                if (isfinite(hio)) bo = fmax(bo, fabs(hio));
                nrm[1] += bb * bb;
                nrm[3] += bo * bo;
                yr[q] = clampd(a.y_init ? a.y_init[g.vr + i] / d : 0.0, isfinite(u) ? -INFINITY : 0.0,
                               isfinite(l) ? INFINITY : 0.0);
                y0r[q] = yr[q];
            }
            myy[q * BT] = yr[q];
            myy[L::y0 + q * BT] = yr[q];
        }
        wg_sum<BT, 4>(nrm);
        // what all threads know lives in scalar registers
        const double cn = sqrt(nrm[0]), bn = sqrt(nrm[1]);
        const double cnorm = uniform_value(sqrt(nrm[2])), bnorm = uniform_value(sqrt(nrm[3]));
        double omega = uniform_value((cn > 1e-10 && bn > 1e-10) ? cn / bn : 1.0);
        double tau = uniform_value(eta / omega), sigma = uniform_value(eta * omega);
        M.load_rows(a, g, sx);
        // clamp bounds of the dual step at this sigma
        auto dual_bounds = [&]() {
            int32_t t0 = (int32_t)threadIdx.x;
            asm volatile("" : "+v"(t0));
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                const int32_t i = t0 + q * BT;
                if (i < g.m) {
                    lo[q] = -sigma * (Dr[i] * a.uc_o[g.vr + i]);
                    hi[q] = -sigma * (Dr[i] * a.lc_o[g.vr + i]);
                }
            }
        };
        dual_bounds();

        // x^ of the owned columns and s = A~'y, x_ext to LDS; y^ of the owned rows
        auto columns = [&](double (&s)[S], double (&xn)[S]) {
            M.cols(s);
#pragma unroll
            for (int q = 0; q < S; ++q) {
                xn[q] = clamp_quiet(xr[q] - tau * (cr[q] - s[q]), lr[q], ur[q]);
                myx[q * PX] = 2.0 * xn[q] - xr[q];
            }
        };
        auto rows = [&](double (&yn)[SR]) {
            M.rows(yn);
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                const double w = fma(-sigma, yn[q], yr[q]);
                yn[q] = w - clamp_quiet(w, lo[q], hi[q]);
            }
        };

        int64_t t = 0, k = 0, restarts = 0;
        int32_t tc = 0;   // t modulo check_every
        double r_start = 0.0, r_prev = 0.0;
        int32_t status = 0;
        bool anchor_valid = false;   // x0, y0 are the point of a restart
        double ray_scale = 0.0;
        double kkt = 0.0, rel_p = 0.0, rel_d = 0.0, rel_g = 0.0, P = 0.0, D = 0.0;
        for (;;) {
            // iterations t .. t + plain - 1 run without a check, then one that
            // keeps its PDHG point for the check
            int32_t plain = tc == 0 ? 0 : o.check_every - tc;
            if ((int64_t)plain > o.limit - 1 - t) plain = (int32_t)(o.limit - 1 - t);
            plain = __builtin_amdgcn_readfirstlane(plain);
            for (int32_t p = 0; p < plain; p += kResSteps) {
                const int32_t cnt = plain - p < kResSteps ? plain - p : kResSteps;
                // x <- A x^ - G x + B x0 in iterations p .. p + cnt - 1
                if ((int32_t)threadIdx.x < cnt) {
                    const int32_t u = (int32_t)threadIdx.x;
                    double A, G, B;
                    momentum_factors((double)(k + p + u), gam, A, G, B);
                    stp[4 * u] = A;
                    stp[4 * u + 1] = G;
                    stp[4 * u + 2] = B;
                }
                __syncthreads();
#pragma unroll 1
                for (int32_t it = 0; it < cnt; ++it) {
                    const double A = stp[4 * it], G = stp[4 * it + 1], B = stp[4 * it + 2];
                    double s[S], xn[S], yn[SR];
                    columns(s, xn);
#pragma unroll
                    for (int q = 0; q < S; ++q) xr[q] = A * xn[q] - G * xr[q] + B * x0r[q];
                    __syncthreads();
                    rows(yn);
#pragma unroll
                    for (int q = 0; q < SR; ++q) {
                        yr[q] = A * yn[q] - G * yr[q] + B * y0r[q];
                        myy[q * BT] = yr[q];
                    }
                    __syncthreads();
                }
            }
            t += plain;
            k += plain;
            const bool last = t + 1 >= o.limit;
            // the iteration before the check: its PDHG point replaces x_ext and y in LDS
            {
                double s[S], xn[S], yn[SR];
                columns(s, xn);
#pragma unroll
                for (int q = 0; q < S; ++q) myaty[q * BT] = s[q];
                __syncthreads();
                rows(yn);
                __syncthreads();
#pragma unroll
                for (int q = 0; q < S; ++q) myx[q * PX] = xn[q];
#pragma unroll
                for (int q = 0; q < SR; ++q) myy[q * BT] = yn[q];
            }
            __syncthreads();
            // KKT sums, then the ray sums: v[10], v[11] over the columns
            // (bound terms, c'dx), v[12] over the rows; rmx the ray violations
            int32_t t0 = (int32_t)threadIdx.x;
            asm volatile("" : "+v"(t0));   // addresses are formed here, not kept over the loop
            const bool rays = o.detect && anchor_valid;
            double v[13], rmx[2] = {0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 13; ++q) v[q] = 0.0;
            // one slot at a time, x^, x0, y^, y0 from LDS, the rows first: their
            // entries are loaded again after the check, so that the columns'
            // terms have room beside the registers that live on
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                const int32_t i = t0 + q * BT;
                if (i < g.m) {
                    const double d = Dr[i], loo = a.lc_o[g.vr + i], hio = a.uc_o[g.vr + i], yh = myy[q * BT];
                    const double p = M.row(q, 0);
                    const double ax = p / d;
                    const double rpr = ax - clampd(ax, loo, hio);
                    v[6] += rpr * rpr;
                    const double yo = d * yh;
                    v[7] += (isfinite(loo) ? loo * fmax(yo, 0.0) : 0.0) - (isfinite(hio) ? hio * fmax(-yo, 0.0) : 0.0);
                    const double dy = yh - yr[q];
                    v[8] += dy * dy;
                    const double d0 = yh - myy[L::y0 + q * BT];
                    v[9] += d0 * d0;
                    if (rays) {
                        double s1[1], m2[2];
                        ray_row_terms(p, M.row(q, L::x0 - L::x), d, d0, loo, hio, s1, m2);
                        v[12] += s1[0];
                        rmx[0] = fmax(rmx[0], m2[0]);
                        rmx[1] = fmax(rmx[1], m2[1]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t j = t0 + q * BT;
                if (j < g.n) {
                    const double d = Dc[j], xh = myx[q * PX];
                    const double qq = M.col(q, 0);
                    const double dx = xh - xr[q];
                    v[0] += dx * dx;
                    v[1] += (qq - myaty[q * BT]) * dx;
                    const double d0 = xh - myx0[q * PX];
                    v[2] += d0 * d0;
                    const double gr = cr[q] - qq;   // D_c times the original-space gradient
                    const bool lf = isfinite(lr[q]), uf = isfinite(ur[q]);
                    const double lam = (!lf && !uf) ? 0.0 : (lf && !uf) ? fmax(gr, 0.0) : (!lf && uf) ? fmin(gr, 0.0) : gr;
                    const double rd = (gr - lam) / d;
                    v[3] += rd * rd;
                    v[4] += cr[q] * xh;
                    v[5] += (lf ? lr[q] * fmax(lam, 0.0) : 0.0) - (uf ? ur[q] * fmax(-lam, 0.0) : 0.0);
                    if (rays) {
                        double s2[2], m2[2];
                        ray_col_terms(qq, M.col(q, L::y0), d, d0, cr[q] / d, lr[q] * d, ur[q] * d, s2, m2);
                        v[10] += s2[0];
                        v[11] += s2[1];
                        rmx[0] = fmax(rmx[0], m2[0]);
                        rmx[1] = fmax(rmx[1], m2[1]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            wg_sum<BT, 13>(v);
            P = uniform_value(v[4]);
            D = uniform_value(v[7] + v[5]);
            rel_p = uniform_value(sqrt(v[6]) / (1.0 + bnorm));
            rel_d = uniform_value(sqrt(v[3]) / (1.0 + cnorm));
            rel_g = uniform_value(fabs(P - D) / (1.0 + fabs(P) + fabs(D)));
            kkt = rel_p;
            if (rel_d > kkt || isnan(rel_d)) kkt = rel_d;
            if (rel_g > kkt || isnan(rel_g)) kkt = rel_g;
            if (isnan(kkt)) {
                status = PDHG_NUMERICAL_ERROR;
                break;
            }
            if (kkt <= o.eps) {
                status = PDHG_OPTIMAL;
                break;
            }
            if (rays) {
                wg_max<BT, 2>(rmx);
                const double obj_d = v[10] + v[12], obj_p = v[11];
                if (o.eps_pinf > 0.0 && obj_d > 0.0 && rmx[0] <= o.eps_pinf * obj_d) {
                    status = PDHG_PRIMAL_INFEASIBLE;
                    ray_scale = uniform_value(1.0 / obj_d);
                    break;
                }
                if (o.eps_dinf > 0.0 && obj_p < 0.0 && rmx[1] <= o.eps_dinf * (-obj_p)) {
                    status = PDHG_DUAL_INFEASIBLE;
                    ray_scale = uniform_value(-1.0 / obj_p);
                    break;
                }
            }
            if (last) {
                status = PDHG_ITERATION_LIMIT;
                break;
            }
            const double r2 = v[0] / tau + v[8] / sigma + 2.0 * v[1];
            const double r = uniform_value(r2 > 0.0 ? sqrt(r2) : 0.0);
            bool restart = false;
            if (t == 0) {
                r_start = r;
                r_prev = r;
            } else if (r <= o.beta_suff * r_start || (r <= o.beta_nec * r_start && r > r_prev) ||
                       (double)k >= o.beta_art * (double)t) {
                restart = true;
            } else {
                r_prev = r;
            }
            if (restart) {
                // exp(log(dyr / dxr) / 2 + log(omega) / 2), without a call that
                // would save half of the registers
                const double dxr = sqrt(v[2]), dyr = sqrt(v[9]);
                if (dxr > 1e-10 && dyr > 1e-10) omega = uniform_value(sqrt(dyr / dxr) * sqrt(omega));
                tau = uniform_value(eta / omega);
                sigma = uniform_value(eta * omega);
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    xr[q] = myx[q * PX];
                    x0r[q] = xr[q];
                    myx0[q * PX] = xr[q];
                }
#pragma unroll
                for (int q = 0; q < SR; ++q) {
                    yr[q] = myy[q * BT];
                    y0r[q] = yr[q];
                    myy[L::y0 + q * BT] = yr[q];
                }
                dual_bounds();
                anchor_valid = true;
                k = 0;
                r_start = r;
                r_prev = r;
                ++restarts;
            } else {
                double A, G, B;
                momentum_factors((double)k, gam, A, G, B);
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    x0r[q] = myx0[q * PX];
                    xr[q] = A * myx[q * PX] - G * xr[q] + B * x0r[q];
                }
#pragma unroll
                for (int q = 0; q < SR; ++q) {
                    y0r[q] = myy[L::y0 + q * BT];
                    yr[q] = A * myy[q * BT] - G * yr[q] + B * y0r[q];
                    myy[q * BT] = yr[q];
                }
                ++k;
            }
            M.load_rows(a, g, sx);
            ++t;
            tc = o.check_every == 1 ? 0 : 1;
            __syncthreads();
        }
        // original-space output of the last PDHG point, or the certifying ray
        const bool xray = status == PDHG_DUAL_INFEASIBLE, yray = status == PDHG_PRIMAL_INFEASIBLE;
        int32_t t0 = (int32_t)threadIdx.x;
        asm volatile("" : "+v"(t0));
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = t0 + q * BT;
            const double xh = myx[q * PX];
            if (j < g.n) a.x_out[g.vc + j] = Dc[j] * (xray ? (xh - myx0[q * PX]) * ray_scale : xh);
        }
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = t0 + q * BT;
            const double yh = myy[q * BT];
            if (i < g.m) a.y_out[g.vr + i] = Dr[i] * (yray ? (yh - myy[L::y0 + q * BT]) * ray_scale : yh);
        }
        if (threadIdx.x == 0) {
            BatchRes r;
            r.pobj = P;
            r.dobj = D;
            r.rel_p = rel_p;
            r.rel_d = rel_d;
            r.rel_g = rel_g;
            r.kkt = kkt;
            r.omega = omega;
            r.eta = eta;
            r.iterations = t + 1;
            r.restarts = restarts;
            r.status = status;
            r.power_iters = a.power_iters[0];
            a.res[b] = r;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// on-chip solve of any instance with at most 2 columns and rows per thread

// Pairs of entries of each owned column (row) that stay in registers: as measured,
// not as fits. Of a thread's registers 16 to 23 are in scratch memory at one column
// (5 at 1,024 threads) and 92 to 132 at two (22 to 37), most of them across checks
// only; an iteration reloads at most 34.
template <int BT, int S, int SR>
struct LdsShape {
    static constexpr int KC = BT == 1024 ? 0 : S == 1 ? 8 : 6;
    static constexpr int KR = BT == 1024 ? 0 : S == 1 ? 14 : SR == 1 ? 12 : 6;
    static constexpr int U = 4;
    static constexpr bool ahead = BT < 1024;
    static constexpr int32_t x = SR * BT;                  // x_ext after y
    static constexpr int32_t step = x + S * BT;            // momentum factors
    static constexpr size_t bytes = ((size_t)step + 4 * kResSteps) * sizeof(double);
};

typedef __attribute__((address_space(3))) char LdsByte;

// sell_pair for a vector in LDS.
__device__ __forceinline__ double lds_pair(uint32_t c, double2 a, const LdsDouble *v, double acc) {
    const LdsByte *p = (const LdsByte *)v;
    acc = fma(a.x, *(const LdsDouble *)(p + (c & 0xffffu)), acc);
    return fma(a.y, *(const LdsDouble *)(p + (c >> 16)), acc);
}

// The pairs of one position of a SELL-64 slice: the first K in registers, the
// next lc in LDS, the rest streamed. In LDS a slice's pair takes kPairBytes:
// 64 pairs of values, then 64 words of positions.
constexpr int kPairBytes = 64 * (16 + 4);
typedef double DoublePair __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) DoublePair LdsDoublePair;
typedef __attribute__((address_space(3))) uint32_t LdsWord;

template <int K, int U, bool AHEAD>
struct SellRow {
    uint32_t c[K > 0 ? K : 1];
    double2 v[K > 0 ? K : 1];
    int32_t w, lc;   // pairs of the slice, of them in LDS (scalars)
    int32_t e0;      // this lane's first pair
    LdsByte *lv;     // and its first pair of values in LDS

    // cache: room pairs at byte off are the slice's share of the LDS
    __device__ __forceinline__ void load(const uint32_t *__restrict__ ci, const double2 *__restrict__ va, int32_t first,
                                         int32_t end, int32_t lane, LdsByte *cache, int32_t off, int32_t room) {
        w = __builtin_amdgcn_readfirstlane(end - first);
        lc = __builtin_amdgcn_readfirstlane(w - K < room ? (w > K ? w - K : 0) : room);
        e0 = 64 * first + lane;
        lv = cache + off + 16 * lane;
#pragma unroll
        for (int u = 0; u < K; ++u) {
            c[u] = u < w ? ci[e0 + 64 * u] : 0;
            v[u] = u < w ? va[e0 + 64 * u] : double2{0.0, 0.0};
        }
        LdsByte *p = cache + off;
        for (int32_t k = 0; k < lc; ++k, p += kPairBytes) {
            const double2 t = va[e0 + 64 * (K + k)];
            *(LdsDoublePair *)(p + 16 * lane) = DoublePair{t.x, t.y};
            *(LdsWord *)(p + 1024 + 4 * lane) = ci[e0 + 64 * (K + k)];
        }
    }
    // row sum in row order; the streamed pairs come in groups of U (AHEAD: one
    // group ahead of the products)
    __device__ __forceinline__ double dot(const uint32_t *__restrict__ ci, const double2 *__restrict__ va,
                                          const LdsDouble *vec, int32_t lane) const {
        uint32_t nc[U];
        double2 nv[U];
        auto fetch = [&](int32_t k) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t kk = k + u < w ? k + u : w - 1;
                nc[u] = ci[e0 + 64 * kk];
                nv[u] = va[e0 + 64 * kk];
            }
        };
        if (AHEAD && w > K + lc) fetch(K + lc);
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < K; k += 2)
            if (k < w) {
#pragma unroll
                for (int u = k; u < k + 2 && u < K; ++u) acc = lds_pair(c[u], v[u], vec, acc);
            }
        const LdsByte *p = lv, *pw = lv + 1024 - 12 * lane;
#pragma unroll 1
        for (int32_t k = 0; k < lc; k += 2) {
            // the second pair of an odd count lies in the next slice's share or
            // past it, inside the allocation; it is read and not used
            const DoublePair v0 = *(const LdsDoublePair *)p, v1 = *(const LdsDoublePair *)(p + kPairBytes);
            const uint32_t c0 = *(const LdsWord *)pw, c1 = *(const LdsWord *)(pw + kPairBytes);
            acc = lds_pair(c0, double2{v0.x, v0.y}, vec, acc);
            if (k + 1 < lc) acc = lds_pair(c1, double2{v1.x, v1.y}, vec, acc);
            p += 2 * kPairBytes;
            pw += 2 * kPairBytes;
        }
#pragma unroll 1
        for (int32_t k = K + lc; k < w; k += U) {
            if (!AHEAD) fetch(k);
            uint32_t cc[U];
            double2 cv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cc[u] = nc[u];
                cv[u] = nv[u];
            }
            if (AHEAD && k + U < w) fetch(k + U);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k + u < w) acc = lds_pair(cc[u], cv[u], vec, acc);
        }
        return acc;
    }
};

// The iteration of k_batch_solve on chip: a workgroup's instance lives in
// position space (see BArgs), S columns and SR rows per thread in whole
// SELL-64 slices; iterates, anchors, costs and bounds in registers, the
// gathered vectors x_ext and y (at checks the PDHG point) in LDS, the first
// pairs of every row and column in registers and the others streamed from L2
// or the memory-side cache. Iterations between checks, the dual step and the
// momentum factors are those of k_batch_solve_res.
//
// What bounds it: up to about 300 rows (5% dense) the latency of the two
// phases - gathers, the sum of a row in its order, a barrier -, beyond that
// the entries that neither registers nor LDS hold. Rows sorted by length cut
// the padding from 1.6 to 1.1, positions of 16 bits and pairs the bytes from
// 12 to 10 an entry at half the loads. Per iteration of 256 instances, 1,024
// in the batch, n = 2 m: m = 57 0.98 -> 0.36 us, 120 2.45 -> 0.77, 250 8.2 ->
// 2.6, 480 33 -> 11.2 (4.9 TB/s from the memory-side cache).
template <int BT, int S, int SR>
__global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(BT == 1024 ? 4 : 2))) void
k_batch_solve_lds(BArgs a, BOpts o, int32_t cache_pairs) {
    using L = LdsShape<BT, S, SR>;
    constexpr int NW = BT / 64;
    extern __shared__ __attribute__((aligned(16))) double lds[];
    LdsByte *const cache = (LdsByte *)(LdsDouble *)lds + L::bytes;
    LdsDouble *const sy = (LdsDouble *)lds, *const sx = sy + L::x, *const stp = sy + L::step;
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= a.B) return;
        const Geo g = geometry(a, b);
        const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x >> 6);
        const int32_t lane = (int32_t)(threadIdx.x & 63);
        const double *Dr = a.Dr + g.dr, *Dc = a.Dc + g.dc;
        const double *lc_o = a.lc_o + g.vr, *uc_o = a.uc_o + g.vr;
        const double eta = a.eta[g.sidx];
        const double gam = o.gamma;
        SellRow<L::KC, L::U, L::ahead> col[S];
        SellRow<L::KR, L::U, L::ahead> row[SR];
        double xr[S], x0r[S], cr[S], lr[S], ur[S];
        double yr[SR], y0r[SR], lo[SR], hi[SR];   // lo, hi: -sigma u_c, -sigma l_c
        LdsDouble *const myx = sx + (int32_t)threadIdx.x, *const myy = sy + (int32_t)threadIdx.x;
        // an equal share of the cache for every slice
        const int32_t ncs = (g.n + 63) >> 6, nrs = (g.m + 63) >> 6, room = cache_pairs / (ncs + nrs);
        double nrm[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = (int32_t)threadIdx.x + q * BT, sl = wave + q * NW;
            int32_t k0 = 0, k1 = 0;
            if (64 * sl < g.n) {
                const int32_t f = a.shared ? 0 : a.tsfirst[b];
                k0 = a.tsp[f + sl];
                k1 = a.tsp[f + sl + 1];
            }
            col[q].load(a.tsci, a.tsva, k0, k1, lane, cache, kPairBytes * room * sl, room);
            xr[q] = cr[q] = lr[q] = ur[q] = 0.0;
            if (j < g.n) {
                const int32_t jo = row_at(a.tperm, g.c0, j);
                const double d = Dc[jo], co = a.c_o[g.vc + jo];
                cr[q] = d * co;
                lr[q] = a.lv_o[g.vc + jo] / d;
                ur[q] = a.uv_o[g.vc + jo] / d;
                nrm[0] += cr[q] * cr[q];
                nrm[2] += co * co;
                xr[q] = clampd(a.x_init ? a.x_init[g.vc + jo] / d : 0.0, lr[q], ur[q]);
            }
            x0r[q] = xr[q];
        }
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = (int32_t)threadIdx.x + q * BT, sl = wave + q * NW;
            int32_t k0 = 0, k1 = 0;
            if (64 * sl < g.m) {
                const int32_t f = a.shared ? 0 : a.asfirst[b];
                k0 = a.asp[f + sl];
                k1 = a.asp[f + sl + 1];
            }
            row[q].load(a.asci, a.asva, k0, k1, lane, cache, kPairBytes * room * (ncs + sl), room);
            yr[q] = lo[q] = hi[q] = 0.0;
            if (i < g.m) {
                const int32_t io = row_at(a.aperm, g.r0, i);
                const double d = Dr[io], loo = lc_o[io], hio = uc_o[io];
                const double l = d * loo, u = d * hio;
                double bb = 0.0, bo = 0.0;
                if (isfinite(l)) bb = fmax(bb, fabs(l));
                if (isfinite(u)) bb = fmax(bb, fabs(u));
                if (isfinite(loo)) bo = fmax(bo, fabs(loo));
                if (isfinite(hio)) bo = fmax(bo, fabs(hio));
                nrm[1] += bb * bb;
                nrm[3] += bo * bo;
                yr[q] = clampd(a.y_init ? a.y_init[g.vr + io] / d : 0.0, isfinite(u) ? -INFINITY : 0.0,
                               isfinite(l) ? INFINITY : 0.0);
            }
            y0r[q] = yr[q];
            myy[q * BT] = yr[q];
        }
        wg_sum<BT, 4>(nrm);
        const double cn = sqrt(nrm[0]), bn = sqrt(nrm[1]);
        const double cnorm = uniform_value(sqrt(nrm[2])), bnorm = uniform_value(sqrt(nrm[3]));
        double omega = uniform_value((cn > 1e-10 && bn > 1e-10) ? cn / bn : 1.0);
        double tau = uniform_value(eta / omega), sigma = uniform_value(eta * omega);
        auto dual_bounds = [&]() {
            int32_t t0 = (int32_t)threadIdx.x;
            asm volatile("" : "+v"(t0));
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                const int32_t i = t0 + q * BT;
                if (i < g.m) {
                    const int32_t io = row_at(a.aperm, g.r0, i);
                    lo[q] = -sigma * (Dr[io] * uc_o[io]);
                    hi[q] = -sigma * (Dr[io] * lc_o[io]);
                }
            }
        };
        dual_bounds();
        // s = A~'y, x^ of the owned columns, x_ext to LDS; y^ of the owned rows
        auto columns = [&](double (&s)[S], double (&xn)[S]) {
#pragma unroll
            for (int q = 0; q < S; ++q) {
                s[q] = xn[q] = 0.0;
                if (64 * (wave + q * NW) < g.n) {
                    s[q] = col[q].dot(a.tsci, a.tsva, sy, lane);
                    xn[q] = clamp_quiet(xr[q] - tau * (cr[q] - s[q]), lr[q], ur[q]);
                    myx[q * BT] = 2.0 * xn[q] - xr[q];
                }
            }
        };
        auto rows = [&](double (&yn)[SR]) {
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                yn[q] = 0.0;
                if (64 * (wave + q * NW) < g.m) {
                    const double w = fma(-sigma, row[q].dot(a.asci, a.asva, sx, lane), yr[q]);
                    yn[q] = w - clamp_quiet(w, lo[q], hi[q]);
                }
            }
        };

        int64_t t = 0, k = 0, restarts = 0;
        int32_t tc = 0;   // t modulo check_every
        double r_start = 0.0, r_prev = 0.0;
        int32_t status = 0;
        bool anchor_valid = false;   // the anchor's products are stored (after a restart)
        double ray_scale = 0.0;
        double kkt = 0.0, rel_p = 0.0, rel_d = 0.0, rel_g = 0.0, P = 0.0, D = 0.0;
        for (;;) {
            // iterations t .. t + plain - 1 run without a check, then one that
            // keeps its PDHG point for the check
            int32_t plain = tc == 0 ? 0 : o.check_every - tc;
            if ((int64_t)plain > o.limit - 1 - t) plain = (int32_t)(o.limit - 1 - t);
            plain = __builtin_amdgcn_readfirstlane(plain);
            for (int32_t p = 0; p < plain; p += kResSteps) {
                const int32_t cnt = plain - p < kResSteps ? plain - p : kResSteps;
                for (int32_t u = (int32_t)threadIdx.x; u < cnt; u += BT) {
                    double A, G, B;
                    momentum_factors((double)(k + p + u), gam, A, G, B);
                    stp[4 * u] = A;
                    stp[4 * u + 1] = G;
                    stp[4 * u + 2] = B;
                }
                __syncthreads();
#pragma unroll 1
                for (int32_t it = 0; it < cnt; ++it) {
                    const double A = stp[4 * it], G = stp[4 * it + 1], B = stp[4 * it + 2];
                    double s[S], xn[S], yn[SR];
                    columns(s, xn);
#pragma unroll
                    for (int q = 0; q < S; ++q) xr[q] = A * xn[q] - G * xr[q] + B * x0r[q];
                    __syncthreads();
                    rows(yn);
#pragma unroll
                    for (int q = 0; q < SR; ++q) {
                        yr[q] = A * yn[q] - G * yr[q] + B * y0r[q];
                        myy[q * BT] = yr[q];
                    }
                    __syncthreads();
                }
            }
            t += plain;
            k += plain;
            const bool last = t + 1 >= o.limit;
            // the iteration before the check: its PDHG point replaces x_ext and y in LDS
            double s[S];
            {
                double xn[S], yn[SR];
                columns(s, xn);
                __syncthreads();
                rows(yn);
                __syncthreads();
#pragma unroll
                for (int q = 0; q < S; ++q) myx[q * BT] = xn[q];
#pragma unroll
                for (int q = 0; q < SR; ++q) myy[q * BT] = yn[q];
            }
            __syncthreads();
            // KKT sums, then the ray sums: v[10], v[11] over the columns
            // (bound terms, c'dx), v[12] over the rows; rmx the ray violations
            int32_t t0 = (int32_t)threadIdx.x;
            asm volatile("" : "+v"(t0));   // addresses are formed here, not kept over the loop
            const bool rays = o.detect && anchor_valid;
            double v[13], rmx[2] = {0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 13; ++q) v[q] = 0.0;
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                const int32_t i = t0 + q * BT;
                if (64 * (wave + q * NW) < g.m) {
                    const double p = row[q].dot(a.asci, a.asva, sx, lane);
                    if (i < g.m) {
                        const int32_t io = row_at(a.aperm, g.r0, i);
                        const double d = Dr[io], loo = lc_o[io], hio = uc_o[io], yh = myy[q * BT];
                        const double ax = p / d;
                        const double rpr = ax - clampd(ax, loo, hio);
                        v[6] += rpr * rpr;
                        const double yo = d * yh;
                        v[7] += (isfinite(loo) ? loo * fmax(yo, 0.0) : 0.0) -
                                (isfinite(hio) ? hio * fmax(-yo, 0.0) : 0.0);
                        const double dy = yh - yr[q];
                        v[8] += dy * dy;
                        const double d0 = yh - y0r[q];
                        v[9] += d0 * d0;
                        if (o.detect) a.ph[g.vr + i] = p;
                        if (rays) {
                            double s1[1], m2[2];
                            ray_row_terms(p, a.p0[g.vr + i], d, d0, loo, hio, s1, m2);
                            v[12] += s1[0];
                            rmx[0] = fmax(rmx[0], m2[0]);
                            rmx[1] = fmax(rmx[1], m2[1]);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t j = t0 + q * BT;
                if (64 * (wave + q * NW) < g.n) {
                    const double qq = col[q].dot(a.tsci, a.tsva, sy, lane);
                    if (j < g.n) {
                        const int32_t jo = row_at(a.tperm, g.c0, j);
                        const double d = Dc[jo], xh = myx[q * BT];
                        const double dx = xh - xr[q];
                        v[0] += dx * dx;
                        v[1] += (qq - s[q]) * dx;
                        const double d0 = xh - x0r[q];
                        v[2] += d0 * d0;
                        const double c = cr[q], l = lr[q], u = ur[q];
                        const double gr = c - qq;   // D_c times the original-space gradient
                        const bool lf = isfinite(l), uf = isfinite(u);
                        const double lam = (!lf && !uf) ? 0.0 : (lf && !uf) ? fmax(gr, 0.0) : (!lf && uf) ? fmin(gr, 0.0) : gr;
                        const double rd = (gr - lam) / d;
                        v[3] += rd * rd;
                        v[4] += c * xh;
                        v[5] += (lf ? l * fmax(lam, 0.0) : 0.0) - (uf ? u * fmax(-lam, 0.0) : 0.0);
                        if (o.detect) a.qh[g.vc + j] = qq;
                        if (rays) {
                            double s2[2], m2[2];
                            ray_col_terms(qq, a.q0[g.vc + j], d, d0, c / d, l * d, u * d, s2, m2);
                            v[10] += s2[0];
                            v[11] += s2[1];
                            rmx[0] = fmax(rmx[0], m2[0]);
                            rmx[1] = fmax(rmx[1], m2[1]);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            wg_sum<BT, 13>(v);
            P = uniform_value(v[4]);
            D = uniform_value(v[7] + v[5]);
            rel_p = uniform_value(sqrt(v[6]) / (1.0 + bnorm));
            rel_d = uniform_value(sqrt(v[3]) / (1.0 + cnorm));
            rel_g = uniform_value(fabs(P - D) / (1.0 + fabs(P) + fabs(D)));
            kkt = rel_p;
            if (rel_d > kkt || isnan(rel_d)) kkt = rel_d;
            if (rel_g > kkt || isnan(rel_g)) kkt = rel_g;
            if (isnan(kkt)) {
                status = PDHG_NUMERICAL_ERROR;
                break;
            }
            if (kkt <= o.eps) {
                status = PDHG_OPTIMAL;
                break;
            }
            if (rays) {
                wg_max<BT, 2>(rmx);
                const double obj_d = v[10] + v[12], obj_p = v[11];
                if (o.eps_pinf > 0.0 && obj_d > 0.0 && rmx[0] <= o.eps_pinf * obj_d) {
                    status = PDHG_PRIMAL_INFEASIBLE;
                    ray_scale = uniform_value(1.0 / obj_d);
                    break;
                }
                if (o.eps_dinf > 0.0 && obj_p < 0.0 && rmx[1] <= o.eps_dinf * (-obj_p)) {
                    status = PDHG_DUAL_INFEASIBLE;
                    ray_scale = uniform_value(-1.0 / obj_p);
                    break;
                }
            }
            if (last) {
                status = PDHG_ITERATION_LIMIT;
                break;
            }
            const double r2 = v[0] / tau + v[8] / sigma + 2.0 * v[1];
            const double r = uniform_value(r2 > 0.0 ? sqrt(r2) : 0.0);
            bool restart = false;
            if (t == 0) {
                r_start = r;
                r_prev = r;
            } else if (r <= o.beta_suff * r_start || (r <= o.beta_nec * r_start && r > r_prev) ||
                       (double)k >= o.beta_art * (double)t) {
                restart = true;
            } else {
                r_prev = r;
            }
            if (restart) {
                // exp(log(dyr / dxr) / 2 + log(omega) / 2), without a call that
                // would save half of the registers
                const double dxr = sqrt(v[2]), dyr = sqrt(v[9]);
                if (dxr > 1e-10 && dyr > 1e-10) omega = uniform_value(sqrt(dyr / dxr) * sqrt(omega));
                tau = uniform_value(eta / omega);
                sigma = uniform_value(eta * omega);
                // the check's products are those of the new anchor
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const int32_t j = t0 + q * BT;
                    xr[q] = x0r[q] = j < g.n ? myx[q * BT] : 0.0;
                    if (o.detect && j < g.n) a.q0[g.vc + j] = a.qh[g.vc + j];
                }
#pragma unroll
                for (int q = 0; q < SR; ++q) {
                    const int32_t i = t0 + q * BT;
                    yr[q] = y0r[q] = myy[q * BT];
                    if (o.detect && i < g.m) a.p0[g.vr + i] = a.ph[g.vr + i];
                }
                dual_bounds();
                anchor_valid = true;
                k = 0;
                r_start = r;
                r_prev = r;
                ++restarts;
            } else {
                double A, G, B;
                momentum_factors((double)k, gam, A, G, B);
#pragma unroll
                for (int q = 0; q < S; ++q) xr[q] = A * myx[q * BT] - G * xr[q] + B * x0r[q];
#pragma unroll
                for (int q = 0; q < SR; ++q) {
                    yr[q] = A * myy[q * BT] - G * yr[q] + B * y0r[q];
                    myy[q * BT] = yr[q];
                }
                ++k;
            }
            ++t;
            tc = o.check_every == 1 ? 0 : 1;
            __syncthreads();
        }
        // original-space output of the last PDHG point, or the certifying ray
        const bool xray = status == PDHG_DUAL_INFEASIBLE, yray = status == PDHG_PRIMAL_INFEASIBLE;
        int32_t t0 = (int32_t)threadIdx.x;
        asm volatile("" : "+v"(t0));
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = t0 + q * BT;
            if (j < g.n) {
                const int32_t jo = row_at(a.tperm, g.c0, j);
                const double xh = myx[q * BT];
                a.x_out[g.vc + jo] = Dc[jo] * (xray ? (xh - x0r[q]) * ray_scale : xh);
            }
        }
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = t0 + q * BT;
            if (i < g.m) {
                const int32_t io = row_at(a.aperm, g.r0, i);
                const double yh = myy[q * BT];
                a.y_out[g.vr + io] = Dr[io] * (yray ? (yh - y0r[q]) * ray_scale : yh);
            }
        }
        if (threadIdx.x == 0) {
            BatchRes r;
            r.pobj = P;
            r.dobj = D;
            r.rel_p = rel_p;
            r.rel_d = rel_d;
            r.rel_g = rel_g;
            r.kkt = kkt;
            r.omega = omega;
            r.eta = eta;
            r.iterations = t + 1;
            r.restarts = restarts;
            r.status = status;
            r.power_iters = a.power_iters[g.sidx];
            a.res[b] = r;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// on-chip solve that streams its entries

// Row sum over the SELL-64 slice whose pairs `first` .. `end` - 1 (wave-uniform)
// are this wave's, in row order: four pairs' loads in flight, the last ones in
// groups of two and one.
__device__ __forceinline__ double stream_dot(const uint32_t *__restrict__ ci, const double2 *__restrict__ va,
                                             int32_t first, int32_t end, int32_t lane, const LdsDouble *vec) {
    double acc = 0.0;
    int32_t e = 64 * first + lane, w = end - first;
    auto pairs = [&](auto width) {
        constexpr int U = decltype(width)::value;
        uint32_t c[U];
        double2 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = ci[e + 64 * u];
            v[u] = va[e + 64 * u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc = lds_pair(c[u], v[u], vec, acc);
        e += 64 * U;
    };
    for (; w >= 4; w -= 4) pairs(std::integral_constant<int, 4>());
    if (w & 2) pairs(std::integral_constant<int, 2>());
    if (w & 1) pairs(std::integral_constant<int, 1>());
    return acc;
}

// LDS of k_batch_solve_stream, in doubles: x_ext, then y, and the clamp bounds
// -sigma u_c, -sigma l_c of the dual step.
static size_t stream_doubles(int32_t n, int32_t m) { return (size_t)n + 3 * (size_t)m; }

// The iteration of k_batch_solve on chip for instances of S > 2 columns or rows
// per thread, or of two on a shared matrix with long slices: the gathered vectors
// and the rows' bounds in LDS, the columns' iterate, anchor, cost and bounds in
// registers, and every matrix entry streamed from the SELL-64 slices on every
// product. The point and the dual anchor of a check live in memory (xh, aty, yh,
// y, y0: read at checks, y0 once per row and iteration), by position like
// everything here.
//
// What bounds it: the latency of the slices' pairs, four in flight a lane, from
// L2 or the memory-side cache. Holding pairs in registers or LDS as
// k_batch_solve_lds does left no registers at four or eight columns a thread: its
// forms kept up to 2,400 of them in scratch memory. 600 instances of one matrix,
// 193 iterations, ray tests on / off: 1,500 x 3,000 14.1 / 13.6 -> 7.2 / 6.1 ms,
// 2,000 x 4,100 19.9 / 19.4 -> 11.3 / 9.6, 4,500 x 1,500 19.9 / 19.4 -> 8.0 / 7.2;
// 700 ragged 2,000 x 4,100 14.7 / 14.1 -> 10.6 / 9.7.
template <int BT, int S, bool RAYS>
__global__ __launch_bounds__(BT) void k_batch_solve_stream(BArgs a, BOpts o, int32_t nmax, int32_t mmax) {
    constexpr int NW = BT / 64;
    extern __shared__ __attribute__((aligned(16))) double lds[];
    LdsDouble *const sx = (LdsDouble *)lds, *const sy = sx + nmax, *const slo = sy + mmax, *const shi = slo + mmax;
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= a.B) return;
        const Geo g = geometry(a, b);
        const int32_t lane = (int32_t)(threadIdx.x & 63);
        const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x >> 6);
        const int32_t *tsp = a.tsp + (a.shared ? 0 : a.tsfirst[b]), *asp = a.asp + (a.shared ? 0 : a.asfirst[b]);
        const double *Dr = a.Dr + g.dr, *Dc = a.Dc + g.dc;
        const double *c_o = a.c_o + g.vc, *lv_o = a.lv_o + g.vc, *uv_o = a.uv_o + g.vc;
        const double *lc_o = a.lc_o + g.vr, *uc_o = a.uc_o + g.vr;
        double *__restrict__ xh = a.xh + g.vc;
        double *__restrict__ aty = a.aty + g.vc;
        double *__restrict__ y = a.y + g.vr;
        double *__restrict__ yh = a.yh + g.vr;
        double *__restrict__ y0 = a.y0 + g.vr;
        const double eta = a.eta[g.sidx];
        const double gam = o.gamma;
        double xr[S], x0r[S], cr[S], lr[S], ur[S];
        double nrm[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = (int32_t)threadIdx.x + q * BT;
            xr[q] = x0r[q] = cr[q] = lr[q] = ur[q] = 0.0;
            if (j < g.n) {
                const int32_t jo = row_at(a.tperm, g.c0, j);
                const double d = Dc[jo], co = c_o[jo];
                cr[q] = d * co;
                lr[q] = lv_o[jo] / d;
                ur[q] = uv_o[jo] / d;
                nrm[0] += cr[q] * cr[q];
                nrm[2] += co * co;
                xr[q] = clampd(a.x_init ? a.x_init[g.vc + jo] / d : 0.0, lr[q], ur[q]);
                x0r[q] = xr[q];
            }
        }
        for (int32_t i = (int32_t)threadIdx.x; i < g.m; i += BT) {
            const int32_t io = row_at(a.aperm, g.r0, i);
            const double d = Dr[io], loo = lc_o[io], hio = uc_o[io];
            const double l = d * loo, u = d * hio;
            double bb = 0.0, bo = 0.0;
            if (isfinite(l)) bb = fmax(bb, fabs(l));
            if (isfinite(u)) bb = fmax(bb, fabs(u));
            if (isfinite(loo)) bo = fmax(bo, fabs(loo));
            if (isfinite(hio)) bo = fmax(bo, fabs(hio));
            nrm[1] += bb * bb;
            nrm[3] += bo * bo;
            const double yv = clampd(a.y_init ? a.y_init[g.vr + io] / d : 0.0, isfinite(u) ? -INFINITY : 0.0,
                                     isfinite(l) ? INFINITY : 0.0);
            sy[i] = yv;
            y0[i] = yv;
        }
        wg_sum<BT, 4>(nrm);
        const double cn = sqrt(nrm[0]), bn = sqrt(nrm[1]);
        const double cnorm = uniform_value(sqrt(nrm[2])), bnorm = uniform_value(sqrt(nrm[3]));
        double omega = uniform_value((cn > 1e-10 && bn > 1e-10) ? cn / bn : 1.0);
        double tau = uniform_value(eta / omega), sigma = uniform_value(eta * omega);
        // clamp bounds of the dual step at this sigma, by the thread that reads them
        auto dual_bounds = [&]() {
            for (int32_t i = (int32_t)threadIdx.x; i < g.m; i += BT) {
                const int32_t io = row_at(a.aperm, g.r0, i);
                slo[i] = -sigma * (Dr[io] * uc_o[io]);
                shi[i] = -sigma * (Dr[io] * lc_o[io]);
            }
        };
        dual_bounds();
        auto col_dot = [&](int q) {
            const int32_t sl = wave + q * NW;
            return stream_dot(a.tsci, a.tsva, tsp[sl], tsp[sl + 1], lane, sy);
        };
        auto row_dot = [&](int q) {
            const int32_t sl = wave + q * NW;
            return stream_dot(a.asci, a.asva, asp[sl], asp[sl + 1], lane, sx);
        };
        __syncthreads();

        int64_t t = 0, k = 0, restarts = 0;
        int32_t tc = 0;   // t modulo check_every
        double r_start = 0.0, r_prev = 0.0;
        int32_t status = 0;
        bool anchor_valid = false;   // the anchor's products are stored (after a restart)
        double ray_scale = 0.0;
        double kkt = 0.0, rel_p = 0.0, rel_d = 0.0, rel_g = 0.0, P = 0.0, D = 0.0;
        for (;;) {
            // an opaque copy of the thread index: the element addresses are
            // formed in each iteration instead of being kept in registers
            int32_t tid = (int32_t)threadIdx.x;
            asm volatile("" : "+v"(tid));
            const bool last = t + 1 >= o.limit;
            const bool keep = tc == 0 || last;
            double A, G, B;
            momentum_factors((double)k, gam, A, G, B);
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t j = tid + q * BT;
                if (64 * (wave + q * NW) < g.n) {
                    const double s = col_dot(q);
                    if (j < g.n) {
                        const double xn = clamp_quiet(xr[q] - tau * (cr[q] - s), lr[q], ur[q]);
                        sx[j] = 2.0 * xn - xr[q];
                        if (keep) {
                            xh[j] = xn;
                            aty[j] = s;
                        } else {
                            xr[q] = A * xn - G * xr[q] + B * x0r[q];
                        }
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t i = tid + q * BT;
                if (64 * (wave + q * NW) < g.m) {
                    const double ya = i < g.m ? y0[i] : 0.0;
                    const double s = row_dot(q);
                    if (i < g.m) {
                        const double yv = sy[i], w = fma(-sigma, s, yv), yn = w - clamp_quiet(w, slo[i], shi[i]);
                        if (keep) {
                            yh[i] = yn;
                            y[i] = yv;
                        } else {
                            sy[i] = A * yn - G * yv + B * ya;
                        }
                    }
                }
            }
            __syncthreads();
            if (!keep) {
                ++k;
                ++t;
                tc = tc + 1 == o.check_every ? 0 : tc + 1;
                continue;
            }
            // check: the PDHG point replaces x_ext and y in LDS for the products
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t j = tid + q * BT;
                if (j < g.n) sx[j] = xh[j];
                if (j < g.m) sy[j] = yh[j];
            }
            __syncthreads();
            // KKT sums, then (RAYS) the ray sums: v[10], v[11] over the columns
            // (bound terms, c'dx), v[12] over the rows; rmx the ray violations
            constexpr int NV = RAYS ? 13 : 10;
            double v[NV], rmx[2] = {0.0, 0.0};
#pragma unroll
            for (int q = 0; q < NV; ++q) v[q] = 0.0;
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t j = tid + q * BT;
                if (64 * (wave + q * NW) < g.n) {
                    const double qq = col_dot(q);
                    if (j < g.n) {
                        const int32_t jo = row_at(a.tperm, g.c0, j);
                        const double xn = xh[j], dx = xn - xr[q], d0 = xn - x0r[q];
                        v[0] += dx * dx;
                        v[1] += (qq - aty[j]) * dx;
                        v[2] += d0 * d0;
                        const double d = Dc[jo], co = c_o[jo], lo = lv_o[jo], hi = uv_o[jo];
                        const double gr = co - qq / d;
                        const bool lf = isfinite(lo), uf = isfinite(hi);
                        const double lam = (!lf && !uf) ? 0.0 : (lf && !uf) ? fmax(gr, 0.0) : (!lf && uf) ? fmin(gr, 0.0) : gr;
                        const double rd = gr - lam;
                        v[3] += rd * rd;
                        v[4] += co * (d * xn);
                        v[5] += (lf ? lo * fmax(lam, 0.0) : 0.0) - (uf ? hi * fmax(-lam, 0.0) : 0.0);
                        if constexpr (RAYS) {
                            a.qh[g.vc + j] = qq;
                            if (anchor_valid) {
                                double s2[2], m2[2];
                                ray_col_terms(qq, a.q0[g.vc + j], d, d0, co, lo, hi, s2, m2);
                                v[10] += s2[0];
                                v[11] += s2[1];
                                rmx[0] = fmax(rmx[0], m2[0]);
                                rmx[1] = fmax(rmx[1], m2[1]);
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int32_t i = tid + q * BT;
                if (64 * (wave + q * NW) < g.m) {
                    const double p = row_dot(q);
                    if (i < g.m) {
                        const int32_t io = row_at(a.aperm, g.r0, i);
                        const double d = Dr[io], lo = lc_o[io], hi = uc_o[io];
                        const double ax = p / d;
                        const double rpr = ax - clampd(ax, lo, hi);
                        v[6] += rpr * rpr;
                        const double yn = yh[i], yo = d * yn;
                        v[7] += (isfinite(lo) ? lo * fmax(yo, 0.0) : 0.0) - (isfinite(hi) ? hi * fmax(-yo, 0.0) : 0.0);
                        const double dy = yn - y[i], d0 = yn - y0[i];
                        v[8] += dy * dy;
                        v[9] += d0 * d0;
                        if constexpr (RAYS) {
                            a.ph[g.vr + i] = p;
                            if (anchor_valid) {
                                double s1[1], m2[2];
                                ray_row_terms(p, a.p0[g.vr + i], d, d0, lo, hi, s1, m2);
                                v[12] += s1[0];
                                rmx[0] = fmax(rmx[0], m2[0]);
                                rmx[1] = fmax(rmx[1], m2[1]);
                            }
                        }
                    }
                }
            }
            wg_sum<BT, NV>(v);
            P = uniform_value(v[4]);
            D = uniform_value(v[7] + v[5]);
            rel_p = uniform_value(sqrt(v[6]) / (1.0 + bnorm));
            rel_d = uniform_value(sqrt(v[3]) / (1.0 + cnorm));
            rel_g = uniform_value(fabs(P - D) / (1.0 + fabs(P) + fabs(D)));
            kkt = rel_p;
            if (rel_d > kkt || isnan(rel_d)) kkt = rel_d;
            if (rel_g > kkt || isnan(rel_g)) kkt = rel_g;
            if (isnan(kkt)) {
                status = PDHG_NUMERICAL_ERROR;
                break;
            }
            if (kkt <= o.eps) {
                status = PDHG_OPTIMAL;
                break;
            }
            if (RAYS && anchor_valid) {
                wg_max<BT, 2>(rmx);
                const double obj_d = v[RAYS ? 10 : 0] + v[RAYS ? 12 : 0], obj_p = v[RAYS ? 11 : 0];
                if (o.eps_pinf > 0.0 && obj_d > 0.0 && rmx[0] <= o.eps_pinf * obj_d) {
                    status = PDHG_PRIMAL_INFEASIBLE;
                    ray_scale = uniform_value(1.0 / obj_d);
                    break;
                }
                if (o.eps_dinf > 0.0 && obj_p < 0.0 && rmx[1] <= o.eps_dinf * (-obj_p)) {
                    status = PDHG_DUAL_INFEASIBLE;
                    ray_scale = uniform_value(-1.0 / obj_p);
                    break;
                }
            }
            if (last) {
                status = PDHG_ITERATION_LIMIT;
                break;
            }
            const double r2 = v[0] / tau + v[8] / sigma + 2.0 * v[1];
            const double r = uniform_value(r2 > 0.0 ? sqrt(r2) : 0.0);
            bool restart = false;
            if (t == 0) {
                r_start = r;
                r_prev = r;
            } else if (r <= o.beta_suff * r_start || (r <= o.beta_nec * r_start && r > r_prev) ||
                       (double)k >= o.beta_art * (double)t) {
                restart = true;
            } else {
                r_prev = r;
            }
            // (yh, y and sy of a row belong to the thread that wrote them)
            if (restart) {
                // exp(log(dyr / dxr) / 2 + log(omega) / 2), without a call
                const double dxr = sqrt(v[2]), dyr = sqrt(v[9]);
                if (dxr > 1e-10 && dyr > 1e-10) omega = uniform_value(sqrt(dyr / dxr) * sqrt(omega));
                tau = uniform_value(eta / omega);
                sigma = uniform_value(eta * omega);
                // the check's products are those of the new anchor
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const int32_t j = tid + q * BT;
                    if (j < g.n) {
                        xr[q] = x0r[q] = xh[j];
                        if (RAYS) a.q0[g.vc + j] = a.qh[g.vc + j];
                    }
                    if (j < g.m) {
                        y0[j] = yh[j];   // sy holds it already
                        if (RAYS) a.p0[g.vr + j] = a.ph[g.vr + j];
                    }
                }
                dual_bounds();
                anchor_valid = true;
                k = 0;
                r_start = r;
                r_prev = r;
                ++restarts;
            } else {
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const int32_t j = tid + q * BT;
                    if (j < g.n) xr[q] = A * xh[j] - G * xr[q] + B * x0r[q];
                    if (j < g.m) sy[j] = A * yh[j] - G * y[j] + B * y0[j];
                }
                ++k;
            }
            ++t;
            tc = o.check_every == 1 ? 0 : 1;
            __syncthreads();
        }
        // original-space output of the last PDHG point, or the certifying ray
        const bool xray = status == PDHG_DUAL_INFEASIBLE, yray = status == PDHG_PRIMAL_INFEASIBLE;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = (int32_t)threadIdx.x + q * BT;
            if (j < g.n) {
                const int32_t jo = row_at(a.tperm, g.c0, j);
                a.x_out[g.vc + jo] = Dc[jo] * (xray ? (xh[j] - x0r[q]) * ray_scale : xh[j]);
            }
            if (j < g.m) {
                const int32_t io = row_at(a.aperm, g.r0, j);
                a.y_out[g.vr + io] = Dr[io] * (yray ? (yh[j] - y0[j]) * ray_scale : yh[j]);
            }
        }
        if (threadIdx.x == 0) {
            BatchRes r;
            r.pobj = P;
            r.dobj = D;
            r.rel_p = rel_p;
            r.rel_d = rel_d;
            r.rel_g = rel_g;
            r.kkt = kkt;
            r.omega = omega;
            r.eta = eta;
            r.iterations = t + 1;
            r.restarts = restarts;
            r.status = status;
            r.power_iters = a.power_iters[g.sidx];
            a.res[b] = r;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// unrolled iterations with a frozen schedule, and their reverse pass

struct UArgs {
    int64_t T;
    int32_t replay;                       // 1: take restarts / weights from the schedule
    uint8_t *restart;                     // [B][T]
    double *omega;                        // [B][T]
    int32_t *kk;                          // [B][T]
    uint64_t *xmask, *ymask;              // bit-packed projection states
    const int64_t *xm_off, *ym_off;       // per-instance word offsets
    const double *gx, *gy;                // cotangents of the outputs
    double *gc, *glc, *guc;               // gradients (original space)
    double *ba;                           // scratch, like lc
};

// Exactly T iterations of Algorithm 1 per instance. Restart tests run at the
// check cadence (no termination test) unless replayed; every iteration
// records omega, k, the restart flag, the set of x inside its box and the
// clamp state of every row (bit 0: at -u_c, bit 1: at -l_c).
// ONCHIP: y and x_ext live in LDS and the products walk the SELL-64 copies
// (instances whose n + m fits the LDS budget); otherwise everything stays in
// memory and the products walk the CSR arrays. Same arithmetic either way.
template <int BT, bool ONCHIP>
__global__ __launch_bounds__(BT) void k_batch_unrolled(BArgs a, BOpts o, UArgs u, int32_t nmax) {
    extern __shared__ double lds[];
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= a.B) return;
        const Geo g = geometry(a, b);
        const int32_t *arp = a.arp + g.r0, *trp = a.trp + g.c0;
        const int32_t *aci = a.aci, *tci = a.tci;
        const double *ava = a.ava, *tva = a.tva;
        // on chip the instance lives in position space: only its inputs and
        // outputs go through the permutations
        const int32_t *aperm = ONCHIP ? a.aperm : nullptr, *tperm = ONCHIP ? a.tperm : nullptr;
        const double *Dr = a.Dr + g.dr, *Dc = a.Dc + g.dc;
        const double *c_o = a.c_o + g.vc, *lv_o = a.lv_o + g.vc, *uv_o = a.uv_o + g.vc;
        const double *lc_o = a.lc_o + g.vr, *uc_o = a.uc_o + g.vr;
        double *c = a.c + g.vc, *lv = a.lv + g.vc, *uv = a.uv + g.vc;
        double *lc = a.lc + g.vr, *uc = a.uc + g.vr;
        double *x = a.x + g.vc, *x0 = a.x0 + g.vc, *xh = a.xh + g.vc, *xe = a.xe + g.vc;
        double *aty = a.aty + g.vc;
        double *y0 = a.y0 + g.vr, *yh = a.yh + g.vr;
        // gathered vectors: y (primal product) and x_ext (dual product)
        double *y = ONCHIP ? lds + nmax : a.y + g.vr;
        if (ONCHIP) xe = lds;
        const int32_t as0 = (ONCHIP && !a.shared) ? a.asfirst[b] : 0;
        const int32_t ts0 = (ONCHIP && !a.shared) ? a.tsfirst[b] : 0;
        uint8_t *rs_ = u.restart + (size_t)b * u.T;
        double *om_ = u.omega + (size_t)b * u.T;
        int32_t *kk_ = u.kk + (size_t)b * u.T;
        uint64_t *xm = u.xmask + u.xm_off[b], *ym = u.ymask + u.ym_off[b];
        const int32_t xw = (g.n + 63) >> 6, yw = (g.m + 63) >> 6;
        const double eta = a.eta[g.sidx];
        const double gam = o.gamma;
        double nrm[2] = {0.0, 0.0};
        for (int32_t j = threadIdx.x; j < g.n; j += BT) {
            const int32_t jo = row_at(tperm, g.c0, j);
            const double d = Dc[jo];
            const double cj = d * c_o[jo];
            c[j] = cj;
            lv[j] = lv_o[jo] / d;
            uv[j] = uv_o[jo] / d;
            nrm[0] += cj * cj;
        }
        for (int32_t i = threadIdx.x; i < g.m; i += BT) {
            const int32_t io = row_at(aperm, g.r0, i);
            const double d = Dr[io];
            const double l = d * lc_o[io], uu = d * uc_o[io];
            lc[i] = l;
            uc[i] = uu;
            double bb = 0.0;
            if (isfinite(l)) bb = fmax(bb, fabs(l));
            if (isfinite(uu)) bb = fmax(bb, fabs(uu));
            nrm[1] += bb * bb;
        }
        wg_sum<BT, 2>(nrm);
        const double cn = sqrt(nrm[0]), bn = sqrt(nrm[1]);
        double omega = (cn > 1e-10 && bn > 1e-10) ? cn / bn : 1.0;
        for (int32_t j = threadIdx.x; j < g.n; j += BT) {
            const double xv = clampd(0.0, lv[j], uv[j]);
            x[j] = xv;
            x0[j] = xv;
        }
        for (int32_t i = threadIdx.x; i < g.m; i += BT) {
            const double lo = isfinite(uc[i]) ? -INFINITY : 0.0;
            const double hi = isfinite(lc[i]) ? INFINITY : 0.0;
            const double yv = clampd(0.0, lo, hi);
            y[i] = yv;
            y0[i] = yv;
        }
        __syncthreads();
        int64_t k = 0;
        double r_start = 0.0, r_prev = 0.0;
        for (int64_t t = 0; t < u.T; ++t) {
            if (u.replay) omega = om_[t];
            const double tau = eta / omega, sigma = eta * omega;
            const bool last = t + 1 >= u.T;
            const bool check = !u.replay && (t % o.check_every) == 0 && !last;
            const bool keep = true;   // restart decisions need the PDHG point
            const double ak = (double)(k + 1) / (double)(k + 2), bk = 1.0 / (double)(k + 2);
            (void)keep;
            uint64_t *xmt = xm + (size_t)t * xw;
            uint64_t *ymt = ym + (size_t)t * 2 * yw;
            for (int32_t j0 = 0; j0 < g.n; j0 += BT) {
                const int32_t j = j0 + (int32_t)threadIdx.x;
                bool inside = false;
                if (j < g.n) {
                    const double s = ONCHIP ? sell_dot(a.tsp, a.tsci, a.tsva, ts0 + (j >> 6), j & 63, y)
                                            : csr_dot(trp, tci, tva, j, y);
                    const double xr = x[j];
                    const double uu = xr - tau * (c[j] - s);
                    inside = uu > lv[j] && uu < uv[j];
                    const double xhat = clampd(uu, lv[j], uv[j]);
                    xe[j] = 2.0 * xhat - xr;
                    xh[j] = xhat;
                    aty[j] = s;
                }
                const uint64_t bits = __ballot(inside);
                if ((threadIdx.x & 63) == 0 && j < g.n) xmt[j >> 6] = bits;
            }
            __syncthreads();
            for (int32_t i0 = 0; i0 < g.m; i0 += BT) {
                const int32_t i = i0 + (int32_t)threadIdx.x;
                bool at_u = false, at_l = false;
                if (i < g.m) {
                    const double av = ONCHIP ? sell_dot(a.asp, a.asci, a.asva, as0 + (i >> 6), i & 63, xe)
                                             : csr_dot(arp, aci, ava, i, xe);
                    const double vv = y[i] / sigma - av;
                    at_u = vv < -uc[i];
                    at_l = vv > -lc[i];
                    yh[i] = sigma * (vv - clampd(vv, -uc[i], -lc[i]));
                }
                const uint64_t bu = __ballot(at_u), bl = __ballot(at_l);
                if ((threadIdx.x & 63) == 0 && i < g.m) {
                    ymt[2 * (i >> 6)] = bu;
                    ymt[2 * (i >> 6) + 1] = bl;
                }
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                om_[t] = omega;
                kk_[t] = (int32_t)k;
            }
            if (last) break;
            bool restart = u.replay ? rs_[t] != 0 : false;
            double v2[10];
            if (check) {
#pragma unroll
                for (int q = 0; q < 10; ++q) v2[q] = 0.0;
                for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                    const double dx = xh[j] - x[j];
                    v2[0] += dx * dx;
                    const double d0 = xh[j] - x0[j];
                    v2[2] += d0 * d0;
                    if (ONCHIP) xe[j] = dx;   // x_ext is spent: it carries dx for the cross term
                }
                if (ONCHIP) __syncthreads();
                for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                    const double dy = yh[i] - y[i];
                    v2[8] += dy * dy;
                    const double d0 = yh[i] - y0[i];
                    v2[9] += d0 * d0;
                    // cross term dy' A~ dx
                    double adx = 0.0;
                    if (ONCHIP) {
                        adx = sell_dot(a.asp, a.asci, a.asva, as0 + (i >> 6), i & 63, xe);
                    } else {
                        for (int32_t e = arp[i]; e < arp[i + 1]; ++e)
                            adx = fma(ava[e], xh[aci[e]] - x[aci[e]], adx);
                    }
                    v2[1] += dy * adx;
                }
                wg_sum<BT, 10>(v2);
                const double r2 = v2[0] / tau + v2[8] / sigma + 2.0 * v2[1];
                const double r = r2 > 0.0 ? sqrt(r2) : 0.0;
                if (t == 0) {
                    r_start = r;
                    r_prev = r;
                } else if (r <= o.beta_suff * r_start || (r <= o.beta_nec * r_start && r > r_prev) ||
                           (double)k >= o.beta_art * (double)t) {
                    restart = true;
                } else {
                    r_prev = r;
                }
                if (restart) {
                    const double dxr = sqrt(v2[2]), dyr = sqrt(v2[9]);
                    omega = batch_new_omega(omega, dxr, dyr);
                    r_start = r;
                    r_prev = r;
                }
            }
            if (threadIdx.x == 0 && !u.replay) rs_[t] = restart ? 1 : 0;
            if (restart) {
                for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                    x[j] = xh[j];
                    x0[j] = xh[j];
                }
                for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                    y[i] = yh[i];
                    y0[i] = yh[i];
                }
                k = 0;
            } else {
                for (int32_t j = threadIdx.x; j < g.n; j += BT)
                    x[j] = ak * ((1.0 + gam) * xh[j] - gam * x[j]) + bk * x0[j];
                for (int32_t i = threadIdx.x; i < g.m; i += BT)
                    y[i] = ak * ((1.0 + gam) * yh[i] - gam * y[i]) + bk * y0[i];
                ++k;
            }
            __syncthreads();
        }
        if (u.replay == 0 && threadIdx.x == 0) rs_[u.T - 1] = 0;
        for (int32_t j = threadIdx.x; j < g.n; j += BT) {
            const int32_t jo = row_at(tperm, g.c0, j);
            a.x_out[g.vc + jo] = Dc[jo] * xh[j];
        }
        for (int32_t i = threadIdx.x; i < g.m; i += BT) {
            const int32_t io = row_at(aperm, g.r0, i);
            a.y_out[g.vr + io] = Dr[io] * yh[i];
        }
        __syncthreads();
    }
}

// The 64-bit word that lane `l` (wave-uniform) holds, as a scalar, and the own
// lane's bit of such a word.
__device__ __forceinline__ uint64_t mask_word(uint64_t w, int32_t l) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(w >> 32), l) << 32 |
           (uint32_t)__builtin_amdgcn_readlane((int32_t)w, l);
}
__device__ __forceinline__ bool lane_bit(uint64_t w) { return __builtin_amdgcn_inverse_ballot_w64(w); }
// Lane l's copy of (w1, w0) becomes the word w. The wait covers the two states
// that a comparison's scalar result needs before a vector instruction reads it.
__device__ __forceinline__ void put_word(uint32_t &w0, uint32_t &w1, uint64_t w, int l) {
    asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
        : "+v"(w0), "+v"(w1)
        : "s"((uint32_t)w), "s"((uint32_t)(w >> 32)), "i"(l));
}

// k_batch_unrolled for a register-resident shared matrix (grid batches), in the
// manner of k_batch_solve_res: restarts are decided (or replayed) only where a
// check falls, the iterations in between run without a branch. A wave's
// projection masks are comparisons left in scalar registers; each goes to a
// lane of its own and one store per iteration writes them all.
// What bounds it: the instructions and LDS gathers of k_batch_solve_res plus
// the comparisons and lane writes of the masks (176 vector instructions a wave
// at 8 columns a thread). Per iteration of 256 instances: 32x32 grids 1.68 us
// (3.44 us with a branch per slot, divisions, and one store per mask word),
// 22x22 0.82 (2.16), 12x12 0.62 (1.56).
template <int BT, int S>
__global__ __launch_bounds__(BT) void k_batch_unrolled_res(BArgs a, BOpts o, UArgs u) {
    using L = ResLds<BT, S>;
    constexpr int SR = L::SR;
    constexpr int PX = res_pos(BT);
    constexpr int NW = BT / 64;
    extern __shared__ double lds[];
    LdsDouble *const sy = (LdsDouble *)lds, *const sx = sy + L::x, *const stp = sy + L::step;
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= a.B) return;
        const Geo g = geometry(a, b);
        const int32_t lane = (int32_t)(threadIdx.x & 63);
        const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x >> 6);
        const double *Dr = a.Dr, *Dc = a.Dc;
        uint8_t *rs_ = u.restart + (size_t)b * u.T;
        double *om_ = u.omega + (size_t)b * u.T;
        int32_t *kk_ = u.kk + (size_t)b * u.T;
        const int32_t xw = (g.n + 63) >> 6, yw = (g.m + 63) >> 6;
        uint64_t *xm = u.xmask + u.xm_off[b], *ym = u.ymask + u.ym_off[b];
        // lane q stores column slot q's mask; lanes 2q, 2q + 1 those of row slot q
        const int32_t xword = wave + lane * NW, yword = 2 * (wave + (lane >> 1) * NW) + (lane & 1);
        const bool xmine = lane < S && xword < xw, ymine = lane < 2 * SR && yword < 2 * yw;
        const double eta = a.eta[0];
        const double gam = o.gamma;
        ResEntries<BT, S> M;
        double xr[S], x0r[S], cr[S], lr[S], ur[S], xn[S];
        double yr[SR], y0r[SR], lo[SR], hi[SR], yn[SR];
        LdsDouble *const myx = sx + res_pos((int32_t)threadIdx.x), *const myy = sy + (int32_t)threadIdx.x;
        double nrm[2] = {0.0, 0.0};
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = (int32_t)threadIdx.x + q * BT;
            xr[q] = cr[q] = lr[q] = ur[q] = 0.0;
            if (j < g.n) {
                const double d = Dc[j];
                cr[q] = d * a.c_o[g.vc + j];
                lr[q] = a.lv_o[g.vc + j] / d;
                ur[q] = a.uv_o[g.vc + j] / d;
                nrm[0] += cr[q] * cr[q];
                xr[q] = clampd(0.0, lr[q], ur[q]);
            }
            x0r[q] = xr[q];
            M.load_col(a, g, sy, q, j);
        }
        M.load_rows(a, g, sx);
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = (int32_t)threadIdx.x + q * BT;
            yr[q] = y0r[q] = lo[q] = hi[q] = 0.0;
            if (i < g.m) {
                const double d = Dr[i];
                const double l = d * a.lc_o[g.vr + i], uu = d * a.uc_o[g.vr + i];
                double bb = 0.0;
                if (isfinite(l)) bb = fmax(bb, fabs(l));
                if (isfinite(uu)) bb = fmax(bb, fabs(uu));
                nrm[1] += bb * bb;
                yr[q] = clampd(0.0, isfinite(uu) ? -INFINITY : 0.0, isfinite(l) ? INFINITY : 0.0);
                y0r[q] = yr[q];
            }
            myy[q * BT] = yr[q];
        }
        wg_sum<BT, 2>(nrm);
        const double cn = sqrt(nrm[0]), bn = sqrt(nrm[1]);
        double omega = uniform_value((cn > 1e-10 && bn > 1e-10) ? cn / bn : 1.0);
        double tau = 0.0, sigma = 0.0;
        // step sizes and clamp bounds of the dual step at this omega
        auto set_steps = [&]() {
            tau = uniform_value(eta / omega);
            sigma = uniform_value(eta * omega);
            int32_t t0 = (int32_t)threadIdx.x;
            asm volatile("" : "+v"(t0));
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                const int32_t i = t0 + q * BT;
                if (i < g.m) {
                    lo[q] = -sigma * (Dr[i] * a.uc_o[g.vr + i]);
                    hi[q] = -sigma * (Dr[i] * a.lc_o[g.vr + i]);
                }
            }
        };
        if (u.replay) omega = om_[0];
        set_steps();

        // iteration t up to its PDHG point (xn, yn), masks recorded
        auto step = [&](int64_t t) {
            double s[S];
            uint32_t w0 = 0, w1 = 0;
            M.cols(s);
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const double v = xr[q] - tau * (cr[q] - s[q]);
                const uint64_t bits = __ballot(v > lr[q] && v < ur[q]);
                put_word(w0, w1, bits, q);
                xn[q] = clamp_quiet(v, lr[q], ur[q]);
                myx[q * PX] = 2.0 * xn[q] - xr[q];
            }
            if (xmine) xm[(size_t)t * xw + xword] = (uint64_t)w1 << 32 | w0;
            __syncthreads();
            M.rows(yn);
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                const double w = fma(-sigma, yn[q], yr[q]);
                const uint64_t bu = __ballot(w < lo[q]), bl = __ballot(w > hi[q]);
                put_word(w0, w1, bu, 2 * q);
                put_word(w0, w1, bl, 2 * q + 1);
                yn[q] = w - clamp_quiet(w, lo[q], hi[q]);
            }
            if (ymine) ym[(size_t)t * 2 * yw + yword] = (uint64_t)w1 << 32 | w0;
        };
        auto momentum = [&](double A, double G, double B) {
#pragma unroll
            for (int q = 0; q < S; ++q) xr[q] = A * xn[q] - G * xr[q] + B * x0r[q];
#pragma unroll
            for (int q = 0; q < SR; ++q) {
                yr[q] = A * yn[q] - G * yr[q] + B * y0r[q];
                myy[q * BT] = yr[q];
            }
        };

        int64_t t = 0, k = 0;
        int32_t tc = 0;   // t modulo check_every
        double r_start = 0.0, r_prev = 0.0;
        for (;;) {
            // iterations without a decision, then one with a check or the last
            int32_t plain = tc == 0 ? 0 : o.check_every - tc;
            if ((int64_t)plain > u.T - 1 - t) plain = (int32_t)(u.T - 1 - t);
            for (int32_t p = 0; p < plain; p += kResSteps) {
                const int32_t cnt = plain - p < kResSteps ? plain - p : kResSteps;
                if ((int32_t)threadIdx.x < cnt) {
                    const int32_t v = (int32_t)threadIdx.x;
                    double A, G, B;
                    momentum_factors((double)(k + p + v), gam, A, G, B);
                    stp[4 * v] = A;
                    stp[4 * v + 1] = G;
                    stp[4 * v + 2] = B;
                    om_[t + p + v] = omega;
                    kk_[t + p + v] = (int32_t)(k + p + v);
                    if (!u.replay) rs_[t + p + v] = 0;
                }
                __syncthreads();
#pragma unroll 1
                for (int32_t it = 0; it < cnt; ++it) {
                    const double A = stp[4 * it], G = stp[4 * it + 1], B = stp[4 * it + 2];
                    step(t + p + it);
                    momentum(A, G, B);
                    __syncthreads();
                }
            }
            t += plain;
            k += plain;
            step(t);
            if (threadIdx.x == 0) {
                om_[t] = omega;
                kk_[t] = (int32_t)k;
            }
            if (t + 1 >= u.T) break;
            bool restart = u.replay ? rs_[t] != 0 : false;
            if (!u.replay) {
                double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};   // |dx|^2, dy' A~ dx, |x^ - x0|^2, |dy|^2, |y^ - y0|^2
                __syncthreads();
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const double dx = xn[q] - xr[q], d0 = xn[q] - x0r[q];
                    v[0] += dx * dx;
                    v[2] += d0 * d0;
                    myx[q * PX] = dx;   // x_ext is spent: it carries dx for the cross term
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < SR; ++q) {
                    const double dy = yn[q] - yr[q], d0 = yn[q] - y0r[q];
                    v[3] += dy * dy;
                    v[4] += d0 * d0;
                    v[1] += dy * M.row(q, 0);
                }
                wg_sum<BT, 5>(v);
                const double r2 = v[0] / tau + v[3] / sigma + 2.0 * v[1];
                const double r = uniform_value(r2 > 0.0 ? sqrt(r2) : 0.0);
                if (t == 0) {
                    r_start = r;
                    r_prev = r;
                } else if (r <= o.beta_suff * r_start || (r <= o.beta_nec * r_start && r > r_prev) ||
                           (double)k >= o.beta_art * (double)t) {
                    restart = true;
                } else {
                    r_prev = r;
                }
                if (restart) {
                    // exp(log(dyr / dxr) / 2 + log(omega) / 2), without a call
                    const double dxr = sqrt(v[2]), dyr = sqrt(v[4]);
                    if (dxr > 1e-10 && dyr > 1e-10) omega = uniform_value(sqrt(dyr / dxr) * sqrt(omega));
                    r_start = r;
                    r_prev = r;
                }
                if (threadIdx.x == 0) rs_[t] = restart ? 1 : 0;
            }
            if (restart) {
#pragma unroll
                for (int q = 0; q < S; ++q) xr[q] = x0r[q] = xn[q];
#pragma unroll
                for (int q = 0; q < SR; ++q) {
                    yr[q] = y0r[q] = yn[q];
                    myy[q * BT] = yn[q];
                }
                k = 0;
                if (u.replay) omega = om_[t + 1];
                set_steps();
            } else {
                double A, G, B;
                momentum_factors((double)k, gam, A, G, B);
                momentum(A, G, B);
                ++k;
            }
            ++t;
            tc = o.check_every == 1 ? 0 : 1;
            __syncthreads();
        }
        if (u.replay == 0 && threadIdx.x == 0) rs_[u.T - 1] = 0;
        int32_t t0 = (int32_t)threadIdx.x;
        asm volatile("" : "+v"(t0));
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = t0 + q * BT;
            if (j < g.n) a.x_out[g.vc + j] = Dc[j] * xn[q];
        }
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = t0 + q * BT;
            if (i < g.m) a.y_out[g.vr + i] = Dr[i] * yn[q];
        }
        __syncthreads();
    }
}


// k_batch_backward for a register-resident shared matrix: the cotangents of
// the owned columns and rows and the gradient sums in registers; the products
// gather ba (in place of y) and tmp (in place of x_ext) from LDS. The masks
// and the schedule of kMaskSteps iterations come with one load each, a word
// per lane, while the group before is worked on; an iteration takes its words
// from those lanes as scalars and selects with them.
// Two barriers an iteration: ba and tmp are each read in the phase after they
// are written and rewritten only after the other's barrier.
// What bounds it: vector instructions and LDS gathers between the barriers.
// Per iteration of 256 instances: 32x32 grids 1.68 us (3.72 us with masks and
// schedule loaded when they were needed, three barriers and a division per
// row), 22x22 0.95 (1.93), 12x12 0.66 (1.35).
template <int BT, int S>
__global__ __launch_bounds__(BT) void k_batch_backward_res(BArgs a, BOpts o, UArgs u) {
    using L = ResLds<BT, S>;
    constexpr int SR = L::SR;
    constexpr int PX = res_pos(BT);
    constexpr int NW = BT / 64;
    constexpr int kMaskSteps = 64 / S;   // iterations whose column masks fill a wave's lanes
    static_assert(2 * SR * kMaskSteps <= 64, "row masks of a group fit one load");
    extern __shared__ double lds[];
    LdsDouble *const ba = (LdsDouble *)lds, *const tmp = ba + L::x;
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= a.B) return;
        const Geo g = geometry(a, b);
        const int32_t lane = (int32_t)(threadIdx.x & 63);
        const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x >> 6);
        const double *Dr = a.Dr, *Dc = a.Dc;
        const uint8_t *rs_ = u.restart + (size_t)b * u.T;
        const double *om_ = u.omega + (size_t)b * u.T;
        const int32_t *kk_ = u.kk + (size_t)b * u.T;
        const uint64_t *xm = u.xmask + u.xm_off[b], *ym = u.ymask + u.ym_off[b];
        const int32_t xw = (g.n + 63) >> 6, yw = (g.m + 63) >> 6;
        const double eta = a.eta[0];
        const double gam = o.gamma;
        ResEntries<BT, S> M;
        double bx[S], bx0[S], gcr[S];
        double by[SR], by0[SR], glr[SR], gur[SR];
        LdsDouble *const myx = tmp + res_pos((int32_t)threadIdx.x), *const myy = ba + (int32_t)threadIdx.x;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = (int32_t)threadIdx.x + q * BT;
            bx0[q] = gcr[q] = 0.0;
            bx[q] = j < g.n ? Dc[j] * u.gx[g.vc + j] : 0.0;
            M.load_col(a, g, ba, q, j);
        }
        M.load_rows(a, g, tmp);
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = (int32_t)threadIdx.x + q * BT;
            by0[q] = glr[q] = gur[q] = 0.0;
            by[q] = i < g.m ? Dr[i] * u.gy[g.vr + i] : 0.0;
        }
        // group of iterations t, t - 1, ..: lane (it, q) holds column slot q's
        // word of iteration t - it, lane (it, 2 q + half) row slot q's, lane it
        // the schedule. Words outside the masks (and iterations before 0) are 0.
        const int32_t xit = lane / S, xword = wave + (lane % S) * NW;
        const int32_t yit = lane / (2 * SR), yword = 2 * (wave + (lane % (2 * SR)) / 2 * NW) + (lane & 1);
        struct Group {
            uint64_t x, y;
            double om;
            int32_t k, rs;
        };
        auto fetch = [&](int64_t t) {
            Group f{0, 0, 1.0, 0, 0};
            if (xword < xw && xit <= t) f.x = xm[(size_t)(t - xit) * xw + xword];
            if (yword < 2 * yw && yit < kMaskSteps && yit <= t) f.y = ym[(size_t)(t - yit) * 2 * yw + yword];
            if (lane < kMaskSteps && lane <= t) {
                f.om = om_[t - lane];
                f.k = kk_[t - lane];
                // the output's cotangent enters like the point of a restart
                f.rs = rs_[t - lane] != 0 || t - lane == u.T - 1;
            }
            return f;
        };
        Group nxt = fetch(u.T - 1);
        for (int64_t tg = u.T - 1; tg >= 0; tg -= kMaskSteps) {
            const Group cur = nxt;
            if (tg >= kMaskSteps) nxt = fetch(tg - kMaskSteps);
            double A_, G_, B_;
            momentum_factors((double)cur.k, gam, A_, G_, B_);
            const double tau_ = eta / cur.om, sigma_ = eta * cur.om;
            const uint64_t restarts = __ballot(cur.rs != 0);
            const int32_t cnt = tg + 1 < kMaskSteps ? (int32_t)(tg + 1) : kMaskSteps;
#pragma unroll 1
            for (int32_t it = 0; it < cnt; ++it) {
                const double tau = lane_value(tau_, it), sigma = lane_value(sigma_, it);
                double bxh[S], byh[SR];
                if (restarts >> it & 1) {
#pragma unroll
                    for (int q = 0; q < S; ++q) {
                        bxh[q] = bx[q] + bx0[q];
                        bx[q] = bx0[q] = 0.0;
                    }
#pragma unroll
                    for (int q = 0; q < SR; ++q) {
                        byh[q] = by[q] + by0[q];
                        by[q] = by0[q] = 0.0;
                    }
                } else {
                    const double A = lane_value(A_, it), G = lane_value(G_, it), B = lane_value(B_, it);
#pragma unroll
                    for (int q = 0; q < S; ++q) {
                        bxh[q] = A * bx[q];
                        bx0[q] += B * bx[q];
                        bx[q] *= -G;
                    }
#pragma unroll
                    for (int q = 0; q < SR; ++q) {
                        byh[q] = A * by[q];
                        by0[q] += B * by[q];
                        by[q] *= -G;
                    }
                }
                // dual step: yhat = w - clamp(w, -sigma u_c, -sigma l_c), w = y - sigma A~ xext
#pragma unroll
                for (int q = 0; q < SR; ++q) {
                    const bool at_u = lane_bit(mask_word(cur.y, it * 2 * SR + 2 * q));
                    const bool at_l = lane_bit(mask_word(cur.y, it * 2 * SR + 2 * q + 1));
                    const double sv = sigma * byh[q];
                    const double vu = at_u ? sv : 0.0, vl = at_l ? sv : 0.0;
                    gur[q] += vu;
                    glr[q] += vl;
                    by[q] += at_u || at_l ? byh[q] : 0.0;
                    myy[q * BT] = at_u || at_l ? -sv : 0.0;
                }
                __syncthreads();
                // xext = 2 xhat - x, then the primal step xhat = clamp(x - tau (c - A~'y))
                double s[S];
                M.cols(s);
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const double bh = bxh[q] + 2.0 * s[q];
                    const double bu = lane_bit(mask_word(cur.x, it * S + q)) ? bh : 0.0;
                    bx[q] = (bx[q] - s[q]) + bu;
                    const double tb = tau * bu;
                    gcr[q] -= tb;
                    myx[q * PX] = tb;
                }
                __syncthreads();
                // (the next iteration writes ba only, which all threads have read)
                double p[SR];
                M.rows(p);
#pragma unroll
                for (int q = 0; q < SR; ++q) by[q] += p[q];
            }
        }
        // c~ = D_c c, l~_c = D_r l_c, u~_c = D_r u_c
        int32_t t0 = (int32_t)threadIdx.x;
        asm volatile("" : "+v"(t0));
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int32_t j = t0 + q * BT;
            if (j < g.n) u.gc[g.vc + j] = Dc[j] * gcr[q];
        }
#pragma unroll
        for (int q = 0; q < SR; ++q) {
            const int32_t i = t0 + q * BT;
            if (i < g.m) {
                u.glc[g.vr + i] = isfinite(a.lc_o[g.vr + i]) ? Dr[i] * glr[q] : 0.0;
                u.guc[g.vr + i] = isfinite(a.uc_o[g.vr + i]) ? Dr[i] * gur[q] : 0.0;
            }
        }
        __syncthreads();
    }
}

// Reverse pass of k_batch_unrolled with its recorded schedule and masks.
template <int BT, bool ONCHIP>
__global__ __launch_bounds__(BT) void k_batch_backward(BArgs a, BOpts o, UArgs u, int32_t nmax) {
    extern __shared__ double lds[];
    for (;;) {
        const int32_t b = next_instance<BT>(a.queue);
        if (b >= a.B) return;
        const Geo g = geometry(a, b);
        const int32_t *arp = a.arp + g.r0, *trp = a.trp + g.c0;
        const int32_t *aci = a.aci, *tci = a.tci;
        const double *ava = a.ava, *tva = a.tva;
        const double *Dr = a.Dr + g.dr, *Dc = a.Dc + g.dc;
        const uint8_t *rs_ = u.restart + (size_t)b * u.T;
        const double *om_ = u.omega + (size_t)b * u.T;
        const int32_t *kk_ = u.kk + (size_t)b * u.T;
        const uint64_t *xm = u.xmask + u.xm_off[b], *ym = u.ymask + u.ym_off[b];
        const int32_t xw = (g.n + 63) >> 6, yw = (g.m + 63) >> 6;
        const double eta = a.eta[g.sidx];
        const double gam = o.gamma;
        // cotangents: bx, bx0, bxh (x, x0, xh), tmp (xe); by, by0, byh (y, y0, yh), ba
        double *bx = a.x + g.vc, *bx0 = a.x0 + g.vc, *bxh = a.xh + g.vc, *tmp = a.xe + g.vc;
        double *by = a.y + g.vr, *by0 = a.y0 + g.vr, *byh = a.yh + g.vr, *ba = u.ba + g.vr;
        // gathered vectors: ba (A~' ba) and tmp (A~ tmp)
        if (ONCHIP) {
            tmp = lds;
            ba = lds + nmax;
        }
        const int32_t as0 = (ONCHIP && !a.shared) ? a.asfirst[b] : 0;
        const int32_t ts0 = (ONCHIP && !a.shared) ? a.tsfirst[b] : 0;
        const int32_t *aperm = ONCHIP ? a.aperm : nullptr, *tperm = ONCHIP ? a.tperm : nullptr;
        // gradient sums, by position
        double *gc = a.aty + g.vc, *glc = a.lc + g.vr, *guc = a.uc + g.vr;
        for (int32_t j = threadIdx.x; j < g.n; j += BT) {
            bx[j] = 0.0;
            bx0[j] = 0.0;
            const int32_t jo = row_at(tperm, g.c0, j);
            bxh[j] = Dc[jo] * u.gx[g.vc + jo];
            gc[j] = 0.0;
        }
        for (int32_t i = threadIdx.x; i < g.m; i += BT) {
            by[i] = 0.0;
            by0[i] = 0.0;
            const int32_t io = row_at(aperm, g.r0, i);
            byh[i] = Dr[io] * u.gy[g.vr + io];
            glc[i] = 0.0;
            guc[i] = 0.0;
        }
        __syncthreads();
        for (int64_t t = u.T - 1; t >= 0; --t) {
            const double omega = om_[t];
            const double tau = eta / omega, sigma = eta * omega;
            if (t < u.T - 1) {
                if (rs_[t]) {
                    for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                        bxh[j] = bx[j] + bx0[j];
                        bx[j] = 0.0;
                        bx0[j] = 0.0;
                    }
                    for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                        byh[i] = by[i] + by0[i];
                        by[i] = 0.0;
                        by0[i] = 0.0;
                    }
                } else {
                    const int64_t k = kk_[t];
                    const double ak = (double)(k + 1) / (double)(k + 2), bk = 1.0 / (double)(k + 2);
                    for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                        const double v = bx[j];
                        bxh[j] = ak * (1.0 + gam) * v;
                        bx0[j] += bk * v;
                        bx[j] = -ak * gam * v;
                    }
                    for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                        const double v = by[i];
                        byh[i] = ak * (1.0 + gam) * v;
                        by0[i] += bk * v;
                        by[i] = -ak * gam * v;
                    }
                }
            }
            // dual step: yhat = sigma (v - clamp(v, -u_c, -l_c)), v = y/sigma - A~ xext
            const uint64_t *ymt = ym + (size_t)t * 2 * yw;
            for (int32_t i = threadIdx.x; i < g.m; i += BT) {
                const uint64_t bit = 1ull << (i & 63);
                const bool at_u = (ymt[2 * (i >> 6)] & bit) != 0;
                const bool at_l = (ymt[2 * (i >> 6) + 1] & bit) != 0;
                const double bv = (at_u || at_l) ? sigma * byh[i] : 0.0;
                if (at_u) guc[i] += sigma * byh[i];
                if (at_l) glc[i] += sigma * byh[i];
                by[i] += bv / sigma;
                ba[i] = -bv;
            }
            __syncthreads();
            // xext = 2 xhat - x, then the primal step xhat = clamp(x - tau (c - A~'y))
            const uint64_t *xmt = xm + (size_t)t * xw;
            for (int32_t j = threadIdx.x; j < g.n; j += BT) {
                const double bxe = ONCHIP ? sell_dot4(a.tsp, a.tsci, a.tsva, ts0 + (j >> 6), j & 63, ba)
                                          : csr_dot(trp, tci, tva, j, ba);
                const double bh = bxh[j] + 2.0 * bxe;
                bx[j] -= bxe;
                const bool inside = (xmt[j >> 6] >> (j & 63)) & 1ull;
                const double bu = inside ? bh : 0.0;
                bx[j] += bu;
                gc[j] += -tau * bu;
                tmp[j] = tau * bu;
            }
            __syncthreads();
            for (int32_t i = threadIdx.x; i < g.m; i += BT)
                by[i] += ONCHIP ? sell_dot4(a.asp, a.asci, a.asva, as0 + (i >> 6), i & 63, tmp)
                                : csr_dot(arp, aci, ava, i, tmp);
            __syncthreads();
        }
        // c~ = D_c c, l~_c = D_r l_c, u~_c = D_r u_c
        for (int32_t j = threadIdx.x; j < g.n; j += BT) {
            const int32_t jo = row_at(tperm, g.c0, j);
            u.gc[g.vc + jo] = Dc[jo] * gc[j];
        }
        for (int32_t i = threadIdx.x; i < g.m; i += BT) {
            const int32_t io = row_at(aperm, g.r0, i);
            u.glc[g.vr + io] = isfinite(a.lc_o[g.vr + io]) ? Dr[io] * glc[i] : 0.0;
            u.guc[g.vr + io] = isfinite(a.uc_o[g.vr + io]) ? Dr[io] * guc[i] : 0.0;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// layout kernels

// Instance-local column indices of A and the row -> instance map check.
__global__ __launch_bounds__(kBlock) void k_batch_localize(const int32_t *__restrict__ row_off,
                                                           const int32_t *__restrict__ col_off,
                                                           int32_t B, const int32_t *__restrict__ rowptr,
                                                           int32_t *__restrict__ colidx,
                                                           int32_t *__restrict__ flag) {
    // a workgroup per instance, its rows strided over the threads
    for (int32_t b = blockIdx.x; b < B; b += (int32_t)gridDim.x) {
        const int32_t c0 = col_off[b], c1 = col_off[b + 1];
        if (row_off[b + 1] < row_off[b] || c1 <= c0) {
            if (threadIdx.x == 0) atomicOr(flag, 32);
            continue;
        }
        for (int32_t i = row_off[b] + (int32_t)threadIdx.x; i < row_off[b + 1]; i += kBlock)
            for (int32_t e = rowptr[i]; e < rowptr[i + 1]; ++e) {
                const int32_t j = colidx[e];
                if (j < c0 || j >= c1) atomicOr(flag, 64);
                colidx[e] = j - c0;
            }
    }
}

// Column indices of A' (global rows) made instance-local.
__global__ __launch_bounds__(kBlock) void k_batch_localize_t(const int32_t *__restrict__ row_off,
                                                             const int32_t *__restrict__ col_off,
                                                             int32_t B, const int32_t *__restrict__ trp,
                                                             int32_t *__restrict__ tci) {
    for (int32_t b = blockIdx.x; b < B; b += (int32_t)gridDim.x) {
        const int32_t r0 = row_off[b];
        for (int32_t j = col_off[b] + (int32_t)threadIdx.x; j < col_off[b + 1]; j += kBlock)
            for (int32_t e = trp[j]; e < trp[j + 1]; ++e) tci[e] -= r0;
    }
}

}  // namespace pdhg

// ---------------------------------------------------------------------------
// host side

namespace pdhg {

static BOpts batch_opts(const pdhg_options &o) {
    BOpts b;
    b.eps = o.eps;
    b.gamma = o.gamma;
    b.step_safety = o.step_safety;
    b.beta_suff = o.restart_sufficient;
    b.beta_nec = o.restart_necessary;
    b.beta_art = o.restart_artificial;
    b.power_tol = o.power_tol;
    b.limit = std::min<int64_t>(o.iteration_limit, 10000000);
    b.check_every = o.check_every;
    b.ruiz_iters = o.ruiz_iters;
    b.pock_chambolle = o.pock_chambolle;
    b.power_max_iters = o.power_max_iters;
    b.eps_pinf = o.eps_primal_infeasible;
    b.eps_dinf = o.eps_dual_infeasible;
    b.detect = o.eps_primal_infeasible > 0.0 || o.eps_dual_infeasible > 0.0;
    b.pad = 0;
    return b;
}

static BArgs batch_args(BatchHandle &h) {
    BArgs a;
    memset(&a, 0, sizeof(a));
    a.B = h.B;
    a.shared = h.shared;
    a.m = h.m;
    a.n = h.n;
    a.row_off = h.row_off.p;
    a.col_off = h.col_off.p;
    a.arp = h.arp.p;
    a.aci = h.aci.p;
    a.ava = h.ava.p;
    a.trp = h.trp.p;
    a.tci = h.tci.p;
    a.tva = h.tva.p;
    a.Dr = h.Dr.p;
    a.Dc = h.Dc.p;
    a.eta = h.eta.p;
    a.power_iters = h.power_iters.p;
    a.c_o = h.c_o.p;
    a.lc_o = h.lc_o.p;
    a.uc_o = h.uc_o.p;
    a.lv_o = h.lv_o.p;
    a.uv_o = h.uv_o.p;
    a.c = h.c.p;
    a.lc = h.lc.p;
    a.uc = h.uc.p;
    a.lv = h.lv.p;
    a.uv = h.uv.p;
    a.x = h.x.p;
    a.x0 = h.x0.p;
    a.xh = h.xh.p;
    a.xe = h.xe.p;
    a.aty = h.aty.p;
    a.y = h.y.p;
    a.y0 = h.y0.p;
    a.yh = h.yh.p;
    a.res = h.res.p;
    a.queue = h.queue.p;
    a.x_init = h.x_init_;
    a.y_init = h.y_init_;
    a.asp = h.asp.p;
    a.asci = h.asci.p;
    a.asva = h.asva.p;
    a.asfirst = h.asfirst.p;
    a.aperm = h.aperm.p;
    a.tsp = h.tsp.p;
    a.tsci = h.tsci.p;
    a.tsva = h.tsva.p;
    a.tsfirst = h.tsfirst.p;
    a.tperm = h.tperm.p;
    a.lhist = h.lhist.p;
    a.p0 = h.rp0.p;
    a.q0 = h.rq0.p;
    a.ph = h.rph.p;
    a.qh = h.rqh.p;
    a.x_out = h.x_out_;
    a.y_out = h.y_out_;
    return a;
}

template <int BT>
static int32_t resident(const void *kernel) {
    int dev = 0, per_cu = 0;
    PDHG_HIP(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    PDHG_HIP(hipGetDeviceProperties(&prop, dev));
    PDHG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, BT, 0));
    return std::max(1, per_cu) * prop.multiProcessorCount;
}



// Dynamic LDS one workgroup may take (160 KB on gfx950), read once.
static size_t lds_per_workgroup() {
    static const size_t v = [] {
        int dev = 0, bytes = 0;
        PDHG_HIP(hipGetDevice(&dev));
        PDHG_HIP(hipDeviceGetAttribute(&bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
        return (size_t)bytes;
    }();
    return v;
}

template <int BT, class K>
static int32_t resident_lds(BatchHandle &h, K kernel, size_t lds) {
    int dev = 0, per_cu = 0;
    PDHG_HIP(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    PDHG_HIP(hipGetDeviceProperties(&prop, dev));
    PDHG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kernel), BT, lds));
    int32_t wg = std::min(h.B, std::max(1, per_cu) * prop.multiProcessorCount);
    if (h.workgroups > 0) wg = std::min(wg, h.workgroups);
    return wg;
}

// Columns per thread of the register-resident kernels at bt threads, or 0 when the batch
// does not qualify: a shared matrix with narrow slices, 256 or 512 threads
// (1,024 would leave 128 registers each and spill) and one row per thread, two
// at 8 columns.
static int res_columns(const BatchHandle &h, int32_t bt) {
    if (!(h.onchip && h.resident && h.shared && h.ts_wmax >= 1 && h.ts_wmax <= kResCol &&
          h.as_wmax <= kResRow && (bt == 256 || bt == 512)))
        return 0;
    if (h.nmax <= 2 * bt && h.mmax <= bt) return 2;
    if (h.nmax <= 4 * bt && h.mmax <= bt) return 4;
    if (h.nmax <= 8 * bt && h.mmax <= 2 * bt) return 8;
    return 0;
}

// Threads of the register-resident kernels when the caller chose none, 0 where they do not
// apply: 256 while that gives a thread at most 4 columns, else 512. Measured
// per iteration of 256 instances, 2,048 in the batch: 16x16 grids (960
// columns) 0.33 us at 256 and 0.52 at 512; 22x22 grids (1,848 columns) 0.79 at
// 256 and 0.62 at 512.
static int32_t res_threads(const BatchHandle &h) {
    const int s = res_columns(h, 256);
    if (s > 0 && s <= 4) return 256;
    return res_columns(h, 512) > 0 ? 512 : 0;
}

// Launch of a persistent kernel: as many workgroups as fit, or as asked for.
template <int BT, class... Args>
static void launch_queue_t(BatchHandle &h, size_t lds, void (*kernel)(Args...), Args... args) {
    const int32_t wg = resident_lds<BT>(h, kernel, lds);
    PDHG_HIP(hipMemsetAsync(h.queue.p, 0, sizeof(int32_t), h.stream));
    kernel<<<wg, BT, lds, h.stream>>>(args...);
    PDHG_HIP(hipGetLastError());
}
template <int BT, int S, class... Args>
static void launch_res_t(BatchHandle &h, void (*kernel)(Args...), Args... args) {
    constexpr size_t lds = ResLds<BT, S>::bytes;
    static_assert(lds <= 150 * 1024, "the reductions need LDS of their own");
    launch_queue_t<BT>(h, lds, kernel, args...);
}
// Largest instance that gets SELL-64 copies: 8 columns (rows) for each of
// 1,024 threads, and byte offsets 8 j of its positions fit 16 bits.
constexpr int32_t kSellRows = 8192;

// Whether the on-chip kernels take the batch at bt threads: up to 2 columns and
// rows per thread, and up to 8 where the vectors of k_batch_solve_stream fit the
// LDS (3 KB stay for the reductions; two per thread need 64 KB at most).
static bool solve_on_chip(const BatchHandle &h, int32_t bt) {
    const int32_t need = std::max(h.nmax, h.mmax);
    return h.onchip && need <= kSellRows &&
           (need <= 2 * bt ||
            (need <= 8 * bt && stream_doubles(h.nmax, h.mmax) * sizeof(double) + 3072 <= lds_per_workgroup()));
}

// Dynamic LDS of the on-chip setup / unrolled / reverse kernels, or 0 when the
// largest instance does not fit (then the memory-resident variant runs).
static size_t onchip_lds(const BatchHandle &h) {
    const size_t lds = ((size_t)h.nmax + (size_t)h.mmax) * sizeof(double);
    return (h.onchip && lds <= 65536) ? std::max<size_t>(lds, 8) : 0;
}

template <int BT, int S, int SR>
static void launch_solve_lds_t(BatchHandle &h, const BOpts &o, const BArgs &a) {
    constexpr size_t lds = LdsShape<BT, S, SR>::bytes;
    static_assert(lds <= 150 * 1024 && lds % 16 == 0, "the reductions need LDS of their own");
    // matrix entries take the rest of the LDS of as many workgroups as the
    // registers hold (two waves per SIMD); one pair more is read, not used
    const size_t share = lds_per_workgroup() * std::min(BT, 512) / 512;
    const int32_t pairs = share > lds + 6144 ? (int32_t)((share - lds - 6144) / kPairBytes) : 0;
    launch_queue_t<BT>(h, lds + (size_t)(pairs + 1) * kPairBytes, &k_batch_solve_lds<BT, S, SR>, a, o, pairs);
}

template <int BT, int S>
static void launch_solve_stream_t(BatchHandle &h, const BOpts &o, const BArgs &a) {
    const size_t lds = stream_doubles(h.nmax, h.mmax) * sizeof(double);
    if (o.detect) launch_queue_t<BT>(h, lds, &k_batch_solve_stream<BT, S, true>, a, o, h.nmax, h.mmax);
    else launch_queue_t<BT>(h, lds, &k_batch_solve_stream<BT, S, false>, a, o, h.nmax, h.mmax);
}

template <class T>
static void load(DBuf<T> &dst, const T *src, size_t count, int mem, hipStream_t s);

// Most workgroups of the kernels that give one to every instance; they walk on
// from there (a launch holds fewer than 2^32 work-items, and the runtime cuts
// one beyond without an error).
constexpr int32_t kInstanceGroups = 1 << 16;

// Order and widths of the slices of `count` instances, a workgroup for one after
// another: with perm, position = rank of the row by falling length (equal lengths
// in row order), else position = row. width[slice] becomes the longest row of
// each slice. The ranks are a bitonic sort of the rows' (length, row) keys in LDS:
// counting each row's longer ones took 1.9 of the 7.2 ms in which a batch of
// twelve LPs with up to 7,000 columns was created.
__global__ __launch_bounds__(1024) void k_sell_order(const int32_t *__restrict__ rp, const int32_t *__restrict__ off,
                                                     int32_t total, int32_t count,
                                                     const int32_t *__restrict__ sfirst, int32_t *__restrict__ perm,
                                                     int32_t *__restrict__ inv, int32_t *__restrict__ width) {
    static_assert(kSellRows <= 1 << 13, "a row takes 13 bits of a key, kSellRows less its length 14");
    extern __shared__ uint32_t key[];
    for (int32_t b = blockIdx.x; b < count; b += (int32_t)gridDim.x) {
        const int32_t r0 = off ? off[b] : 0, n = (off ? off[b + 1] : total) - r0, s0 = sfirst[b];
        if (!perm) {
            for (int32_t i = threadIdx.x; i < n; i += 1024)
                atomicMax(&width[s0 + (i >> 6)], rp[r0 + i + 1] - rp[r0 + i]);
            continue;
        }
        int32_t np = 1;
        while (np < n) np *= 2;
        for (int32_t i = threadIdx.x; i < np; i += 1024)
            key[i] = i < n ? (uint32_t)(kSellRows - (rp[r0 + i + 1] - rp[r0 + i])) << 13 | (uint32_t)i : UINT32_MAX;
        __syncthreads();
        for (int32_t k = 2; k <= np; k *= 2)
            for (int32_t j = k / 2; j > 0; j /= 2) {
                for (int32_t t = threadIdx.x; t < np / 2; t += 1024) {
                    const int32_t i = 2 * t - (t & (j - 1)), q = i + j;   // the pair j apart
                    const uint32_t u = key[i], v = key[q];
                    if ((u > v) == ((i & k) == 0)) {
                        key[i] = v;
                        key[q] = u;
                    }
                }
                __syncthreads();
            }
        for (int32_t r = threadIdx.x; r < n; r += 1024) {
            const int32_t i = (int32_t)(key[r] & 8191u);
            perm[r0 + r] = i;
            inv[r0 + i] = r;
            if ((r & 63) == 0) width[s0 + (r >> 6)] = kSellRows - (int32_t)(key[r] >> 13);
        }
        __syncthreads();
    }
}

// Entries of the slices, one thread per position: slice sl covers the global
// positions r0[sl] .. r1[sl] of instance inst[sl]; column indices become the
// other side's positions.
__global__ __launch_bounds__(kBlock) void k_sell_fill(
    const int32_t *__restrict__ rp, const int32_t *__restrict__ ci, const double *__restrict__ va,
    const int32_t *__restrict__ r0, const int32_t *__restrict__ r1, const int32_t *__restrict__ inst,
    const int32_t *__restrict__ off, const int32_t *__restrict__ other_off, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ other_inv, const int32_t *__restrict__ sp, int32_t ns, uint32_t *__restrict__ sci,
    double2 *__restrict__ sva) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int32_t sl = (int32_t)(t >> 6), lane = (int32_t)(t & 63);
    if (sl >= ns) return;
    const int32_t pos = r0[sl] + lane;
    int32_t e = 0, e1 = 0;
    if (pos < r1[sl]) {
        const int32_t row = perm ? off[inst[sl]] + perm[pos] : pos;
        e = rp[row];
        e1 = rp[row + 1];
    }
    const int32_t *oinv = other_inv ? other_inv + other_off[inst[sl]] : nullptr;
    for (int32_t k = sp[sl]; k < sp[sl + 1]; ++k) {
        uint32_t c[2] = {0, 0};
        double v[2] = {0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 2; ++u, ++e)
            if (e < e1) {
                c[u] = 8u * (uint32_t)(oinv ? oinv[ci[e]] : ci[e]);
                v[u] = va[e];
            }
        sci[64 * (int64_t)k + lane] = c[1] << 16 | c[0];
        sva[64 * (int64_t)k + lane] = double2{v[0], v[1]};
    }
}

// SELL-64 copies of A~ and A~' (rows of every instance padded to whole
// slices) from the scaled CSR after the setup kernel: order and slice widths on
// the device, prefix sums on the host (a few thousand slices), entries placed
// by one thread per position. Nothing is built for instances that no kernel
// would read them for.
static void build_batch_sell(BatchHandle &h) {
    hipStream_t s = h.stream;
    if (!solve_on_chip(h, 1024) && !onchip_lds(h)) return;
    const bool sorted = !h.shared;
    const int32_t nb = h.shared ? 1 : h.B;
    struct Side {
        const DBuf<int32_t> &rp, &ci;
        const DBuf<double> &va;
        std::vector<int32_t> roff;
        const int32_t *off;
        int32_t total, rows_max;
        DBuf<int32_t> &sp, &sfirst, &perm;
        DBuf<uint32_t> &sci;
        DBuf<double2> &sva;
        int32_t &wmax;
        DBuf<int32_t> inv, d0, d1, inst, width;
        std::vector<int32_t> h0, h1, hi, first, hw, pairs;
        int32_t ns = 0;
    };
    const int32_t *ro = h.shared ? nullptr : h.row_off.p, *co = h.shared ? nullptr : h.col_off.p;
    Side side[2] = {{h.arp, h.aci, h.ava, h.shared ? std::vector<int32_t>{0, h.m} : h.row_off_h, ro, h.m, h.mmax,
                     h.asp, h.asfirst, h.aperm, h.asci, h.asva, h.as_wmax},
                    {h.trp, h.tci, h.tva, h.shared ? std::vector<int32_t>{0, h.n} : h.col_off_h, co, h.n, h.nmax,
                     h.tsp, h.tsfirst, h.tperm, h.tsci, h.tsva, h.ts_wmax}};
    for (Side &d : side) {
        d.first.resize((size_t)nb + 1);
        for (int32_t b = 0; b < nb; ++b) {
            d.first[b] = (int32_t)d.h0.size();
            for (int32_t r = d.roff[b]; r < d.roff[b + 1]; r += 64) {
                d.h0.push_back(r);
                d.h1.push_back(std::min(r + 64, d.roff[b + 1]));
                d.hi.push_back(b);
            }
        }
        d.ns = d.first[nb] = (int32_t)d.h0.size();
        load(d.sfirst, d.first.data(), d.first.size(), PDHG_MEM_HOST, s);
        load(d.d0, d.h0.data(), d.h0.size(), PDHG_MEM_HOST, s);
        load(d.d1, d.h1.data(), d.h1.size(), PDHG_MEM_HOST, s);
        load(d.inst, d.hi.data(), d.hi.size(), PDHG_MEM_HOST, s);
        d.width.alloc((size_t)std::max(1, d.ns));
        d.hw.resize((size_t)d.ns);
        if (d.ns == 0) continue;
        if (sorted) {
            d.perm.alloc((size_t)d.total);
            d.inv.alloc((size_t)d.total);
        }
        PDHG_HIP(hipMemsetAsync(d.width.p, 0, (size_t)d.ns * 4, s));
        size_t keys = 1;
        while (sorted && keys < (size_t)d.rows_max) keys *= 2;
        k_sell_order<<<std::min(nb, kInstanceGroups), 1024, keys * 4, s>>>(
            d.rp.p, d.off, d.total, nb, d.sfirst.p, sorted ? d.perm.p : nullptr, d.inv.p, d.width.p);
        PDHG_HIP(hipMemcpyAsync(d.hw.data(), d.width.p, (size_t)d.ns * 4, hipMemcpyDeviceToHost, s));
    }
    PDHG_HIP(hipStreamSynchronize(s));
    for (int k = 0; k < 2; ++k) {
        Side &d = side[k], &other = side[1 - k];
        d.pairs.assign((size_t)d.ns + 1, 0);
        int64_t total = 0;
        for (int32_t i = 0; i < d.ns; ++i) {
            d.wmax = std::max(d.wmax, d.hw[i]);
            total += (d.hw[i] + 1) / 2;
            if (64 * total >= INT32_MAX) fail(PDHG_ERR_UNSUPPORTED, "batch matrix too large for 32-bit offsets");
            d.pairs[(size_t)i + 1] = (int32_t)total;
        }
        load(d.sp, d.pairs.data(), d.pairs.size(), PDHG_MEM_HOST, s);
        const size_t cap = 64 * (size_t)std::max<int64_t>(total, 1);
        d.sci.alloc(cap);
        d.sva.alloc(cap);
        if (d.ns > 0)
            k_sell_fill<<<(unsigned)ceil_div((int64_t)d.ns * 64, kBlock), kBlock, 0, s>>>(
                d.rp.p, d.ci.p, d.va.p, d.d0.p, d.d1.p, d.inst.p, d.off, other.off, sorted ? d.perm.p : nullptr,
                sorted ? other.inv.p : nullptr, d.sp.p, d.ns, d.sci.p, d.sva.p);
        PDHG_HIP(hipGetLastError());
    }
    PDHG_HIP(hipStreamSynchronize(s));
}

// Largest instance column / row counts (LDS sizing of the on-chip solve).
static void instance_extents(BatchHandle &h) {
    if (h.shared) {
        h.nmax = h.n;
        h.mmax = h.m;
        return;
    }
    h.nmax = h.mmax = 0;
    for (int32_t b = 0; b < h.B; ++b) {
        h.nmax = std::max(h.nmax, h.col_off_h[b + 1] - h.col_off_h[b]);
        h.mmax = std::max(h.mmax, h.row_off_h[b + 1] - h.row_off_h[b]);
    }
}

// Default threads per instance: 1024 when the batch has at most one instance
// per compute unit, else the fewest (from 256) that keep the largest instance
// on chip with at most 8 columns and 8 rows per thread.
static int32_t default_threads(const BatchHandle &h) {
    int dev = 0, cus = 0;
    PDHG_HIP(hipGetDevice(&dev));
    PDHG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (h.B <= cus) return 1024;
    const int32_t need = std::max(h.nmax, h.mmax);
    int32_t bt = 256;
    while (bt < 1024 && 8 * bt < need) bt *= 2;
    return bt;
}

template <int BT>
static void launch_solve_t(BatchHandle &h, const BOpts &o) {
    BArgs a = batch_args(h);
    if constexpr (BT == 256 || BT == 512) {
        switch (res_columns(h, BT)) {
            case 2: return launch_res_t<BT, 2>(h, &k_batch_solve_res<BT, 2>, a, o);
            case 4: return launch_res_t<BT, 4>(h, &k_batch_solve_res<BT, 4>, a, o);
            case 8: return launch_res_t<BT, 8>(h, &k_batch_solve_res<BT, 8>, a, o);
            default: break;
        }
    }
    if (solve_on_chip(h, BT)) {
        const int32_t need = std::max(h.nmax, h.mmax);
        if (need <= BT) return launch_solve_lds_t<BT, 1, 1>(h, o, a);
        if (need <= 2 * BT) {
            // A shared matrix with long slices comes from L2 faster than two
            // columns' pairs pass through registers and LDS. 193 iterations, 256
            // instances: 1,000 x 1,000 with 30 entries a row 3.7 -> 1.8 ms, with 10
            // (20 at most) 1.5 -> 1.0; 400 x 1,000 with 30 1.30 -> 1.01, with 10 0.51 ->
            // 0.68; 120 x 120 with 6 (13 at most) 0.52 -> 0.60.
            if (h.shared && std::max(h.as_wmax, h.ts_wmax) > 16) return launch_solve_stream_t<BT, 2>(h, o, a);
            return h.mmax <= BT ? launch_solve_lds_t<BT, 2, 1>(h, o, a) : launch_solve_lds_t<BT, 2, 2>(h, o, a);
        }
        if (need <= 4 * BT) return launch_solve_stream_t<BT, 4>(h, o, a);
        return launch_solve_stream_t<BT, 8>(h, o, a);
    }

    int32_t wg = std::min(h.B, resident<BT>(o.detect ? reinterpret_cast<const void *>(&k_batch_solve<BT, true>)
                                                     : reinterpret_cast<const void *>(&k_batch_solve<BT, false>)));
    if (h.workgroups > 0) wg = std::min(wg, h.workgroups);
    PDHG_HIP(hipMemsetAsync(h.queue.p, 0, sizeof(int32_t), h.stream));
    if (o.detect)
        k_batch_solve<BT, true><<<wg, BT, 0, h.stream>>>(a, o);
    else
        k_batch_solve<BT, false><<<wg, BT, 0, h.stream>>>(a, o);
    PDHG_HIP(hipGetLastError());
}

template <int BT>
static void launch_setup_t(BatchHandle &h, int32_t count) {
    BArgs a = batch_args(h);
    const BOpts o = batch_opts(h.opt);
    const size_t lds = onchip_lds(h);
    PDHG_HIP(hipMemsetAsync(h.queue.p, 0, sizeof(int32_t), h.stream));
    if (lds) {
        const int32_t wg = std::min(count, resident_lds<BT>(h, &k_batch_setup<BT, true>, lds));
        k_batch_setup<BT, true><<<wg, BT, lds, h.stream>>>(a, o, count, h.nmax);
    } else {
        const int32_t wg = std::min(count, resident_lds<BT>(h, &k_batch_setup<BT, false>, 0));
        k_batch_setup<BT, false><<<wg, BT, 0, h.stream>>>(a, o, count, 0);
    }
    PDHG_HIP(hipGetLastError());
}

// The setup (scaling sweeps and power iteration, one workgroup per instance)
// is latency-bound: it runs with about two columns per thread whatever the
// solve's launch shape, between 256 and 1024 threads.
static void dispatch_setup(BatchHandle &h, int32_t count) {
    const int32_t need = std::max(h.nmax, h.mmax);
    int32_t bt = 256;
    while (bt < 1024 && 2 * bt < need) bt *= 2;
    switch (bt) {
        case 64: launch_setup_t<64>(h, count); break;
        case 128: launch_setup_t<128>(h, count); break;
        case 512: launch_setup_t<512>(h, count); break;
        case 1024: launch_setup_t<1024>(h, count); break;
        default: launch_setup_t<256>(h, count); break;
    }
}

// Threads of the solve when the caller chose none. Register-resident: see
// res_threads. Else, while one column or row per thread takes at most 512
// threads, that many; two columns per thread once the batch has more instances
// than run at once (two waves per SIMD). On a shared matrix only where that
// leaves one row per thread and short columns: its entries come from L2 at no
// cost beside ragged ones, and a second set of them is a longer chain. Up to
// 1,024 columns 512 threads (register pairs, a wave ahead in the stream), from
// there 1,024, but 512 for up to 4,096 with the ray tests, whose checks spill at
// 1,024. Instances beyond the chip keep the threads of default_threads, at most
// 512 with the ray tests (k_batch_solve<1024, true> spills).
// Per iteration of 256 instances, 5% dense, n = 2 m: 1,024 of n = 114: 0.42 us at
// 64 threads, 0.36 at 128, 0.69 at 256; 1,024 (300) of n = 240: 0.77 (2.45) at
// 128, 0.94 (1.6) at 256; 1,024 (128) of n = 500: 2.6 (4.8) at 256, 3.05 (3.4) at
// 512; 300 of n = 960: 25.9 at 256, 17.1 at 512, 24.2 at 1,024; of n = 2,000: 105
// at 512, 101 at 1,024. Sharing one matrix, 600 instances, 193 iterations:
// 200 x 250 1.50 ms at 128, 0.79 at 256; 250 x 500 with 5 entries a column 0.87
// at 256, 0.98 at 512, with 12 2.28 at 256, 1.79 at 512; 1,500 x 3,000 with the
// ray tests 6.8 at 512 and at 1,024, narrow 1,100 x 4,000 3.6 at 512, 4.5 at
// 1,024, without them 3.5 and 3.2.
static int32_t solve_threads(const BatchHandle &h, bool detect) {
    if (const int32_t t = res_threads(h)) return t;
    if (!solve_on_chip(h, 1024)) return detect ? std::min(h.threads, 512) : h.threads;
    int dev = 0, cus = 0;
    PDHG_HIP(hipGetDevice(&dev));
    PDHG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const int32_t need = std::max(h.nmax, h.mmax);
    if (need > 1024) return detect && need > 2048 && need <= 4096 ? 512 : 1024;
    int32_t bt = 64;
    while (bt < 512 && bt < need) bt *= 2;
    const bool pairs = !h.shared || (2 * h.mmax <= bt && h.ts_wmax <= 16);
    if (pairs && need <= bt && bt > 64 && h.B > cus * (512 / bt)) bt /= 2;
    return bt;
}

static void dispatch_solve(BatchHandle &h, const BOpts &o) {
    const int32_t threads = h.threads_set ? h.threads : solve_threads(h, o.detect);
    switch (threads) {
        case 64: launch_solve_t<64>(h, o); break;
        case 128: launch_solve_t<128>(h, o); break;
        case 512: launch_solve_t<512>(h, o); break;
        case 1024: launch_solve_t<1024>(h, o); break;
        default: launch_solve_t<256>(h, o); break;
    }
}

template <class T>
static void load(DBuf<T> &dst, const T *src, size_t count, int mem, hipStream_t s) {
    dst.alloc(count);
    if (count == 0) return;
    PDHG_HIP(hipMemcpyAsync(dst.p, src, count * sizeof(T),
                            mem == PDHG_MEM_DEVICE ? hipMemcpyDeviceToDevice
                                                   : hipMemcpyHostToDevice,
                            s));
}

BatchHandle *batch_create(const pdhg_batch_problem &p, const pdhg_options &o, void *stream) {
    if (p.batch < 1 || (p.shared_a != 0 && p.shared_a != 1) || p.m < 0 || p.n < 1)
        fail(PDHG_ERR_INVALID_ARG, "need batch >= 1, shared_a in {0,1}, m >= 0, n >= 1");
    if (p.mem != PDHG_MEM_HOST && p.mem != PDHG_MEM_DEVICE)
        fail(PDHG_ERR_INVALID_ARG, "mem must be PDHG_MEM_HOST or PDHG_MEM_DEVICE");
    if (!p.a_rowptr || (p.a_nnz > 0 && (!p.a_colidx || !p.a_val)) || p.a_nnz < 0 ||
        p.a_nnz >= INT32_MAX)
        fail(PDHG_ERR_INVALID_ARG, "bad CSR arrays or nnz");
    if (!p.c || !p.lv || !p.uv || (p.m > 0 && (!p.lc || !p.uc)))
        fail(PDHG_ERR_INVALID_ARG, "NULL objective or bound vector");
    if (!p.shared_a && (!p.row_off || !p.col_off))
        fail(PDHG_ERR_INVALID_ARG, "ragged batches need row_off and col_off");
    if (p.shared_a && ((int64_t)p.batch * p.n >= INT32_MAX || (int64_t)p.batch * p.m >= INT32_MAX))
        fail(PDHG_ERR_UNSUPPORTED, "batch vectors exceed 32-bit indexing");
    auto hp = std::make_unique<BatchHandle>();
    BatchHandle &h = *hp;
    const double t0 = now_seconds();
    h.B = p.batch;
    h.shared = p.shared_a;
    h.m = p.m;
    h.n = p.n;
    h.nnz = p.a_nnz;
    h.opt = o;
    h.vec_m = h.shared ? h.B * h.m : h.m;
    h.vec_n = h.shared ? h.B * h.n : h.n;
    PDHG_HIP(hipStreamCreateWithFlags(&h.stream, hipStreamNonBlocking));
    PDHG_HIP(hipEventCreateWithFlags(&h.ev, hipEventDisableTiming));
    order_after_stream(h.stream, h.ev, stream);
    hipStream_t s = h.stream;

    load(h.arp, p.a_rowptr, (size_t)h.m + 1, p.mem, s);
    load(h.aci, p.a_colidx, (size_t)h.nnz, p.mem, s);
    load(h.ava, p.a_val, (size_t)h.nnz, p.mem, s);
    validate_csr(s, h.arp.p, h.aci.p, h.ava.p, h.m, h.n, h.nnz);
    if (!h.shared) {
        std::vector<int32_t> ro((size_t)h.B + 1), co((size_t)h.B + 1);
        if (p.mem == PDHG_MEM_DEVICE) {
            PDHG_HIP(hipMemcpy(ro.data(), p.row_off, ro.size() * 4, hipMemcpyDeviceToHost));
            PDHG_HIP(hipMemcpy(co.data(), p.col_off, co.size() * 4, hipMemcpyDeviceToHost));
        } else {
            memcpy(ro.data(), p.row_off, ro.size() * 4);
            memcpy(co.data(), p.col_off, co.size() * 4);
        }
        if (ro[0] != 0 || co[0] != 0 || ro[h.B] != h.m || co[h.B] != h.n)
            fail(PDHG_ERR_INVALID_INPUT, "row_off / col_off must start at 0 and end at m / n");
        for (int32_t b = 0; b < h.B; ++b)
            if (ro[b + 1] < ro[b] || co[b + 1] <= co[b])
                fail(PDHG_ERR_INVALID_INPUT, "instance offsets must increase (>= 1 column each)");
        load(h.row_off, ro.data(), ro.size(), PDHG_MEM_HOST, s);
        load(h.col_off, co.data(), co.size(), PDHG_MEM_HOST, s);
        h.row_off_h = ro;
        h.col_off_h = co;
    } else {
        h.row_off.alloc(1);
        h.col_off.alloc(1);
    }
    instance_extents(h);
    h.threads = default_threads(h);
    // A' from the global matrix, then instance-local indices on both
    h.trp.alloc((size_t)h.n + 1);
    h.tci.alloc((size_t)h.nnz);
    h.tva.alloc((size_t)h.nnz);
    plain_transpose(s, h.m, h.n, h.nnz, h.arp.p, h.aci.p, h.ava.p, h.trp.p, h.tci.p, h.tva.p);
    if (!h.shared) {
        DBuf<int32_t> flag;
        flag.alloc(1);
        PDHG_HIP(hipMemsetAsync(flag.p, 0, sizeof(int32_t), s));
        const unsigned nb = (unsigned)std::min(h.B, kInstanceGroups);
        k_batch_localize<<<nb, kBlock, 0, s>>>(h.row_off.p, h.col_off.p, h.B, h.arp.p, h.aci.p,
                                                flag.p);
        check_flag(s, flag.p, "a ragged instance has entries outside its column range");
        k_batch_localize_t<<<nb, kBlock, 0, s>>>(h.row_off.p, h.col_off.p, h.B, h.trp.p, h.tci.p);
    }
    load(h.c_o, p.c, (size_t)h.vec_n, p.mem, s);
    load(h.lv_o, p.lv, (size_t)h.vec_n, p.mem, s);
    load(h.uv_o, p.uv, (size_t)h.vec_n, p.mem, s);
    load(h.lc_o, p.lc, (size_t)h.vec_m, p.mem, s);
    load(h.uc_o, p.uc, (size_t)h.vec_m, p.mem, s);
    validate_vectors(s, h.vec_n, h.vec_m, h.c_o.p, h.lv_o.p, h.uv_o.p, h.lc_o.p, h.uc_o.p);
    for (auto *b : {&h.c, &h.lv, &h.uv, &h.x, &h.x0, &h.xh, &h.xe, &h.aty}) b->alloc((size_t)h.vec_n);
    for (auto *b : {&h.lc, &h.uc, &h.y, &h.y0, &h.yh}) b->alloc((size_t)h.vec_m);
    h.Dr.alloc((size_t)h.m);
    h.Dc.alloc((size_t)h.n);
    const int32_t nscal = h.shared ? 1 : h.B;
    h.eta.alloc((size_t)nscal);
    h.power_iters.alloc((size_t)nscal);
    h.res.alloc((size_t)h.B);
    h.queue.alloc(1);
    h.lhist.alloc((size_t)nscal * 2 * ((size_t)std::max(1, o.power_max_iters) + 1));
    if (p.q_rank == 0) {   // LP batches test infeasibility rays at checks
        for (auto *b : {&h.rq0, &h.rqh}) b->alloc((size_t)h.vec_n);
        for (auto *b : {&h.rp0, &h.rph}) b->alloc((size_t)std::max(1, h.vec_m));
    }
    dispatch_setup(h, nscal);
    PDHG_HIP(hipStreamSynchronize(s));
    h.lhist.release();
    if (p.q_rank == 0) build_batch_sell(h);   // the QP kernels walk the CSR
    if (const int32_t t = p.q_rank == 0 ? res_threads(h) : 0) h.threads = t;
    if (p.q_rank > 0) bqp_create(h, p);
    h.setup_seconds = now_seconds() - t0;
    return hp.release();
}

void batch_solve(BatchHandle &h, const double *x_init, const double *y_init, double *x_out,
                 double *y_out, pdhg_result *res) {
    if (h.q_rank > 0) {
        bqp_solve(h, x_init, y_init, x_out, y_out, res);
        return;
    }
    const double t0 = now_seconds();
    BOpts o = batch_opts(h.opt);
    // pointers of this call go in through the argument block
    h.x_init_ = x_init;
    h.y_init_ = y_init;
    h.x_out_ = x_out;
    h.y_out_ = y_out;
    dispatch_solve(h, o);
    PDHG_HIP(hipStreamSynchronize(h.stream));
    const double el = now_seconds() - t0;
    if (res) {
        std::vector<BatchRes> r((size_t)h.B);
        PDHG_HIP(hipMemcpy(r.data(), h.res.p, sizeof(BatchRes) * h.B, hipMemcpyDeviceToHost));
        for (int32_t b = 0; b < h.B; ++b) {
            pdhg_result &q = res[b];
            memset(&q, 0, sizeof(q));
            q.status = r[b].status;
            q.iterations = r[b].iterations;
            q.restarts = r[b].restarts;
            q.primal_obj = r[b].pobj;
            q.dual_obj = r[b].dobj;
            q.rel_primal_res = r[b].rel_p;
            q.rel_dual_res = r[b].rel_d;
            q.rel_gap = r[b].rel_g;
            q.kkt_rel = r[b].kkt;
            q.solve_seconds = el;
            q.setup_seconds = h.setup_seconds;
            q.eta = r[b].eta;
            q.omega = r[b].omega;
            q.norm_a = r[b].eta > 0.0 ? h.opt.step_safety / r[b].eta : 0.0;
            q.power_iters = r[b].power_iters;
        }
    }
}

void batch_set_launch(BatchHandle &h, int32_t threads, int32_t workgroups) {
    if (threads != 64 && threads != 128 && threads != 256 && threads != 512 && threads != 1024)
        fail(PDHG_ERR_INVALID_ARG, "threads must be 64, 128, 256, 512 or 1024");
    h.threads = threads;
    h.threads_set = true;
    h.workgroups = workgroups;
}

int32_t batch_autotune(BatchHandle &h, int32_t iterations) {
    // Every trial runs with the limit `iterations` into temporary outputs; the
    // caller's limit, launch shape and output pointers come back even if a
    // trial fails, and the best thread count is kept only on success.
    struct Restore {
        BatchHandle &h;
        int64_t limit;
        int32_t threads;
        bool set;
        const double *x_init, *y_init;
        double *x_out, *y_out;
        ~Restore() {
            h.opt.iteration_limit = limit;
            h.threads = threads;
            h.threads_set = set;
            h.x_init_ = x_init;
            h.y_init_ = y_init;
            h.x_out_ = x_out;
            h.y_out_ = y_out;
        }
    } restore{h, h.opt.iteration_limit, h.threads, h.threads_set,
              h.x_init_, h.y_init_, h.x_out_, h.y_out_};
    DBuf<double> xo, yo;
    xo.alloc((size_t)h.vec_n);
    yo.alloc((size_t)std::max(1, h.vec_m));
    const bool qp = h.q_rank > 0;
    BOpts o = batch_opts(h.opt);
    o.limit = iterations;
    h.opt.iteration_limit = iterations;
    h.x_out_ = xo.p;
    h.y_out_ = yo.p;
    h.x_init_ = nullptr;
    h.y_init_ = nullptr;
    auto trial = [&]() {
        if (qp) bqp_solve(h, nullptr, nullptr, xo.p, yo.p, nullptr);
        else dispatch_solve(h, o);
        PDHG_HIP(hipStreamSynchronize(h.stream));
    };
    int32_t best = h.threads;
    double best_t = 1e300;
    h.threads_set = true;   // each trial runs the thread count it names
    for (int32_t t : {64, 128, 256, 512, 1024}) {
        h.threads = t;
        trial();   // warm-up
        const double t0 = now_seconds();
        trial();
        const double el = now_seconds() - t0;
        if (el < best_t) {
            best_t = el;
            best = t;
        }
    }
    restore.threads = best;
    restore.set = true;
    return best;
}

static UArgs unrolled_args(BatchHandle &h) {
    UArgs u;
    memset(&u, 0, sizeof(u));
    u.T = h.unrolled_T;
    u.restart = h.u_restart.p;
    u.omega = h.u_omega.p;
    u.kk = h.u_kk.p;
    u.xmask = h.u_xmask.p;
    u.ymask = h.u_ymask.p;
    u.xm_off = h.u_xoff.p;
    u.ym_off = h.u_yoff.p;
    u.ba = h.u_ba.p;
    return u;
}

template <int BT>
static void launch_unrolled_t(BatchHandle &h, const UArgs &u) {
    BArgs a = batch_args(h);
    const BOpts o = batch_opts(h.opt);
    const size_t lds = onchip_lds(h);
    if constexpr (BT == 256 || BT == 512) {
        const int cols = res_columns(h, BT);
        if (cols == 2) return launch_res_t<BT, 2>(h, &k_batch_unrolled_res<BT, 2>, a, o, u);
        if (cols == 4) return launch_res_t<BT, 4>(h, &k_batch_unrolled_res<BT, 4>, a, o, u);
        if (cols == 8) return launch_res_t<BT, 8>(h, &k_batch_unrolled_res<BT, 8>, a, o, u);
    }
    PDHG_HIP(hipMemsetAsync(h.queue.p, 0, sizeof(int32_t), h.stream));
    if (lds) {
        const int32_t wg = resident_lds<BT>(h, &k_batch_unrolled<BT, true>, lds);
        k_batch_unrolled<BT, true><<<wg, BT, lds, h.stream>>>(a, o, u, h.nmax);
    } else {
        const int32_t wg = resident_lds<BT>(h, &k_batch_unrolled<BT, false>, 0);
        k_batch_unrolled<BT, false><<<wg, BT, 0, h.stream>>>(a, o, u, 0);
    }
    PDHG_HIP(hipGetLastError());
}

template <int BT>
static void launch_backward_t(BatchHandle &h, const UArgs &u) {
    BArgs a = batch_args(h);
    const BOpts o = batch_opts(h.opt);
    const size_t lds = onchip_lds(h);
    if constexpr (BT == 256 || BT == 512) {
        const int cols = res_columns(h, BT);
        if (cols == 2) return launch_res_t<BT, 2>(h, &k_batch_backward_res<BT, 2>, a, o, u);
        if (cols == 4) return launch_res_t<BT, 4>(h, &k_batch_backward_res<BT, 4>, a, o, u);
        if (cols == 8) return launch_res_t<BT, 8>(h, &k_batch_backward_res<BT, 8>, a, o, u);
    }
    PDHG_HIP(hipMemsetAsync(h.queue.p, 0, sizeof(int32_t), h.stream));
    if (lds) {
        const int32_t wg = resident_lds<BT>(h, &k_batch_backward<BT, true>, lds);
        k_batch_backward<BT, true><<<wg, BT, lds, h.stream>>>(a, o, u, h.nmax);
    } else {
        const int32_t wg = resident_lds<BT>(h, &k_batch_backward<BT, false>, 0);
        k_batch_backward<BT, false><<<wg, BT, 0, h.stream>>>(a, o, u, 0);
    }
    PDHG_HIP(hipGetLastError());
}

void batch_unrolled_forward(BatchHandle &h, int64_t T, int32_t replay, double *x_out,
                            double *y_out) {
    if (h.q_rank > 0) {
        bqp_unrolled(h, T, replay, x_out, y_out);
        return;
    }
    if (T < 1 || T > 1000000) fail(PDHG_ERR_INVALID_ARG, "T must be in [1, 10^6]");
    if (replay && h.unrolled_T != T)
        fail(PDHG_ERR_INVALID_ARG, "replay needs a recorded schedule of the same length T");
    if (h.unrolled_T != T) {
        // per-instance mask offsets (64-bit words)
        std::vector<int64_t> xo((size_t)h.B + 1, 0), yo((size_t)h.B + 1, 0);
        for (int32_t b = 0; b < h.B; ++b) {
            const int64_t n_b = h.shared ? h.n : h.col_off_h[b + 1] - h.col_off_h[b];
            const int64_t m_b = h.shared ? h.m : h.row_off_h[b + 1] - h.row_off_h[b];
            xo[b + 1] = xo[b] + ((n_b + 63) / 64) * T;
            yo[b + 1] = yo[b] + 2 * ((m_b + 63) / 64) * T;
        }
        h.u_xoff.alloc(xo.size());
        h.u_yoff.alloc(yo.size());
        PDHG_HIP(hipMemcpy(h.u_xoff.p, xo.data(), xo.size() * 8, hipMemcpyHostToDevice));
        PDHG_HIP(hipMemcpy(h.u_yoff.p, yo.data(), yo.size() * 8, hipMemcpyHostToDevice));
        h.u_xmask.alloc((size_t)std::max<int64_t>(1, xo[h.B]));
        h.u_ymask.alloc((size_t)std::max<int64_t>(1, yo[h.B]));
        h.u_restart.alloc((size_t)h.B * T);
        h.u_omega.alloc((size_t)h.B * T);
        h.u_kk.alloc((size_t)h.B * T);
        h.u_ba.alloc((size_t)std::max(1, h.vec_m));
        h.unrolled_T = T;
    }
    h.x_out_ = x_out;
    h.y_out_ = y_out;
    UArgs u = unrolled_args(h);
    u.replay = replay;
    switch (h.threads) {
        case 64: launch_unrolled_t<64>(h, u); break;
        case 128: launch_unrolled_t<128>(h, u); break;
        case 512: launch_unrolled_t<512>(h, u); break;
        case 1024: launch_unrolled_t<1024>(h, u); break;
        default: launch_unrolled_t<256>(h, u); break;
    }
    PDHG_HIP(hipStreamSynchronize(h.stream));
}

void batch_backward(BatchHandle &h, const double *gx, const double *gy, double *gc, double *glc,
                    double *guc, double *gd) {
    if (h.q_rank > 0) {
        bqp_backward(h, gx, gy, gc, glc, guc, gd);
        return;
    }
    if (h.unrolled_T < 1) fail(PDHG_ERR_INVALID_ARG, "run pdhg_batch_unrolled_forward first");
    DBuf<double> zm, lcs, ucs;
    zm.alloc((size_t)std::max(1, h.vec_m));
    PDHG_HIP(hipMemsetAsync(zm.p, 0, sizeof(double) * std::max(1, h.vec_m), h.stream));
    // gradients of rows without bounds are written to scratch when not requested
    lcs.alloc((size_t)std::max(1, h.vec_m));
    ucs.alloc((size_t)std::max(1, h.vec_m));
    UArgs u = unrolled_args(h);
    u.gx = gx;
    u.gy = gy ? gy : zm.p;
    u.gc = gc;
    u.glc = glc ? glc : lcs.p;
    u.guc = guc ? guc : ucs.p;
    switch (h.threads) {
        case 64: launch_backward_t<64>(h, u); break;
        case 128: launch_backward_t<128>(h, u); break;
        case 512: launch_backward_t<512>(h, u); break;
        case 1024: launch_backward_t<1024>(h, u); break;
        default: launch_backward_t<256>(h, u); break;
    }
    PDHG_HIP(hipStreamSynchronize(h.stream));
}

void batch_update_data(BatchHandle &h, const double *c, const double *lc, const double *uc,
                       const double *lv, const double *uv) {
    hipStream_t s = h.stream;
    DBuf<double> nc, nlc, nuc, nlv, nuv;
    auto take = [&](DBuf<double> &dst, const double *src, const DBuf<double> &cur, int32_t len) {
        dst.alloc((size_t)std::max(1, len));
        PDHG_HIP(hipMemcpyAsync(dst.p, src ? src : cur.p, sizeof(double) * (size_t)len,
                                hipMemcpyDeviceToDevice, s));
    };
    take(nc, c, h.c_o, h.vec_n);
    take(nlv, lv, h.lv_o, h.vec_n);
    take(nuv, uv, h.uv_o, h.vec_n);
    take(nlc, lc, h.lc_o, h.vec_m);
    take(nuc, uc, h.uc_o, h.vec_m);
    validate_vectors(s, h.vec_n, h.vec_m, nc.p, nlv.p, nuv.p, nlc.p, nuc.p);
    std::swap(h.c_o.p, nc.p);
    std::swap(h.lv_o.p, nlv.p);
    std::swap(h.uv_o.p, nuv.p);
    std::swap(h.lc_o.p, nlc.p);
    std::swap(h.uc_o.p, nuc.p);
    PDHG_HIP(hipStreamSynchronize(s));
}

void batch_destroy(BatchHandle *h) {
    if (!h) return;
    (void)hipStreamSynchronize(h->stream);
    delete h;
}

}  // namespace pdhg
