// Device-side helpers shared by the kernels: row mapping of the binned CSR
// layout, lane-group dot products and deterministic workgroup sums.
#pragma once

#include "common.hpp"

namespace pdhg {

constexpr int kSellUnroll = 8;   // SELL-64 entries whose loads are in flight together

// Cross-lane moves on the vector unit. A __shfl_xor of a double is two LDS-pipe
// permutes of about a hundred cycles each, one after another in a butterfly;
// these are a few cycles. In the descending order 32, 16, 8, 4, 2, 1 the
// partner sums below equal the xor butterfly's bit for bit: the swaps pair
// lanes i and i ^ 32 (i ^ 16), and a rotation by 8, 4, 2 or 1 inside a row of
// 16 lanes reads lane i ^ 8 (4, 2, 1) once the values repeat with period 16
// (8, 4, 2).
struct Pair {
    double a, b;
};
// Lanes 32..63 of a change places with lanes 0..31 of b.
__device__ __forceinline__ Pair swap32(double a, double b) {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return Pair{__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1])};
}
// Lanes 16..31 and 48..63 of a change places with lanes 0..15 and 32..47 of b.
__device__ __forceinline__ Pair swap16(double a, double b) {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return Pair{__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1])};
}
// The value of another lane of the row of 16 (a DPP control word).
constexpr int kDppRor = 0x120;          // + n: rotate by n
constexpr int kDppXor1 = 0xB1;          // quad permutations [1, 0, 3, 2] and [2, 3, 0, 1]
constexpr int kDppXor2 = 0x4E;
constexpr int kDppHalfMirror = 0x141;   // lane 7 - i of each 8
constexpr int kDppMirror = 0x140;       // lane 15 - i of each 16
template <int CTRL>
__device__ __forceinline__ double dpp_get(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// v of lane `lane` (wave-uniform) as a scalar.
__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// op over the lanes of each aligned group of L = 2^lg lanes, in every lane of
// the group, smallest distance first (a mirror reads lane i ^ 4, or i ^ 8, of
// values that are equal over quads, or over eights).
template <class Op>
__device__ __forceinline__ double group_reduce(double v, int32_t lg, Op op) {
    if (lg > 0) v = op(v, dpp_get<kDppXor1>(v));
    if (lg > 1) v = op(v, dpp_get<kDppXor2>(v));
    if (lg > 2) v = op(v, dpp_get<kDppHalfMirror>(v));
    if (lg > 3) v = op(v, dpp_get<kDppMirror>(v));
    if (lg > 4) {
        const Pair p = swap16(v, v);
        v = op(p.a, p.b);
    }
    if (lg > 5) {
        const Pair p = swap32(v, v);
        v = op(p.a, p.b);
    }
    return v;
}

struct RowCtx {
    int32_t row;
    int32_t lg;    // log2(lanes per row)
    bool valid;    // row exists
    bool lead;     // first lane of the row's lane group
};

// Workgroup blockIdx.x belongs to the last segment whose block_begin <= it.
__device__ __forceinline__ RowCtx row_ctx(const SegTable &T) {
    const int32_t b = blockIdx.x;
    int32_t si = 0;
#pragma unroll 1
    for (int32_t q = 1; q < T.nseg; ++q) si = (b >= T.s[q].block_begin) ? q : si;
    const int32_t lg = T.s[si].lanes_log2;
    RowCtx r;
    r.lg = lg;
    r.row = T.s[si].row_begin + (b - T.s[si].block_begin) * (kBlock >> lg) +
            (int32_t)(threadIdx.x >> lg);
    r.valid = r.row < T.s[si].row_end;
    r.lead = (threadIdx.x & ((1u << lg) - 1u)) == 0u;
    return r;
}

// A matrix entry: non-temporal where the matrices are streamed (HMat::stream).
template <bool NT, class T>
__device__ __forceinline__ T load_entry(const T *__restrict__ p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// The entry `step` past e, or the last of the `left` entries from e on. Formed from
// what is left: e + step may exceed 32 bits at the end of a matrix.
__host__ __device__ constexpr int32_t entry_at(int32_t e, int32_t left, int32_t step) {
    return e + (step < left ? step : left - 1);
}
static_assert(entry_at(INT32_MAX - 3, 3, 7 * 64) == INT32_MAX - 1 && entry_at(INT32_MAX - 99, 99, 64) == INT32_MAX - 35,
              "no overflow among the last entries");

// acc + the products of the lane's entries e, e + L, ..., in that order, U at a
// time: as in sell_group the U loads of a group are unconditional, at indices
// clamped to the row's last entry, so that all of them (and then their gathers)
// are in flight before the first product, and products past the row are dropped
// by a select. One entry at a time, a 2,000-entry column cost its lanes 31
// dependent round trips.
template <int U, bool NT>
__device__ __forceinline__ double lane_entries_dot(const int32_t *__restrict__ colidx,
                                                   const double *__restrict__ val,
                                                   const double *__restrict__ v, int32_t e, int32_t e1,
                                                   int32_t L) {
    double acc = 0.0;
    for (int32_t left = e1 - e; left > 0; left -= U * L, e = (int32_t)((uint32_t)e + (uint32_t)(U * L))) {
        int32_t c[U];
        double a[U], x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t q = entry_at(e, left, u * L);
            c[u] = load_entry<NT>(colidx + q);
            a[u] = load_entry<NT>(val + q);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = v[c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double t = fma(a[u], x[u], acc);
            acc = u * L < left ? t : acc;
        }
    }
    return acc;
}

// sum_e val[e] * v[colidx[e]] over the row, lanes strided; the lane-group
// butterfly leaves the same total in every lane of the group. Rows of at most
// 64 lanes x 4 entries have 2 to 4 entries per lane (make_segments).
template <bool NT>
__device__ __forceinline__ double row_dot(const int32_t *__restrict__ rowptr,
                                          const int32_t *__restrict__ colidx,
                                          const double *__restrict__ val,
                                          const double *__restrict__ v, const RowCtx &rc) {
    double acc = 0.0;
    const int32_t L = 1 << rc.lg;
    if (rc.valid) {
        const int32_t lane = (int32_t)(threadIdx.x & (uint32_t)(L - 1));
        const int32_t e = rowptr[rc.row] + lane, e1 = rowptr[rc.row + 1];
        if (e1 - e <= 4 * L) acc = lane_entries_dot<4, NT>(colidx, val, v, e, e1, L);
        else acc = lane_entries_dot<8, NT>(colidx, val, v, e, e1, L);
    }
    return group_reduce(acc, rc.lg, [](double p, double q) { return p + q; });
}

// Row reduction of |val| (max when MAXNORM, else sum) without a vector.
template <bool MAXNORM>
__device__ __forceinline__ double row_absnorm(const int32_t *__restrict__ rowptr,
                                              const double *__restrict__ val, const RowCtx &rc) {
    double acc = 0.0;
    const int32_t L = 1 << rc.lg;
    if (rc.valid) {
        const int32_t lane = (int32_t)(threadIdx.x & (uint32_t)(L - 1));
        const int32_t e1 = rowptr[rc.row + 1];
        for (int32_t e = rowptr[rc.row] + lane; e < e1; e += L) {
            const double a = fabs(val[e]);
            acc = MAXNORM ? fmax(acc, a) : acc + a;
        }
    }
    return group_reduce(acc, rc.lg, [](double p, double q) { return MAXNORM ? fmax(p, q) : p + q; });
}

struct RowSum {
    double s;
    int32_t row;
    bool valid;   // this thread owns an existing row and holds its full sum
};

// Index of the SELL-64 slice handled by this wave (wave-uniform), or -1 when
// the workgroup belongs to the long-row part.
__device__ __forceinline__ int32_t slice_of(const MatView &M) {
    if ((int32_t)blockIdx.x < M.seg.nblocks) return -1;
    return ((int32_t)blockIdx.x - M.seg.nblocks) * (kBlock / 64) + (int32_t)(threadIdx.x >> 6);
}

// acc + the products of entries [k, k + U) of a SELL-64 lane whose row has w
// entries (entry e at ci[64 e], va[64 e]; k < w, wave-uniform), in entry
// order. The loads are unconditional at indices clamped to the last entry, so
// the compiler issues all of them before the first product (with predicated
// loads it waits on each in turn); products of entries past w are dropped by a
// select, so the sum is exactly that of the entries < w.
template <int U, bool NT, class Idx, class Gather>
__device__ __forceinline__ double sell_group(const Idx *__restrict__ ci,
                                             const double *__restrict__ va, int32_t k,
                                             int32_t w, double acc, Gather gather) {
    int32_t c[U];
    double a[U], xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int32_t e = 64 * min(k + u, w - 1);
        c[u] = (int32_t)load_entry<NT>(ci + e);
        a[u] = load_entry<NT>(va + e);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = gather(c[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const double t = fma(a[u], xv[u], acc);
        acc = (k + u < w) ? t : acc;
    }
    return acc;
}

// Sum of the w entries of a SELL-64 lane in entry order: groups of
// kSellUnroll, then one tail group of 1, 2, 4 or kSellUnroll (w is
// wave-uniform, so the group sizes are too).
template <bool NT, class Idx, class Gather>
__device__ __forceinline__ double sell_lane_sum(const Idx *__restrict__ ci,
                                                const double *__restrict__ va, int32_t w,
                                                Gather gather) {
    double acc = 0.0;
    int32_t k = 0;
    for (; k + kSellUnroll <= w; k += kSellUnroll)
        acc = sell_group<kSellUnroll, NT>(ci, va, k, w, acc, gather);
    const int32_t rest = w - k;
    if (rest > 4) acc = sell_group<kSellUnroll, NT>(ci, va, k, w, acc, gather);
    else if (rest > 2) acc = sell_group<4, NT>(ci, va, k, w, acc, gather);
    else if (rest == 2) acc = sell_group<2, NT>(ci, va, k, w, acc, gather);
    else if (rest == 1) acc = sell_group<1, NT>(ci, va, k, w, acc, gather);
    return acc;
}

template <class Idx, class Gather>
__device__ __forceinline__ double sell_lane_dot(int32_t stream, const Idx *__restrict__ ci,
                                                const double *__restrict__ va, int32_t w,
                                                Gather gather) {
    return stream ? sell_lane_sum<true>(ci, va, w, gather) : sell_lane_sum<false>(ci, va, w, gather);
}

// Row sum over SELL-64 slice sl (wave-uniform) for the row of this lane:
// entries walked in order with independent, coalesced loads.
__device__ __forceinline__ RowSum sell_row_dot(const MatView &M, const double *__restrict__ x,
                                               int32_t sl) {
    RowSum r;
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    r.row = M.R_long + sl * 64 + lane;
    r.valid = sl < M.nslices && r.row < M.rows;
    double acc = 0.0;
    if (sl < M.nslices) {
        const int32_t b = __builtin_amdgcn_readfirstlane(M.slice_ptr[sl]);
        const int32_t w = (__builtin_amdgcn_readfirstlane(M.slice_ptr[sl + 1]) - b) >> 6;
        const int32_t *__restrict__ ci = M.colidx + b + lane;
        const double *__restrict__ va = M.val + b + lane;
        acc = sell_lane_dot(M.stream, ci, va, w, [&](int32_t c) { return x[c]; });
    }
    r.s = acc;
    return r;
}

// Row sum of val * x[col] for the row owned by this thread (hybrid layout).
// Long rows: lane groups with a butterfly; short rows: one thread per row,
// entries walked in order with independent, coalesced loads.
__device__ __forceinline__ RowSum mat_row_dot(const MatView &M, const double *__restrict__ x) {
    const int32_t sl = slice_of(M);
    if (sl < 0) {
        RowSum r;
        const RowCtx rc = row_ctx(M.seg);
        r.s = M.stream ? row_dot<true>(M.rowptr, M.colidx, M.val, x, rc)
                       : row_dot<false>(M.rowptr, M.colidx, M.val, x, rc);
        r.row = rc.row;
        r.valid = rc.valid && rc.lead;
        return r;
    }
    return sell_row_dot(M, x, sl);
}

// Row max (MAXNORM) or sum of |val| in the hybrid layout.
template <bool MAXNORM>
__device__ __forceinline__ RowSum mat_row_absnorm(const MatView &M) {
    RowSum r;
    const int32_t sl = slice_of(M);
    if (sl < 0) {
        const RowCtx rc = row_ctx(M.seg);
        r.s = row_absnorm<MAXNORM>(M.rowptr, M.val, rc);
        r.row = rc.row;
        r.valid = rc.valid && rc.lead;
        return r;
    }
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    r.row = M.R_long + sl * 64 + lane;
    r.valid = sl < M.nslices && r.row < M.rows;
    double acc = 0.0;
    if (sl < M.nslices) {
        const int32_t b = M.slice_ptr[sl];
        const int32_t w = (M.slice_ptr[sl + 1] - b) >> 6;
        for (int32_t k = 0; k < w; ++k) {
            const double a = fabs(M.val[b + 64 * k + lane]);
            acc = MAXNORM ? fmax(acc, a) : acc + a;
        }
    }
    r.s = acc;
    return r;
}

// val <- val / (rfac[i] * cfac[j]) for every stored entry (i, j) of the rows
// of M; transposed: the rows of M are columns j and its column indices rows i.
// Padding entries hold 0.0 and stay 0.0.
__device__ __forceinline__ void mat_scale_entries(const MatView &M, const double *__restrict__ rfac,
                                                  const double *__restrict__ cfac, bool transposed) {
    const int32_t sl = slice_of(M);
    if (sl < 0) {
        const RowCtx rc = row_ctx(M.seg);
        if (!rc.valid) return;
        const int32_t L = 1 << rc.lg;
        const int32_t lane = (int32_t)(threadIdx.x & (uint32_t)(L - 1));
        for (int32_t e = M.rowptr[rc.row] + lane; e < M.rowptr[rc.row + 1]; e += L) {
            const int32_t o = M.colidx[e];
            const double ri = transposed ? rfac[o] : rfac[rc.row];
            const double sj = transposed ? cfac[rc.row] : cfac[o];
            M.val[e] = M.val[e] / (ri * sj);
        }
        return;
    }
    if (sl >= M.nslices) return;
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    const int32_t row = M.R_long + sl * 64 + lane;
    if (row >= M.rows) return;
    const int32_t b = M.slice_ptr[sl];
    const int32_t w = (M.slice_ptr[sl + 1] - b) >> 6;
    for (int32_t k = 0; k < w; ++k) {
        const int32_t e = b + 64 * k + lane;
        const int32_t o = M.colidx[e];
        const double ri = transposed ? rfac[o] : rfac[row];
        const double sj = transposed ? cfac[row] : cfac[o];
        M.val[e] = M.val[e] / (ri * sj);
    }
}

// op over the 64 lanes, in every lane (the xor butterfly from 32 down to 1).
template <class Op>
__device__ __forceinline__ double wave_reduce(double v, Op op) {
    Pair p = swap32(v, v);
    v = op(p.a, p.b);
    p = swap16(v, v);
    v = op(p.a, p.b);
    v = op(v, dpp_get<kDppRor + 8>(v));
    v = op(v, dpp_get<kDppRor + 4>(v));
    v = op(v, dpp_get<kDppRor + 2>(v));
    return op(v, dpp_get<kDppRor + 1>(v));
}

__device__ __forceinline__ double wave_sum(double s) {
    return wave_reduce(s, [](double p, double q) { return p + q; });
}

// Eight wave sums at once: the first two butterfly steps (lane bits 5, 4) each
// halve the values a lane carries (a lane swap pairs two values' halves), the
// third picks one of the last two. Lane l ends with the total of
// value 4 bit3(l) + 2 bit4(l) + bit5(l).
__device__ __forceinline__ double wave_sum_x8(const double (&s)[8]) {
    double a[4], b[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const Pair p = swap32(s[2 * i], s[2 * i + 1]);
        a[i] = p.a + p.b;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const Pair p = swap16(a[2 * i], a[2 * i + 1]);
        b[i] = p.a + p.b;
    }
    const double c0 = b[0] + dpp_get<kDppRor + 8>(b[0]), c1 = b[1] + dpp_get<kDppRor + 8>(b[1]);
    double c = (threadIdx.x & 8) ? c1 : c0;
    return group_reduce(c, 3, [](double p, double q) { return p + q; });
}

// Deterministic workgroup sum of K values per thread: wave butterflies, then
// the BT / 64 wave totals in fixed order (BT: threads of the workgroup).
// Result written by threads 0..K-1 to out.
template <int K, int BT = kBlock>
__device__ __forceinline__ void block_sum_store(const double (&v)[K], double *__restrict__ out) {
    __shared__ double sh[K][BT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const double s = wave_sum(v[q]);
        if (lane == 0) sh[q][wave] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < K) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < BT / 64; ++w) s += sh[threadIdx.x][w];
        out[threadIdx.x] = s;
    }
}

// Same, result broadcast to every thread.
template <int K>
__device__ __forceinline__ void block_sum_all(double (&v)[K]) {
    __shared__ double sh[K][kBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const double s = wave_sum(v[q]);
        if (lane == 0) sh[q][wave] = s;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K; ++q) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) s += sh[q][w];
        v[q] = s;
    }
    __syncthreads();
}

__device__ __forceinline__ double wave_max(double s) {
    return wave_reduce(s, [](double p, double q) { return fmax(p, q); });
}

// Workgroup maxima of K values per thread (order-free), written by threads
// 0..K-1 to out (BT: threads of the workgroup).
template <int K, int BT = kBlock>
__device__ __forceinline__ void block_max_store(const double (&v)[K], double *__restrict__ out) {
    __shared__ double sh[K][BT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const double s = wave_max(v[q]);
        if (lane == 0) sh[q][wave] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < K) {
        double s = sh[threadIdx.x][0];
#pragma unroll
        for (int w = 1; w < BT / 64; ++w) s = fmax(s, sh[threadIdx.x][w]);
        out[threadIdx.x] = s;
    }
}

// Same, result broadcast to every thread.
template <int K>
__device__ __forceinline__ void block_max_all(double (&v)[K]) {
    __shared__ double sh[K][kBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const double s = wave_max(v[q]);
        if (lane == 0) sh[q][wave] = s;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K; ++q) {
        double s = sh[q][0];
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) s = fmax(s, sh[q][w]);
        v[q] = s;
    }
    __syncthreads();
}

__device__ __forceinline__ double clampd(double v, double lo, double hi) {
    return fmin(fmax(v, lo), hi);
}

// Primal-weight update after a restart: log-smoothing (weight 1/2) towards
// |dy| / |dx|. Out of line on purpose: restarts are rare, and inlined into
// the persistent kernels the constants of exp / log would stay in vector
// registers across the whole iteration loop.
static __device__ __noinline__ double batch_new_omega(double omega, double dxr, double dyr) {
    if (dxr > 1e-10 && dyr > 1e-10) return exp(0.5 * log(dyr / dxr) + 0.5 * log(omega));
    return omega;
}

// Infeasibility-ray terms of one column j at a check, in the original space:
// q = (A~'yhat)_j, q0 = (A~'y0)_j, d = D_c[j], dxs = xhat_j - x0_j, c = c_j,
// [lo, hi] = [l_v, u_v]_j. With g = -(A'dy)_j and lam its part in the cone of
// the bounds: s[0] = l_v lam+ - u_v lam-, s[1] = c dx; mx[0] = |g - lam|,
// mx[1] = distance of dx to the recession cone of [l_v, u_v].
__device__ __forceinline__ void ray_col_terms(double q, double q0, double d, double dxs, double c,
                                              double lo, double hi, double (&s)[2], double (&mx)[2]) {
    const bool lf = isfinite(lo), uf = isfinite(hi);
    const double g = -(q - q0) / d;
    const double lam = (!lf && !uf) ? 0.0 : (lf && !uf) ? fmax(g, 0.0) : (!lf && uf) ? fmin(g, 0.0) : g;
    s[0] = (lf ? lo * fmax(lam, 0.0) : 0.0) - (uf ? hi * fmax(-lam, 0.0) : 0.0);
    mx[0] = fabs(g - lam);
    const double dx = d * dxs;
    s[1] = c * dx;
    mx[1] = fabs(dx - clampd(dx, lf ? 0.0 : -INFINITY, uf ? 0.0 : INFINITY));
}

// Same for row i: p = (A~xhat)_i, p0 = (A~x0)_i, d = D_r[i], dys = yhat_i -
// y0_i, [lo, hi] = [l_c, u_c]_i. With yp = proj_Y(dy): s[0] = l_c yp+ - u_c yp-;
// mx[0] = |dy - yp|, mx[1] = distance of (A dx)_i to the recession cone of
// [l_c, u_c].
__device__ __forceinline__ void ray_row_terms(double p, double p0, double d, double dys, double lo,
                                              double hi, double (&s)[1], double (&mx)[2]) {
    const bool lf = isfinite(lo), uf = isfinite(hi);
    const double dy = d * dys;
    const double yp = clampd(dy, uf ? -INFINITY : 0.0, lf ? INFINITY : 0.0);
    s[0] = (lf ? lo * fmax(yp, 0.0) : 0.0) - (uf ? hi * fmax(-yp, 0.0) : 0.0);
    mx[0] = fabs(dy - yp);
    const double a = (p - p0) / d;
    mx[1] = fabs(a - clampd(a, lf ? 0.0 : -INFINITY, uf ? 0.0 : INFINITY));
}

// Dual proximal step of eq. (pdhg-lp): v = y/sigma - a,
// yhat = sigma (v - proj_[-u_c, -l_c](v)); exactly 0 inside, exactly signed outside.
__device__ __forceinline__ double dual_prox(double y, double a, double sigma, double lc, double uc) {
    const double v = y / sigma - a;
    return sigma * (v - clampd(v, -uc, -lc));
}

// f(row) for the Q-value rows p[b * Q, b * Q + Q) of the blocks
// b = threadIdx.x + kBlock * i of one thread, in increasing b; eight blocks'
// loads are issued before their f calls.
template <int Q, class F>
__device__ __forceinline__ void strided_fold(const double *__restrict__ p, int32_t nb, F f) {
    int32_t b = (int32_t)threadIdx.x;
    for (; b + 7 * kBlock < nb; b += 8 * kBlock) {
        double t[8][Q];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int q = 0; q < Q; ++q) t[u][q] = p[(size_t)(b + u * kBlock) * Q + q];
#pragma unroll
        for (int u = 0; u < 8; ++u) f(t[u]);
    }
    for (; b < nb; b += kBlock) {
        double t[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) t[q] = p[(size_t)b * Q + q];
        f(t);
    }
}

// Totals of a check's per-workgroup partials, for the one-workgroup
// controllers (every thread ends with the same totals): vn / vm the six
// column-side and four row-side sums (pn: nbn rows of 6, pm: nbm rows of 4);
// with rays, rs the three ray sums (prn[b * 4 + 0, 1], prm[b * 3]) and rx the
// two ray maxima (prn[b * 4 + 2, 3] with prm[b * 3 + 1, 2]), else zeros.
__device__ __forceinline__ void check_totals(const double *__restrict__ pn, int32_t nbn,
                                             const double *__restrict__ pm, int32_t nbm,
                                             const double *__restrict__ prn,
                                             const double *__restrict__ prm, bool rays,
                                             double (&vn)[6], double (&vm)[4], double (&rs)[3],
                                             double (&rx)[2]) {
#pragma unroll
    for (int q = 0; q < 6; ++q) vn[q] = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) vm[q] = 0.0;
    rs[0] = rs[1] = rs[2] = 0.0;
    rx[0] = rx[1] = 0.0;
    strided_fold<6>(pn, nbn, [&](const double *t) {
#pragma unroll
        for (int q = 0; q < 6; ++q) vn[q] += t[q];
    });
    strided_fold<4>(pm, nbm, [&](const double *t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) vm[q] += t[q];
    });
    block_sum_all<6>(vn);
    block_sum_all<4>(vm);
    if (!rays) return;
    strided_fold<4>(prn, nbn, [&](const double *t) {
        rs[0] += t[0];
        rs[1] += t[1];
        rx[0] = fmax(rx[0], t[2]);
        rx[1] = fmax(rx[1], t[3]);
    });
    strided_fold<3>(prm, nbm, [&](const double *t) {
        rs[2] += t[0];
        rx[0] = fmax(rx[0], t[1]);
        rx[1] = fmax(rx[1], t[2]);
    });
    block_sum_all<3>(rs);
    block_max_all<2>(rx);
}

}  // namespace pdhg
