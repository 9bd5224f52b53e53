// Loss heads around the unrolled solver for end-to-end learning (Section 4,
// the shortest-path and portfolio pipelines): a linear cost model on
// per-variable features, the regret of the decisions under the true costs,
// the weight gradient of the cost model, and the value / gradient of a
// low-rank-plus-diagonal QP objective. All sums are deterministic
// workgroup trees in a fixed order.
#include <algorithm>
#include <mutex>

#include "device.hpp"

namespace pdhg {

constexpr int kHeadWide = 2048;   // columns beyond which an instance gets a workgroup of 1,024 threads
constexpr int kHeadRmax = 32;     // largest factor rank of pdhg_qp_value
constexpr int kHeadPmax = 64;     // most features of the linear cost model
constexpr int kScratchDoubles = 32768;   // partial sums of the weight gradient (64 features x 512 chunks)
constexpr int kGradChunks = 1024;         // most chunks
constexpr int kMaxDevices = 64;
constexpr int64_t kMostEntries = ((int64_t)1 << 32) - 1;   // of a launch that counts them in 32 bits

// Partial sums of the allocation-free weight gradient (256 KB on every GPU the
// library runs on, kept until the process ends). Host code never uses this
// name as an address: it reads the device address once per device with
// hipGetSymbolAddress and passes that to the kernels.
static __device__ __align__(256) double scratch[kScratchDoubles];

// The positions t, t + BT, ... of thread t in [0, n), in groups of 4, the last
// one of 4, 2 or 1: load(u, a) for all of a group (clamped to n - 1), then
// use(u, a) for those that exist. With one position's loads at a time the heads
// of eight 3,968-column instances took 5.2 us where their launch alone is 2; a
// last group of always 4 made the regret of 2,048 x 1,025 columns twice as slow.
template <int BT, class Load, class Use>
__device__ __forceinline__ void strided(uint32_t n, Load load, Use use) {
    uint32_t a0 = 0;
    auto group = [&](auto width) {
        constexpr int U = decltype(width)::value;
        const uint32_t a = a0 + threadIdx.x;
#pragma unroll
        for (int u = 0; u < U; ++u) load(u, min(a + u * BT, n - 1));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (a + u * BT < n) use(u, a + u * BT);
    };
    for (; a0 + 2 * BT < n; a0 += 4 * BT) group(std::integral_constant<int, 4>());
    if (a0 + BT < n) group(std::integral_constant<int, 2>());
    else if (a0 < n) group(std::integral_constant<int, 1>());
}

// Workgroup sum in fixed order (waves in order), in every thread.
template <int BT>
__device__ __forceinline__ double head_sum(double v) {
    __shared__ double sh[BT / 64];
    const double w = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = w;
    __syncthreads();
    double s = sh[0];
#pragma unroll
    for (int q = 1; q < BT / 64; ++q) s += sh[q];
    return s;
}

// Cost model, up to kCostsRow features: a thread per row. A wave's rows lie in a
// few lines, which its loads of one feature after another find in the cache.
// 8 M rows of 1 / 4 features: 21 / 60 us, through LDS 31 / 92.
constexpr int kCostsRow = 4;
__global__ __launch_bounds__(kBlock) void k_linear_costs_row(int64_t N, int32_t p,
                                                             const double *__restrict__ f,
                                                             const double *__restrict__ W,
                                                             double *__restrict__ c) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < N; i += (int64_t)gridDim.x * kBlock) {
        double s = 0.0;
        for (int32_t k = 0; k < p; ++k) s = fma(W[k], f[i * p + k], s);
        c[i] = s;
    }
}

// Up to P features: the workgroup's 256 rows pass through LDS, read from memory
// in one coalesced run (a thread reading its own row of many values touches a
// line per lane and entry), four values of a thread in flight; a row's products
// are added in order. Rows in LDS are p | 1 apart, so that the lanes' banks
// differ. P sets the LDS and with it the workgroups of a compute unit.
constexpr int kCostsLds = 16;   // most features of this variant
template <int P>
__global__ __launch_bounds__(kBlock) void k_linear_costs(int64_t N, int32_t p,
                                                         const double *__restrict__ f,
                                                         const double *__restrict__ W,
                                                         double *__restrict__ c) {
    __shared__ double sh[kBlock * (P + 1)];
    const int32_t r0 = (int32_t)threadIdx.x / p, k0 = (int32_t)threadIdx.x - r0 * p;
    const int32_t dr = kBlock / p, dk = kBlock - dr * p, st = p | 1;
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock; i0 < N; i0 += (int64_t)gridDim.x * kBlock) {
        const int32_t rows = (int32_t)min((int64_t)kBlock, N - i0), len = rows * p;
        const double *__restrict__ src = f + i0 * p;
        int32_t r = r0, k = k0;
        for (int32_t e0 = (int32_t)threadIdx.x; e0 < len; e0 += 4 * kBlock) {
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = src[min(e0 + u * kBlock, len - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (e0 + u * kBlock < len) sh[r * st + k] = v[u];
                r += dr;
                k += dk;
                if (k >= p) {
                    k -= p;
                    ++r;
                }
            }
        }
        __syncthreads();
        if ((int32_t)threadIdx.x < rows) {
            const double *mine = sh + threadIdx.x * st;
            double s = 0.0;
            for (int32_t q = 0; q < p; ++q) s = fma(W[q], mine[q], s);
            c[i0 + threadIdx.x] = s;
        }
        __syncthreads();
    }
}

// Many features: 16 lanes per row, up to four entries each.
__global__ __launch_bounds__(kBlock) void k_linear_costs_wide(int64_t N, int32_t p,
                                                              const double *__restrict__ f,
                                                              const double *__restrict__ W,
                                                              double *__restrict__ c) {
    static_assert(kHeadPmax == 64, "four entries per lane");
    const int32_t lane = threadIdx.x & 15;
    for (int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 4; i < N; i += (int64_t)gridDim.x * (kBlock / 16)) {
        double a[4], w[4], s = 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t k = min(lane + 16 * u, p - 1);
            a[u] = f[i * p + k];
            w[u] = W[k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) s = lane + 16 * u < p ? fma(w[u], a[u], s) : s;
        s = group_reduce(s, 4, [](double x, double y) { return x + y; });
        if (lane == 0) c[i] = s;
    }
}

// One workgroup per instance: loss[b] = c_true_b' x_b - v_star[b].
template <int BT>
__global__ __launch_bounds__(BT) void k_regret(int32_t B, int32_t n, const double *__restrict__ ct,
                                                         const double *__restrict__ x,
                                                         const double *__restrict__ vs,
                                                         double *__restrict__ loss) {
    for (uint32_t b = blockIdx.x;;) {
        const size_t o = (size_t)b * n;
        double v = 0.0, c[4], w[4];
        strided<BT>((uint32_t)n, [&](int u, uint32_t a) { c[u] = ct[o + a]; w[u] = x[o + a]; },
                    [&](int u, uint32_t) { v = fma(c[u], w[u], v); });
        v = head_sum<BT>(v);
        if (threadIdx.x == 0) loss[b] = v - vs[b];
        b += gridDim.x;
        if (b >= (uint32_t)B) return;   // a barrier would wait for the stores
        __syncthreads();
    }
}

// out[k] = the sum of the step values v of the threads k, k + p, ... (t < step p),
// for k < p <= BT: up to eight threads per feature add every eighth of them, then
// one adds theirs.
template <int BT>
__device__ __forceinline__ void feature_totals(double v, int32_t p, int32_t step, double *__restrict__ out) {
    __shared__ double sh[BT];
    const int32_t t = (int32_t)threadIdx.x, groups = min(8, BT / p);
    sh[t] = v;
    __syncthreads();
    const int32_t g = t / p, k = t - g * p;
    double s = 0.0;
    if (g < groups)
        for (int32_t q = g; q < step; q += groups) s += sh[q * p + k];
    __syncthreads();
    sh[t] = s;
    __syncthreads();
    if (t >= p) return;
    s = 0.0;
    for (int32_t q = 0; q < groups; ++q) s += sh[q * p + t];
    out[t] = s;
}

// Partial weight gradients of a run of rows: thread t of the first (BT / p) p
// keeps feature t mod p and takes every (BT / p)-th row, so that the workgroup
// reads f in one coalesced stream; the threads of a feature are then added into
// part[chunk p + k]. (A workgroup per feature read f p times, a line
// per lane.)
template <int BT>
__global__ __launch_bounds__(BT) void k_costs_grad_part(int64_t N, int32_t p, int32_t chunks,
                                                        const double *__restrict__ f,
                                                        const double *__restrict__ gc,
                                                        double *__restrict__ part) {
    const int32_t step = BT / p, live = step * p;
    const int64_t len = (N + chunks - 1) / chunks;
    const int64_t i0 = blockIdx.x * len, i1 = min(N, i0 + len);
    double v = 0.0;
    if ((int32_t)threadIdx.x < live) {
        const int32_t r = (int32_t)threadIdx.x / p, k = (int32_t)threadIdx.x - r * p;
        int64_t base = i0;
        auto rows = [&](auto width) {   // rows base + r, base + r + step, ...
            constexpr int U = decltype(width)::value;
            const int64_t i = base + r;
            double g[U], e[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t q = min(i + (int64_t)u * step, i1 - 1);
                g[u] = gc[q];
                e[u] = f[q * p + k];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) v = i + (int64_t)u * step < i1 ? fma(g[u], e[u], v) : v;
        };
        for (; base + 4 * (int64_t)step < i1; base += 8 * (int64_t)step) rows(std::integral_constant<int, 8>());
        if (base + 2 * step < i1) rows(std::integral_constant<int, 4>());
        else if (base + step < i1) rows(std::integral_constant<int, 2>());
        else if (base < i1) rows(std::integral_constant<int, 1>());
    }
    feature_totals<BT>(v, p, step, part + (size_t)blockIdx.x * p);
}

// gW[k] = the chunks' partial sums of feature k, added as in the partial kernel.
template <int BT>
__global__ __launch_bounds__(BT) void k_costs_grad_final(int32_t p, int32_t chunks,
                                                         const double *__restrict__ part,
                                                         double *__restrict__ gW) {
    const int32_t step = BT / p, live = step * p;
    double v = 0.0;
    if ((int32_t)threadIdx.x < live) {
        const int32_t total = chunks * p;
        for (int32_t e = (int32_t)threadIdx.x; e < total; e += 8 * live) {
            double a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = part[min(e + u * live, total - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) v += e + u * live < total ? a[u] : 0.0;
        }
    }
    feature_totals<BT>(v, p, step, gW);
}

// One workgroup per instance: t = F' x, Qx = F t + d x, value and gradient.
// G: groups of eight factor columns (a runtime rank would put t in scratch
// memory); t reaches the lanes as scalars.
template <int G>
__global__ __launch_bounds__(kBlock) void k_qp_value(int32_t B, int32_t n, int32_t r, const double *__restrict__ F,
                                                     const double *__restrict__ d,
                                                     const double *__restrict__ c,
                                                     const double *__restrict__ x,
                                                     double *__restrict__ value,
                                                     double *__restrict__ gx) {
    constexpr int R = 8 * G;
    __shared__ double sh[R > 0 ? R : 1][kBlock / 64];
    const int32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto factor_row = [&](int32_t j, double (&f)[R > 0 ? R : 1]) {
#pragma unroll
        for (int k = 0; k < R; ++k) f[k] = F[(size_t)j * r + min(k, r - 1)];
#pragma unroll
        for (int k = 0; k < R; ++k) f[k] = k < r ? f[k] : 0.0;
    };
    for (uint32_t b = blockIdx.x;;) {
        const size_t o = (size_t)b * n;
        double t[R > 0 ? R : 1], f[R > 0 ? R : 1];
        if constexpr (G > 0) {
#pragma unroll
            for (int k = 0; k < R; ++k) t[k] = 0.0;
            for (int32_t j = threadIdx.x; j < n; j += kBlock) {
                const double xj = x[o + j];
                factor_row(j, f);
#pragma unroll
                for (int k = 0; k < R; ++k) t[k] = fma(f[k], xj, t[k]);
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                double v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = t[8 * g + k];
                const double w = wave_sum_x8(v);
                if ((lane & 7) == 0) sh[8 * g + 4 * ((lane >> 3) & 1) + 2 * ((lane >> 4) & 1) + ((lane >> 5) & 1)][wave] = w;
            }
            __syncthreads();
            const int32_t p = lane < R ? lane : 0;
            double tp = sh[p][0];
#pragma unroll
            for (int w = 1; w < kBlock / 64; ++w) tp += sh[p][w];
#pragma unroll
            for (int k = 0; k < R; ++k) t[k] = k < r ? lane_value(tp, k) : 0.0;   // 0 x an infinite x is no 0
        }
        double v = 0.0;
        for (int32_t j = threadIdx.x; j < n; j += kBlock) {
            const double xj = x[o + j], cj = c[o + j];
            double qx = d[o + j] * xj;
            if constexpr (G > 0) {
                factor_row(j, f);
#pragma unroll
                for (int k = 0; k < R; ++k) qx = fma(f[k], t[k], qx);
            }
            if (gx) gx[o + j] = qx + cj;
            v += xj * (0.5 * qx + cj);
        }
        v = head_sum<kBlock>(v);
        if (threadIdx.x == 0) value[b] = v;
        b += gridDim.x;
        if (b >= (uint32_t)B) return;   // a barrier would wait for the stores
        __syncthreads();
    }
}

// SPO+ (Elmachtoub-Grigas) for min_{w in S} c'w: the inner problem's costs
// 2 c_hat - c_true, entrywise over the N = B n variables.
__global__ __launch_bounds__(kBlock) void k_spo_costs(int64_t N, const double *__restrict__ ch,
                                                      const double *__restrict__ ct,
                                                      double *__restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < N; i += (int64_t)gridDim.x * kBlock)
        out[i] = 2.0 * ch[i] - ct[i];
}

// One workgroup per instance: with w* optimal under c_true (value z*) and w~
// optimal under 2 c_hat - c_true, loss = -(2 c_hat - c)'w~ + 2 c_hat'w* - z*,
// summed as 2 c_hat'(w* - w~) + c'w~ - z* (the same value, without the
// cancellation of two large products), and the subgradient 2 (w* - w~).
template <int BT>
__global__ __launch_bounds__(BT) void k_spo_plus(int32_t B, int32_t n, const double *__restrict__ ch,
                                                           const double *__restrict__ ct,
                                                           const double *__restrict__ ws,
                                                           const double *__restrict__ zs,
                                                           const double *__restrict__ wt,
                                                           double *__restrict__ loss,
                                                           double *__restrict__ grad) {
    for (uint32_t b = blockIdx.x;;) {
        const size_t o = (size_t)b * n;
        double v = 0.0, h[4], c[4], s[4], w[4];
        strided<BT>(
            (uint32_t)n,
            [&](int u, uint32_t a) {
                h[u] = ch[o + a];
                c[u] = ct[o + a];
                s[u] = ws[o + a];
                w[u] = wt[o + a];
            },
            [&](int u, uint32_t a) {
                const double dw = s[u] - w[u];
                v += 2.0 * h[u] * dw + c[u] * w[u];
                grad[o + a] = 2.0 * dw;
            });
        v = head_sum<BT>(v);
        if (threadIdx.x == 0) loss[b] = v - zs[b];
        b += gridDim.x;
        if (b >= (uint32_t)B) return;   // a barrier would wait for the stores
        __syncthreads();
    }
}

// Perturbed Fenchel-Young (Berthet et al.), minimisation form: sample (b, m)
// has costs c_hat_b + eps Z_bm; entry i of the [B][M][n] output. Rounded as
// a product then a sum, so the costs equal the textbook expression exactly.
// A workgroup takes kPfyTile entries in a row, whatever samples they belong to
// (a workgroup per sample left 256 threads with 24 entries, and grids beyond
// the limit of 2^32 work-items at 2^24 samples). One division a workgroup finds
// its first sample; from there an entry is at most one sample on where a sample
// fills a tile, and shorter samples are counted by a multiplication with magic =
// ceil(2^32 / n), exact while dividend times n is below 2^32 (here below 2^20).
// What bounds it: 16 bytes of memory an entry. 200,000 x 24 samples of one draw
// take 18 us (144 with a workgroup per sample), 2,048 x 4 of 1,025 29 (40). Four
// entries a thread gain up to 10% on the largest calls and lose as much on others.
constexpr int kPfyEach = 2, kPfyTile = kPfyEach * kBlock;
__global__ __launch_bounds__(kBlock) void k_pfy_costs(int64_t N, int32_t M, int32_t n, uint32_t magic,
                                                      const double *__restrict__ ch,
                                                      const double *__restrict__ Z, double eps,
                                                      double *__restrict__ out) {
#pragma clang fp contract(off)
    const int64_t i0 = (int64_t)blockIdx.x * kPfyTile;
    // first sample of the tile, its instance, and the tile's start in the sample
    const uint32_t row = (uint32_t)i0 / (uint32_t)n, b = row / (uint32_t)M;
    const uint32_t first = (uint32_t)i0 - row * (uint32_t)n, m0 = row - b * (uint32_t)M;
    double z[kPfyEach], h[kPfyEach];
#pragma unroll
    for (int u = 0; u < kPfyEach; ++u) {
        const int64_t i = min(i0 + (int32_t)threadIdx.x + u * kBlock, N - 1);
        const uint32_t a = first + (uint32_t)(i - i0);
        uint32_t q, up;   // samples and instances past the first
        if (n >= kPfyTile) {
            q = a >= (uint32_t)n;
            up = m0 + q >= (uint32_t)M;
        } else {
            q = n == 1 ? a : __umulhi(a, magic);
            up = (m0 + q) / (uint32_t)M;
        }
        z[u] = Z[i];
        h[u] = ch[(int64_t)(b + up) * n + (a - q * (uint32_t)n)];
    }
#pragma unroll
    for (int u = 0; u < kPfyEach; ++u) {
        const int64_t i = i0 + (int32_t)threadIdx.x + u * kBlock;
        const double pz = eps * z[u];
        if (i < N) out[i] = h[u] + pz;
    }
}

// One workgroup per instance: with w_m optimal under c_hat + eps Z_m,
// grad = w* - (1/M) sum_m w_m and loss = c_hat'w* - (1/M) sum_m (c_hat +
// eps Z_m)'w_m (the loss up to the constant Omega(w*)); samples summed in m
// order per variable.
template <int BT>
__global__ __launch_bounds__(BT) void k_pfy(int32_t B, int32_t M, int32_t n, const double *__restrict__ ch,
                                                      const double *__restrict__ ws,
                                                      const double *__restrict__ Z, double eps,
                                                      const double *__restrict__ wm,
                                                      double *__restrict__ loss,
                                                      double *__restrict__ grad) {
    for (uint32_t b = blockIdx.x;;) {
        const size_t o = (size_t)b * n;
        const double dm = (double)M;
        double v = 0.0;
        for (int32_t a = threadIdx.x; a < n; a += BT) {
            const double c = ch[o + a], s = ws[o + a];
            const double *pw = wm + o * M + a, *pz = Z + o * M + a;
            double wsum = 0.0, acc = 0.0;
            // the next samples, their loads in flight together
            auto samples = [&](auto width) {
                constexpr int U = decltype(width)::value;
                double w[U], z[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    w[u] = pw[(size_t)u * n];
                    z[u] = pz[(size_t)u * n];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    wsum += w[u];
                    acc += (c + eps * z[u]) * w[u];
                }
                pw += (size_t)U * n;
                pz += (size_t)U * n;
            };
            int32_t m = M;
            for (; m >= 8; m -= 8) samples(std::integral_constant<int, 8>());
            if (m & 4) samples(std::integral_constant<int, 4>());
            if (m & 2) samples(std::integral_constant<int, 2>());
            if (m & 1) samples(std::integral_constant<int, 1>());
            grad[o + a] = s - wsum / dm;
            v += c * s - acc / dm;
        }
        v = head_sum<BT>(v);
        if (threadIdx.x == 0) loss[b] = v;
        b += gridDim.x;
        if (b >= (uint32_t)B) return;   // a barrier would wait for the stores
        __syncthreads();
    }
}

// Workgroups for N threads. A launch holds fewer than 2^32 work-items in a
// dimension, and one beyond is cut without an error: from 2^31 on the kernels
// below walk on by the grid's size.
static unsigned grid1(int64_t N) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(N, kBlock), ((int64_t)1 << 31) / kBlock));
}

// Workgroups (of up to 1,024 threads) for B instances, which walk on likewise.
static unsigned instance_groups(int32_t B) { return (unsigned)std::min(B, 1 << 21); }

void head_linear_costs(hipStream_t s, int32_t B, int32_t n, int32_t p, const double *f,
                       const double *W, double *c) {
    const int64_t N = (int64_t)B * n;
    if (N == 0) return;
    if (p <= kCostsRow) k_linear_costs_row<<<grid1(N), kBlock, 0, s>>>(N, p, f, W, c);
    else if (p <= 8) k_linear_costs<8><<<grid1(N), kBlock, 0, s>>>(N, p, f, W, c);
    else if (p <= kCostsLds) k_linear_costs<kCostsLds><<<grid1(N), kBlock, 0, s>>>(N, p, f, W, c);
    else
        k_linear_costs_wide<<<grid1(N * 16), kBlock, 0, s>>>(N, p, f, W, c);
    PDHG_HIP(hipGetLastError());
}

void head_regret(hipStream_t s, int32_t B, int32_t n, const double *ct, const double *x,
                 const double *vs, double *loss) {
    if (B == 0) return;
    if (n > kHeadWide) k_regret<1024><<<instance_groups(B), 1024, 0, s>>>(B, n, ct, x, vs, loss);
    else k_regret<256><<<instance_groups(B), 256, 0, s>>>(B, n, ct, x, vs, loss);
    PDHG_HIP(hipGetLastError());
}

// The weight gradient with its partial sums in part (kScratchDoubles): a run of
// at least 128 rows per workgroup, as many as the partial sums have room for;
// with many features, and so few runs, larger workgroups. 256 x 3,968 rows of 5
// features 23.5 -> 15 us, 512 x 6,000 rows of 64 1,184 -> 315 us (5.0 TB/s).
static void costs_gradient(hipStream_t s, int64_t N, int32_t p, const double *f, const double *gc, double *part,
                           double *gW) {
    const int32_t chunks = (int32_t)std::max<int64_t>(1, std::min<int64_t>({kScratchDoubles / p, kGradChunks, ceil_div(N, 128)}));
    if (p <= 16) k_costs_grad_part<256><<<(unsigned)chunks, 256, 0, s>>>(N, p, chunks, f, gc, part);
    else k_costs_grad_part<1024><<<(unsigned)chunks, 1024, 0, s>>>(N, p, chunks, f, gc, part);
    if (chunks * p <= 2048) k_costs_grad_final<256><<<1, 256, 0, s>>>(p, chunks, part, gW);
    else k_costs_grad_final<1024><<<1, 1024, 0, s>>>(p, chunks, part, gW);
    PDHG_HIP(hipGetLastError());
}

void head_linear_costs_backward(hipStream_t s, int32_t B, int32_t n, int32_t p, const double *f,
                                const double *gc, double *gW) {
    DBuf<double> part;
    part.alloc(kScratchDoubles);
    costs_gradient(s, (int64_t)B * n, p, f, gc, part.p, gW);
    PDHG_HIP(hipStreamSynchronize(s));
}

// Device address of `scratch` on the device that runs stream s (the current
// device for the NULL stream), looked up once per device with that device
// current.
static double *scratch_address(hipStream_t s) {
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    int cur = 0, dev = 0;
    PDHG_HIP(hipGetDevice(&cur));
    dev = cur;
    if (s) PDHG_HIP(hipStreamGetDevice(s, &dev));
    if (dev < 0 || dev >= kMaxDevices) fail(PDHG_ERR_UNSUPPORTED, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        if (dev != cur) PDHG_HIP(hipSetDevice(dev));
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (dev != cur) PDHG_HIP(hipSetDevice(cur));
        if (e != hipSuccess || !p)
            fail(PDHG_ERR_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        addr[dev] = static_cast<double *>(p);
    }
    return addr[dev];
}

// The same reduction as head_linear_costs_backward into the static scratch
// array: no allocation and no wait; calls that overlap on one GPU race on it.
void head_linear_costs_backward_noalloc(hipStream_t s, int32_t B, int32_t n, int32_t p,
                                        const double *f, const double *gc, double *gW) {
    if (p < 1 || p > kHeadPmax) fail(PDHG_ERR_INVALID_ARG, "need 1 <= p <= 64 (the scratch holds 64 x 512 partials)");
    costs_gradient(s, (int64_t)B * n, p, f, gc, scratch_address(s), gW);
}

void head_qp_value(hipStream_t s, int32_t B, int32_t n, int32_t r, const double *F,
                   const double *d, const double *c, const double *x, double *value, double *gx) {
    if (B == 0) return;
    if (r > kHeadRmax) fail(PDHG_ERR_UNSUPPORTED, "factor rank above 32");
    switch ((r + 7) / 8) {
        case 0: k_qp_value<0><<<instance_groups(B), kBlock, 0, s>>>(B, n, r, F, d, c, x, value, gx); break;
        case 1: k_qp_value<1><<<instance_groups(B), kBlock, 0, s>>>(B, n, r, F, d, c, x, value, gx); break;
        case 2: k_qp_value<2><<<instance_groups(B), kBlock, 0, s>>>(B, n, r, F, d, c, x, value, gx); break;
        case 3: k_qp_value<3><<<instance_groups(B), kBlock, 0, s>>>(B, n, r, F, d, c, x, value, gx); break;
        default: k_qp_value<4><<<instance_groups(B), kBlock, 0, s>>>(B, n, r, F, d, c, x, value, gx); break;
    }
    PDHG_HIP(hipGetLastError());
}

void head_spo_costs(hipStream_t s, int32_t B, int32_t n, const double *c_hat, const double *c_true,
                    double *out) {
    const int64_t N = (int64_t)B * n;
    if (N == 0) return;
    k_spo_costs<<<grid1(N), kBlock, 0, s>>>(N, c_hat, c_true, out);
    PDHG_HIP(hipGetLastError());
}

void head_spo_plus(hipStream_t s, int32_t B, int32_t n, const double *c_hat, const double *c_true,
                   const double *w_star, const double *z_star, const double *w_tilde, double *loss,
                   double *grad) {
    if (B == 0) return;
    if (n > kHeadWide)
        k_spo_plus<1024><<<instance_groups(B), 1024, 0, s>>>(B, n, c_hat, c_true, w_star, z_star, w_tilde, loss, grad);
    else
        k_spo_plus<256><<<instance_groups(B), 256, 0, s>>>(B, n, c_hat, c_true, w_star, z_star, w_tilde, loss, grad);
    PDHG_HIP(hipGetLastError());
}

void head_pfy_costs(hipStream_t s, int32_t B, int32_t M, int32_t n, const double *c_hat,
                    const double *Z, double eps, double *out) {
    if (B == 0 || M == 0 || n == 0) return;
    // the entries of one launch are counted in 32 bits: whole instances, or whole
    // samples of one, as many as that takes
    const int64_t samples = kMostEntries / n, each = samples / M;
    const uint32_t magic = n > 1 ? (uint32_t)((((uint64_t)1 << 32) + (uint32_t)n - 1) / (uint32_t)n) : 0;
    auto launch = [&](int64_t b, int64_t m, int64_t count, int64_t of) {   // samples m .. of instances b ..
        const int64_t N = count * of * n, at = (b * M + m) * n;
        k_pfy_costs<<<(unsigned)ceil_div(N, kPfyTile), kBlock, 0, s>>>(N, (int32_t)of, n, magic, c_hat + b * n, Z + at, eps,
                                                                      out + at);
    };
    if (each > 0)
        for (int64_t b = 0; b < B; b += each) launch(b, 0, std::min<int64_t>(each, B - b), M);
    else
        for (int64_t b = 0; b < B; ++b)
            for (int64_t m = 0; m < M; m += samples) launch(b, m, 1, std::min<int64_t>(samples, M - m));
    PDHG_HIP(hipGetLastError());
}

void head_pfy(hipStream_t s, int32_t B, int32_t M, int32_t n, const double *c_hat,
              const double *w_star, const double *Z, double eps, const double *w_samples, double *loss,
              double *grad) {
    if (B == 0) return;
    if (n > kHeadWide) k_pfy<1024><<<instance_groups(B), 1024, 0, s>>>(B, M, n, c_hat, w_star, Z, eps, w_samples, loss, grad);
    else k_pfy<256><<<instance_groups(B), 256, 0, s>>>(B, M, n, c_hat, w_star, Z, eps, w_samples, loss, grad);
    PDHG_HIP(hipGetLastError());
}

}  // namespace pdhg
