// llr_recon.hip -- FP64 reconstruction kernels (arXiv:1509.08391):
//   ln rho at the interval centres by the trapezium recursion (eq. (kk3a)),
//   in the convention a_k = -d ln rho/dE:  L_{k+1} = L_k - (s/2)(a_k + a_{k+1});
//   canonical moments by the midpoint sums (eqs. (l19)-(l20)):
//   p_k ~ exp(L_k + beta c_k), <E> = sum p_k c_k, Var(E) = sum p_k (c_k - <E>)^2,
//   <u> = <E>/(6V), C_V = Var(E)/(6V) (Sec. 3.4).
#include <hip/hip_runtime.h>

#include "llr_internal.hpp"

namespace llr {

constexpr int kRB = 256;

// ln rho at n centres into L (LDS or global): the recursion is sequential by
// definition, so one thread adds, but the whole block loads the terms, kTerms
// at a time, into LDS first (a thread that also loads waits for memory at every
// step: 20 us at n = 128, against 2).  Every caller's block has kRB threads.
constexpr int kTerms = 1024;

template <typename F>
__device__ __forceinline__ void scan_lnrho(const double* __restrict__ a, int n, double s, double* term, F&& store) {
    double v = 0.0;
    const double f = -(0.5 * s);
    for (int k0 = 0; k0 < n; k0 += kTerms) {
        const int m = min(kTerms, n - k0);
        for (int i = threadIdx.x; i < m; i += kRB) {
            const int k = k0 + i;
            term[i] = k == 0 ? 0.0 : a[k - 1] + a[k];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int i = 0;
            for (; i + 8 <= m; i += 8) {
                double t[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) t[q] = term[i + q];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    v = __fma_rn(f, t[q], v);
                    if (q == 0 && k0 + i == 0) v = 0.0;   // the first centre's by definition, also for an infinite s
                    term[i + q] = v;
                }
            }
            for (; i < m; ++i) {
                v = k0 + i == 0 ? 0.0 : __fma_rn(f, term[i], v);
                term[i] = v;
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < m; i += kRB) store(k0 + i, term[i]);
        __syncthreads();
    }
}

// one block per set of a_k (row r of a and of L at offset r n)
__global__ __launch_bounds__(kRB) void k_lnrho(const double* __restrict__ a, int n, double s, double* __restrict__ L) {
    __shared__ double term[kTerms];
    const size_t r = (size_t)blockIdx.x * (size_t)n;
    scan_lnrho(a + r, n, s, term, [&](int k, double v) { L[r + k] = v; });
}

// ---------------------------------------------------------------------------
// Moments of up to kRowN intervals in registers.  A block-wide reduction per
// sum (four per point, two barriers each) and a second exponential per interval
// made a grid point cost more in barriers than in arithmetic; here G = 16 lanes
// (one DPP row, reduced by rotations) or a whole wavefront hold one point's
// terms, KP per lane, and compute each exponential once.
// ---------------------------------------------------------------------------
constexpr int kRowN = 512;

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// over the 16 lanes of a row, the same value on all of them (row_ror:8, 4, 2, 1)
__device__ __forceinline__ double row_sum(double v) {
    v += dpp_f64<0x128>(v);
    v += dpp_f64<0x124>(v);
    v += dpp_f64<0x122>(v);
    return v + dpp_f64<0x121>(v);
}
__device__ __forceinline__ double row_max(double v) {
    v = fmax(v, dpp_f64<0x128>(v));
    v = fmax(v, dpp_f64<0x124>(v));
    v = fmax(v, dpp_f64<0x122>(v));
    return fmax(v, dpp_f64<0x121>(v));
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
template <int G>
__device__ __forceinline__ double grp_sum(double v) {
    v = row_sum(v);
    if constexpr (G == 64) v = (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
    return v;
}
template <int G>
__device__ __forceinline__ double grp_max(double v) {
    v = row_max(v);
    if constexpr (G == 64) v = fmax(fmax(lane_f64(v, 0), lane_f64(v, 16)), fmax(lane_f64(v, 32), lane_f64(v, 48)));
    return v;
}

// (mean, variance) of E at coupling beta; c, L: this lane's terms (an absent
// one has c = 0, L = -inf)
template <int KP, int G>
__device__ __forceinline__ void lane_moments(const double (&c)[KP], const double (&L)[KP], double beta, double* mean,
                                             double* var) {
    double w[KP], m = -INFINITY;
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        w[q] = __fma_rn(beta, c[q], L[q]);
        m = fmax(m, w[q]);
    }
    m = grp_max<G>(m);
    double z = 0.0, s1 = 0.0;
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        w[q] = exp(w[q] - m);
        z += w[q];
        s1 = __fma_rn(w[q], c[q], s1);
    }
    z = grp_sum<G>(z);
    s1 = grp_sum<G>(s1);
    const double mu = s1 / z;
    double s2 = 0.0;
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        const double d = c[q] - mu;
        s2 = __fma_rn(w[q] * d, d, s2);
    }
    *mean = mu;
    *var = grp_sum<G>(s2) / z;
}

// this lane's terms of a row whose ln rho is in LDS: intervals lane, lane + G, ...
template <int KP, int G>
__device__ __forceinline__ void lane_terms(const double* __restrict__ c, const double* Ls, int n, int lane,
                                           double (&cr)[KP], double (&Lr)[KP]) {
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        const int k = lane + q * G;
        cr[q] = k < n ? c[k] : 0.0;
        Lr[q] = k < n ? Ls[k] : -INFINITY;
    }
}

// Points beta (beta_at[i], or blo + i h) of row blockIdx.y, per_block of them
// to a block, 16 lanes to a point: Var(E) into var, or <u> and C_V into u and
// cv; ln rho into lnrho (first block of a row) where asked for.
template <int KP>
__global__ __launch_bounds__(kRB) void k_row_points(const double* __restrict__ c, const double* __restrict__ a, int n,
                                                     double s, const double* __restrict__ beta_at, double blo, double h,
                                                     long np, int per_block, double six_v, double* __restrict__ lnrho,
                                                     double* __restrict__ var, double* __restrict__ u,
                                                     double* __restrict__ cv) {
    __shared__ double term[kTerms];
    const double* ar = a + (size_t)blockIdx.y * (size_t)n;
    scan_lnrho(ar, n, s, term, [&](int k, double v) {
        if (lnrho && blockIdx.x == 0) lnrho[(size_t)blockIdx.y * (size_t)n + k] = v;
    });
    const int lane = threadIdx.x & 15;
    double cr[KP], Lr[KP];
    lane_terms<KP, 16>(c, term, n, lane, cr, Lr);
    const long i0 = (long)blockIdx.x * per_block, i1 = min(np, i0 + per_block);
    // every lane of a wavefront takes part in the row rotations, so all rows of
    // the block make the same number of turns and the last points are repeated
    for (long ib = i0; ib < i1; ib += kRB / 16) {
        const long i = min(ib + (threadIdx.x >> 4), i1 - 1);
        double mu, v;
        lane_moments<KP, 16>(cr, Lr, beta_at ? beta_at[i] : blo + (double)i * h, &mu, &v);
        if (lane == 0 && ib + (threadIdx.x >> 4) < i1) {
            if (var) {
                var[(size_t)blockIdx.y * (size_t)np + i] = v;
            } else {
                u[i] = mu / six_v;
                cv[i] = v / six_v;
            }
        }
    }
}

// argmax of a row's grid (the first of equal maxima), by the whole block
__device__ __forceinline__ void grid_argmax(const double* __restrict__ var, long ng, double* best, long* at) {
    __shared__ double sv[kRB];
    __shared__ long si[kRB];
    double v = -INFINITY;
    long b = 0;
    for (long i = threadIdx.x; i <= ng; i += kRB)
        if (var[i] > v) { v = var[i]; b = i; }
    sv[threadIdx.x] = v;
    si[threadIdx.x] = b;
    __syncthreads();
    for (int off = kRB / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            const double v2 = sv[threadIdx.x + off];
            const long b2 = si[threadIdx.x + off];
            if (v2 > sv[threadIdx.x] || (v2 == sv[threadIdx.x] && b2 < si[threadIdx.x])) {
                sv[threadIdx.x] = v2;
                si[threadIdx.x] = b2;
            }
        }
        __syncthreads();
    }
    *best = sv[0];
    *at = si[0];
}

// Golden section on [x0, x3] to tol for the function f (variance at a
// coupling); best, bb: the grid's maximum and its coupling
template <typename F>
__device__ __forceinline__ void golden(double x0, double x3, double tol, double best, double bb, double* bc, double* v,
                                       F&& f) {
    const double gr = 0.61803398874989484820;
    double x1 = x3 - gr * (x3 - x0), x2 = x0 + gr * (x3 - x0);
    double f1 = f(x1), f2 = f(x2);
    // (the bound on the steps ends a search whose tol is below the spacing of beta)
    for (int it = 0; x3 - x0 > tol && it < 4096; ++it) {
        if (f1 > f2) {
            x3 = x2; x2 = x1; f2 = f1;
            x1 = x3 - gr * (x3 - x0);
            f1 = f(x1);
        } else {
            x0 = x1; x1 = x2; f1 = f2;
            x2 = x0 + gr * (x3 - x0);
            f2 = f(x2);
        }
    }
    *bc = 0.5 * (x0 + x3);
    *v = f(*bc);
    if (best > *v) { *bc = bb; *v = best; }
}

// argmax of the grid by the block, then golden section by one wavefront, which
// needs no barrier between its ~25 dependent evaluations (one block per row)
template <int KP>
__global__ __launch_bounds__(kRB) void k_row_golden(const double* __restrict__ c, const double* __restrict__ a, int n,
                                                     double s, const double* __restrict__ var_rows, long ng, double blo,
                                                     double bhi, double h, double tol, double six_v,
                                                     double* __restrict__ out_rows) {
    __shared__ double term[kTerms];
    scan_lnrho(a + (size_t)blockIdx.x * (size_t)n, n, s, term, [](int, double) {});
    double best;
    long at;
    grid_argmax(var_rows + (size_t)blockIdx.x * (size_t)(ng + 1), ng, &best, &at);
    if (threadIdx.x >= 64) return;
    double cr[KP], Lr[KP];
    lane_terms<KP, 64>(c, term, n, (int)threadIdx.x, cr, Lr);
    const double bb = blo + (double)at * h;
    double bc, v;
    golden(fmax(blo, bb - h), fmin(bhi, bb + h), tol, best, bb, &bc, &v, [&](double x) {
        double mu, f;
        lane_moments<KP, 64>(cr, Lr, x, &mu, &f);
        return f;
    });
    if (threadIdx.x == 0) {
        out_rows[2 * (size_t)blockIdx.x] = bc;
        out_rows[2 * (size_t)blockIdx.x + 1] = v / six_v;
    }
}

__device__ double block_max(double v, double* sh) {
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = sh[0];
    for (int i = 1; i < kRB / 64; ++i) r = fmax(r, sh[i]);
    __syncthreads();
    return r;
}
__device__ double block_sum(double v, double* sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = 0.0;
    for (int i = 0; i < kRB / 64; ++i) r += sh[i];
    __syncthreads();
    return r;
}

// block-wide (mean, variance) of E at coupling beta
__device__ void moments(const double* __restrict__ c, const double* __restrict__ L, int n, double beta, double* sh,
                        double* mean, double* var) {
    double m = -INFINITY;
    for (int k = threadIdx.x; k < n; k += kRB) m = fmax(m, L[k] + beta * c[k]);
    m = block_max(m, sh);
    double z = 0.0, s1 = 0.0;
    for (int k = threadIdx.x; k < n; k += kRB) {
        const double wk = exp(L[k] + beta * c[k] - m);
        z += wk;
        s1 += wk * c[k];
    }
    z = block_sum(z, sh);
    s1 = block_sum(s1, sh);
    const double mu = s1 / z;
    double s2 = 0.0;
    for (int k = threadIdx.x; k < n; k += kRB) {
        const double wk = exp(L[k] + beta * c[k] - m);
        s2 += wk * (c[k] - mu) * (c[k] - mu);
    }
    s2 = block_sum(s2, sh);
    *mean = mu;
    *var = s2 / z;
}

// one block per beta
__global__ __launch_bounds__(kRB) void k_moments(const double* __restrict__ c, const double* __restrict__ L, int n,
                                                  const double* __restrict__ beta, double six_v, double* __restrict__ u,
                                                  double* __restrict__ cv) {
    __shared__ double sh[kRB / 64];
    double mu, var;
    moments(c, L, n, beta[blockIdx.x], sh, &mu, &var);
    if (threadIdx.x == 0) {
        u[blockIdx.x] = mu / six_v;
        cv[blockIdx.x] = var / six_v;
    }
}

// Var(E) on the grid blo + i h, i = 0..ng (one block per point; blockIdx.y
// selects the set of a_k: L row y, var row y of ng + 1)
__global__ __launch_bounds__(kRB) void k_var_grid(const double* __restrict__ c, const double* __restrict__ L, int n,
                                                   double blo, double h, long ng, double* __restrict__ var) {
    __shared__ double sh[kRB / 64];
    double mu, v;
    moments(c, L + (size_t)blockIdx.y * n, n, blo + (double)blockIdx.x * h, sh, &mu, &v);
    if (threadIdx.x == 0) var[(size_t)blockIdx.y * (size_t)(ng + 1) + blockIdx.x] = v;
}

// argmax of the grid, then golden section on [b* - h, b* + h] to tol (one
// block per set of a_k: L row, var row and out pair selected by blockIdx.x)
__global__ __launch_bounds__(kRB) void k_golden(const double* __restrict__ c, const double* __restrict__ Lrows, int n,
                                                 const double* __restrict__ var_rows, long ng, double blo, double bhi,
                                                 double h, double tol, double six_v, double* __restrict__ out_rows) {
    const double* L = Lrows + (size_t)blockIdx.x * n;
    const double* var = var_rows + (size_t)blockIdx.x * (size_t)(ng + 1);
    double* out = out_rows + 2 * (size_t)blockIdx.x;
    __shared__ double sh[kRB / 64];
    double best;
    long at;
    grid_argmax(var, ng, &best, &at);
    const double bb = blo + (double)at * h;
    double bc, v;
    golden(fmax(blo, bb - h), fmin(bhi, bb + h), tol, best, bb, &bc, &v, [&](double x) {
        double mu, f;
        moments(c, L, n, x, sh, &mu, &f);
        return f;
    });
    if (threadIdx.x == 0) {
        out[0] = bc;
        out[1] = v / six_v;
    }
}

// fewest terms per lane (of 16, or of 64) that hold n <= kRowN intervals
#define LLR_BY_TERMS(G, CALL)                     \
    do {                                          \
        if (n <= 4 * G) { CALL(4); }              \
        else if (n <= 8 * G) { CALL(8); }         \
        else if (n <= 16 * G) { CALL(16); }       \
        else { CALL(32); }                        \
    } while (0)

void launch_recon(const double* c, const double* a, int n, double s, double six_v, const double* beta, int nb,
                  double* lnrho, double* u, double* cv, hipStream_t st) {
    if (nb > 0 && n <= kRowN) {
#define LLR_CALL(KP)                                                                                             \
    hipLaunchKernelGGL(k_row_points<KP>, dim3((unsigned)((nb + 15) / 16)), dim3(kRB), 0, st, c, a, n, s, beta, 0.0, 0.0, \
                       (long)nb, 16, six_v, lnrho, (double*)nullptr, u, cv)
        LLR_BY_TERMS(16, LLR_CALL);
#undef LLR_CALL
        return;
    }
    hipLaunchKernelGGL(k_lnrho, dim3(1), dim3(kRB), 0, st, a, n, s, lnrho);
    if (nb > 0) hipLaunchKernelGGL(k_moments, dim3(nb), dim3(kRB), 0, st, c, lnrho, n, beta, six_v, u, cv);
}

// beta_c and the C_V peak for `rows` sets of a_k (a row r at a + r n);
// scratch holds rows (n + ng + 1) doubles, out2 rows pairs.  Up to kRowN
// intervals a point's terms fit a few registers of a DPP row or a wavefront;
// beyond that a block walks them.  n = 128, 401 points, us by blocks / in
// registers: one row 116 / 34 (recursion 20, grid 10, golden section 86), the
// grid of 1000 bootstrap rows 950 / 110.
void launch_beta_c_rows(const double* c, const double* a, int n, int rows, double s, double six_v, double blo,
                        double bhi, double h, double tol, double* scratch, double* out2, hipStream_t st) {
    const long ng = (long)floor((bhi - blo) / h + 0.5);
    double* L = scratch;
    double* var = scratch + (size_t)rows * n;
    if (n <= kRowN) {
        // a block scans its row's ln rho once for all its points: few blocks of
        // many points where the rows fill the chip, many of few for one row
        const int per = rows >= 64 ? 128 : 16;
#define LLR_CALL(KP)                                                                                                \
    hipLaunchKernelGGL(k_row_points<KP>, dim3((unsigned)((ng + per) / per), (unsigned)rows), dim3(kRB), 0, st, c, a, n, s, \
                       (const double*)nullptr, blo, h, ng + 1, per, six_v, (double*)nullptr, var, (double*)nullptr,    \
                       (double*)nullptr)
        LLR_BY_TERMS(16, LLR_CALL);
#undef LLR_CALL
#define LLR_CALL(KP)                                                                                                   \
    hipLaunchKernelGGL(k_row_golden<KP>, dim3((unsigned)rows), dim3(kRB), 0, st, c, a, n, s, var, ng, blo, bhi, h, tol, \
                       six_v, out2)
        if (n <= 64) { LLR_CALL(1); }
        else if (n <= 128) { LLR_CALL(2); }
        else if (n <= 256) { LLR_CALL(4); }
        else { LLR_CALL(8); }
#undef LLR_CALL
        return;
    }
    hipLaunchKernelGGL(k_lnrho, dim3((unsigned)rows), dim3(kRB), 0, st, a, n, s, L);
    hipLaunchKernelGGL(k_var_grid, dim3((unsigned)(ng + 1), (unsigned)rows), dim3(kRB), 0, st, c, L, n, blo, h, ng,
                       var);
    hipLaunchKernelGGL(k_golden, dim3((unsigned)rows), dim3(kRB), 0, st, c, L, n, var, ng, blo, bhi, h, tol, six_v,
                       out2);
}

void launch_beta_c(const double* c, const double* a, int n, double s, double six_v, double blo, double bhi, double h,
                   double tol, double* lnrho_scratch, double* out2, hipStream_t st) {
    launch_beta_c_rows(c, a, n, 1, s, six_v, blo, bhi, h, tol, lnrho_scratch, out2, st);
}

// ---------------------------------------------------------------------------
// Bootstrap over N_B independent runs (Algorithm 1 repeated N_B times, Sec. 2.4
// and Sec. 3.2): sample b draws n_runs runs with replacement, run j of sample
// b being floor(n_runs w / 2^32) for the first word w of Philox counter
// (j, kind 5, b, 0), and averages their a_k (runs summed in draw order).
// ---------------------------------------------------------------------------
constexpr int kMaxRuns = 1024;

__global__ __launch_bounds__(kRB) void k_boot_mean(const double* __restrict__ a_runs, int n_runs, int n, uint32_t k0,
                                                    uint32_t k1, double* __restrict__ abar) {
    __shared__ int idx[kMaxRuns];
    const uint32_t b = blockIdx.x;
    for (int j = threadIdx.x; j < n_runs; j += kRB) {
        const uint4 w = philox10(make_uint4((uint32_t)j, ctr1_word(0, 0, kBoot, 0), b, 0u), k0, k1);
        idx[j] = (int)(((uint64_t)w.x * (uint64_t)n_runs) >> 32);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += kRB) {
        double sum = 0.0;
        for (int j = 0; j < n_runs; ++j) sum += a_runs[(size_t)idx[j] * n + k];
        abar[(size_t)b * n + k] = sum / (double)n_runs;
    }
}

void launch_boot_mean(const double* a_runs, int n_runs, int n, int n_boot, uint64_t seed, double* abar,
                      hipStream_t st) {
    hipLaunchKernelGGL(k_boot_mean, dim3((unsigned)n_boot), dim3(kRB), 0, st, a_runs, n_runs, n, (uint32_t)seed,
                       (uint32_t)(seed >> 32), abar);
}

// ---------------------------------------------------------------------------
// Probability density P_beta(E) = rho~(E) e^{beta E} / Z (Sec. 3.4) of the
// piecewise-exponential rho~ of eq. (rhoguess): in interval k (centre c_k,
// width s) ln rho~(E) = L_k - a_k (E - c_k), continuous at the edges by the
// trapezium recursion.  Z is the exact integral over the covered range:
// Z = sum_k s e^{L_k + beta c_k} sinh(x_k)/x_k, x_k = (beta - a_k) s / 2.
// ---------------------------------------------------------------------------
__device__ double log_sinhc(double x) {
    const double ax = fabs(x);
    if (ax < 1e-3) return ax * ax * (1.0 / 6.0) - ax * ax * ax * ax * (1.0 / 180.0);
    if (ax < 20.0) return log(sinh(ax) / ax);
    return ax - log(2.0 * ax) + log1p(-exp(-2.0 * ax));
}

// one block: ln Z, with the row maximum subtracted before the sum
__global__ __launch_bounds__(kRB) void k_logz(const double* __restrict__ c, const double* __restrict__ L,
                                               const double* __restrict__ a, int n, double s, double beta,
                                               double* __restrict__ lnz) {
    __shared__ double sh[kRB / 64];
    double m = -INFINITY;
    for (int k = threadIdx.x; k < n; k += kRB)
        m = fmax(m, L[k] + beta * c[k] + log_sinhc((beta - a[k]) * 0.5 * s));
    m = block_max(m, sh);
    double z = 0.0;
    for (int k = threadIdx.x; k < n; k += kRB)
        z += exp(L[k] + beta * c[k] + log_sinhc((beta - a[k]) * 0.5 * s) - m);
    z = block_sum(z, sh);
    if (threadIdx.x == 0) lnz[0] = m + log(s * z);
}

// ln P at m points E (one thread each; -inf outside the covered range)
__global__ void k_logp(const double* __restrict__ c, const double* __restrict__ L, const double* __restrict__ a,
                       int n, double s, double beta, const double* __restrict__ E, int m,
                       const double* __restrict__ lnz, double* __restrict__ logp) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= m) return;
    const double lo = c[0] - 0.5 * s, hi = c[n - 1] + 0.5 * s, e = E[i];
    if (!(e >= lo && e <= hi)) {
        logp[i] = -INFINITY;
        return;
    }
    int k = (int)floor((e - lo) / s);
    k = k < 0 ? 0 : (k > n - 1 ? n - 1 : k);
    logp[i] = (L[k] + beta * c[k] - lnz[0]) + (beta - a[k]) * (e - c[k]);
}

// Interior local maxima of ln P: ln P is linear with slope beta - a_k in
// interval k, so the edge between k and k+1 is a maximum iff beta - a_k > 0
// and beta - a_{k+1} <= 0 (one wavefront; every maximum counted, at most
// max_peaks stored in order of E).
__global__ void k_peaks(const double* __restrict__ c, const double* __restrict__ L, const double* __restrict__ a,
                        int n, double s, double beta, const double* __restrict__ lnz, int max_peaks,
                        double* __restrict__ E_out, double* __restrict__ lp_out, int* __restrict__ n_out) {
    int np = 0;   // one wavefront: 64 edges at a time, in order
    for (int k0 = 0; k0 + 1 < n; k0 += 64) {
        const int k = k0 + (int)threadIdx.x;
        const bool pk = k + 1 < n && beta - a[k] > 0.0 && beta - a[k + 1] <= 0.0;
        const unsigned long long m = __ballot(pk);
        const int at = np + (int)__popcll(m & ((1ull << threadIdx.x) - 1ull));
        if (pk && at < max_peaks) {
            E_out[at] = c[k] + 0.5 * s;
            lp_out[at] = (L[k] + beta * c[k] - lnz[0]) + (beta - a[k]) * (0.5 * s);
        }
        np += (int)__popcll(m);
    }
    if (threadIdx.x == 0) *n_out = np;
}

// scratch: n (ln rho) + 1 (ln Z) doubles
void launch_prob(const double* c, const double* a, int n, double s, double beta, const double* E, int m,
                 double* logp, int max_peaks, double* E_pk, double* lp_pk, int* n_pk, double* scratch,
                 hipStream_t st) {
    double* L = scratch;
    double* lnz = scratch + n;
    hipLaunchKernelGGL(k_lnrho, dim3(1), dim3(kRB), 0, st, a, n, s, L);
    hipLaunchKernelGGL(k_logz, dim3(1), dim3(kRB), 0, st, c, L, a, n, s, beta, lnz);
    if (m > 0) hipLaunchKernelGGL(k_logp, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, c, L, a, n, s, beta,
                                  E, m, lnz, logp);
    if (n_pk) hipLaunchKernelGGL(k_peaks, dim3(1), dim3(64), 0, st, c, L, a, n, s, beta, lnz, max_peaks, E_pk, lp_pk,
                                 n_pk);
}

// ---------------------------------------------------------------------------
// Reweighting of multicanonical samples (Sec. 2.6, eq. (4.7)): with the
// sampling weight W(E) = 1/rho~(E) (first and last pieces continued outside
// the intervals), <O>_beta = <O e^{beta E} / W(E)>_W / <e^{beta E} / W(E)>_W.
// One block per beta: <E>, Var(E) -> <u> = <E>/(6V), C_V = Var(E)/(6V).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double rw_lnw(const double* c, const double* L, const double* a, int n, double s,
                                         double e) {
    int k = (int)floor((e - (c[0] - 0.5 * s)) / s);
    k = k < 0 ? 0 : (k > n - 1 ? n - 1 : k);
    return -L[k] + a[k] * (e - c[k]);
}

__global__ __launch_bounds__(kRB) void k_rw_moments(const double* __restrict__ E, long m,
                                                     const double* __restrict__ c, const double* __restrict__ L,
                                                     const double* __restrict__ a, int n, double s,
                                                     const double* __restrict__ beta, double six_v,
                                                     double* __restrict__ u, double* __restrict__ cv) {
    __shared__ double sh[kRB / 64];
    const double b = beta[blockIdx.x];
    double mx = -INFINITY;
    for (long i = threadIdx.x; i < m; i += kRB) mx = fmax(mx, b * E[i] - rw_lnw(c, L, a, n, s, E[i]));
    mx = block_max(mx, sh);
    double z = 0.0, s1 = 0.0;
    for (long i = threadIdx.x; i < m; i += kRB) {
        const double w = exp(b * E[i] - rw_lnw(c, L, a, n, s, E[i]) - mx);
        z += w;
        s1 += w * E[i];
    }
    z = block_sum(z, sh);
    s1 = block_sum(s1, sh);
    const double mu = s1 / z;
    double s2 = 0.0;
    for (long i = threadIdx.x; i < m; i += kRB) {
        const double w = exp(b * E[i] - rw_lnw(c, L, a, n, s, E[i]) - mx);
        s2 += w * (E[i] - mu) * (E[i] - mu);
    }
    s2 = block_sum(s2, sh);
    if (threadIdx.x == 0) {
        u[blockIdx.x] = mu / six_v;
        cv[blockIdx.x] = s2 / z / six_v;
    }
}

// scratch: n doubles (ln rho)
void launch_reweight(const double* E, long m, const double* c, const double* a, int n, double s, const double* beta,
                     int nb, double six_v, double* u, double* cv, double* scratch, hipStream_t st) {
    hipLaunchKernelGGL(k_lnrho, dim3(1), dim3(kRB), 0, st, a, n, s, scratch);
    hipLaunchKernelGGL(k_rw_moments, dim3((unsigned)nb), dim3(kRB), 0, st, E, m, c, scratch, a, n, s, beta, six_v, u,
                       cv);
}

// ---------------------------------------------------------------------------
// Observables from restricted double brackets (Sec. 2.3, eqs. (l9)-(l10)):
//   <B>_beta = sum_k rho~(c_k) e^{beta c_k} <<B e^{(beta - a_k)(E - c_k)}>>_k
//            / sum_k rho~(c_k) e^{beta c_k} <<e^{(beta - a_k)(E - c_k)}>>_k,
// with <<.>>_k the mean over the m samples (E, B) of interval k (row-major
// m x n, interval fastest).  One block per beta; the interval terms are
// combined in log space.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kRB) void k_obs_bracket(const double* __restrict__ E, const double* __restrict__ B,
                                                      int m, const double* __restrict__ c,
                                                      const double* __restrict__ L, const double* __restrict__ a,
                                                      int n, const double* __restrict__ beta,
                                                      double* __restrict__ out) {
    __shared__ double sh[kRB / 64];
    const double b = beta[blockIdx.x];
    // per interval: ln D_k and N_k / D_k, D_k = <<e^{x}>>, x = (b - a_k)(E - c_k), shifted by the interval's max
    double wmax = -INFINITY;
    for (int k = threadIdx.x; k < n; k += kRB) {
        double xm = -INFINITY;
        for (int j = 0; j < m; ++j) xm = fmax(xm, (b - a[k]) * (E[(size_t)j * n + k] - c[k]));
        double d = 0.0;
        for (int j = 0; j < m; ++j) d += exp((b - a[k]) * (E[(size_t)j * n + k] - c[k]) - xm);
        wmax = fmax(wmax, L[k] + b * c[k] + xm + log(d / m));
    }
    wmax = block_max(wmax, sh);
    double num = 0.0, den = 0.0;
    for (int k = threadIdx.x; k < n; k += kRB) {
        double xm = -INFINITY;
        for (int j = 0; j < m; ++j) xm = fmax(xm, (b - a[k]) * (E[(size_t)j * n + k] - c[k]));
        double d = 0.0, nb = 0.0;
        for (int j = 0; j < m; ++j) {
            const double w = exp((b - a[k]) * (E[(size_t)j * n + k] - c[k]) - xm);
            d += w;
            nb += w * B[(size_t)j * n + k];
        }
        const double wk = exp(L[k] + b * c[k] + xm + log(d / m) - wmax);
        den += wk;
        num += wk * (nb / d);
    }
    den = block_sum(den, sh);
    num = block_sum(num, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = num / den;
}

// scratch: n doubles (ln rho)
void launch_obs_bracket(const double* E, const double* B, int m, const double* c, const double* a, int n, double s,
                        const double* beta, int nb, double* out, double* scratch, hipStream_t st) {
    hipLaunchKernelGGL(k_lnrho, dim3(1), dim3(kRB), 0, st, a, n, s, scratch);
    hipLaunchKernelGGL(k_obs_bracket, dim3((unsigned)nb), dim3(kRB), 0, st, E, B, m, c, scratch, a, n, beta, out);
}

}  // namespace llr
