// paths.hip -- the Monte Carlo path kernel and the fixed-order reduction.
//
// One path per lane, 64 paths per wavefront.  The log-rate state X_i =
// log L(t, T_i) - log L(0, T_i) of all rates lives in registers (slots off ..
// nmax-1 of a compile-time bucket), so every period of the tenor runs code
// specialised to its number of live rates.  Per Euler step k (paper Section 2,
// eqs. (LIBOR-dyn-PT), (log-LIB-SIE); Section 3 for the schemes):
//
//   1. Philox-4x32-10 words for counter (k, p_lo, p_hi, stream word);
//   2. the driver increment dH (FP64: subordinator + normal mixture);
//   3. ell_j = delta_j L_j / (1 + delta_j L_j) of the live rates, from X
//      (FULL) or from the Picard iterate X1 (PICARD, eq. (bdrift));
//   4. the coupling C_i = sum_q W_q E_{i,q} (prod_{l>i} beta_l(x_q) - 1) by a
//      suffix recursion over the rates, node by node:
//          C_i += W_q E_{i,q} R_q,   R_q <- R_q + ell_i E_{i,q} (1 + R_q),
//      which is the product of eq. (LIBOR-drift-PT) with beta_l = 1 + ell_l E_l
//      evaluated once for all i (O(N Q) per step instead of O(N^2 Q));
//      the uniform table entries (E, W E) are wave-uniform scalar operands;
//   5. X_i += (-kappa_i - C_i) dt + lambda_i dH (PICARD also advances
//      X1_i += b0_i dt + lambda_i dH; FROZEN advances only X with b0);
//   6. at the end of period m the rate with maturity T_{m+1} fixes: the FP64
//      payoffs prod_{l>i}(1 + delta_l L_l)(L_i - K)^+ of eq. (caplet) and the
//      martingale factor are summed across the wavefront (butterfly), and lane
//      0 writes the wave's sums; a two-pass fixed-order FP64 reduction follows.
#include <hip/hip_runtime.h>

#include "lll_device.hpp"
#include "lll_internal.hpp"
#include "path_kernel.hpp"

namespace lll {
namespace {

__global__ void __launch_bounds__(kBlock) increments_kernel(const double *__restrict__ steps, int k,
                                                            int s, int64_t p0, int64_t n,
                                                            uint32_t stream_word, uint32_t key0,
                                                            uint32_t key1, int brownian, double *__restrict__ V,
                                                            double *__restrict__ dH) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    const int64_t p = p0 + i;
    const int m = k / s;
    const StepConsts cst{steps[4 * m], steps[4 * m + 1], steps[4 * m + 2], steps[4 * m + 3]};
    const uint4 w = philox4x32_10(
        make_uint4(static_cast<uint32_t>(k), static_cast<uint32_t>(p),
                   static_cast<uint32_t>(static_cast<uint64_t>(p) >> 32), stream_word),
        key0, key1);
    double v;
    dH[i] = increment(w, cst, brownian != 0, &v);
    V[i] = v;
}

__global__ void __launch_bounds__(kBlock) philox_kernel(const uint32_t *__restrict__ ctr,
                                                        const uint32_t *__restrict__ key,
                                                        int64_t n, uint32_t *__restrict__ out) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    const uint4 c = make_uint4(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]);
    const uint4 r = philox4x32_10(c, key[2 * i], key[2 * i + 1]);
    out[4 * i] = r.x;
    out[4 * i + 1] = r.y;
    out[4 * i + 2] = r.z;
    out[4 * i + 3] = r.w;
}

// The increment's FP64 routines on given arguments (fn: LLL_SM_*; LLL_SM_DIV
// reads the pairs x[2i], x[2i+1]); the host has checked the domains.
__global__ void __launch_bounds__(kBlock) sampler_math_kernel(int fn, const double *__restrict__ x,
                                                              int64_t n, double *__restrict__ out) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    double r = 0.0;
    if (fn == LLL_SM_LOG) {
        r = log_unit(x[i]);
    } else if (fn == LLL_SM_SINPI || fn == LLL_SM_COSPI) {
        double sn, cs;
        sincospi_unit(x[i], sn, cs);
        r = fn == LLL_SM_SINPI ? sn : cs;
    } else if (fn == LLL_SM_SQRT) {
        r = sqrt_pos(x[i]);
    } else {
        r = div_pos(x[2 * i], x[2 * i + 1]);
    }
    out[i] = r;
}

constexpr int kReduceBlock = 1024;
constexpr int kChunkRows = 256;     // wavefronts per chunk row
constexpr int kChunkCols = 256;     // columns per block of pass 1
constexpr int kDirectRows = 32;     // up to here pass 2 reads the wave partials itself
constexpr int kMaxCols = LLL_N_MAX_MP * (3 * LLL_S_MAX + 2);

// Sums of rows r0 .. r1 of the columns c_first .. c_end (of cols), into `out`: as
// many row groups as the block holds of the padded columns, each group's rows in
// order, then the groups in order (a fixed order whatever the grid).  The groups
// and the unrolled loads hide the memory latency that one thread per column and
// one row at a time left open (both passes and the results at N = 20, 2^20 paths:
// 86 us, now 18).
__device__ __forceinline__ void sum_rows(const double *__restrict__ in, int64_t r0, int64_t r1,
                                         int cols, int c_first, int c_end,
                                         double *__restrict__ part, double *__restrict__ out) {
    const int width = min(kReduceBlock, (c_end - c_first + 63) / 64 * 64);
    const int groups = kReduceBlock / width;
    const int g = threadIdx.x / width, c0 = threadIdx.x % width;
    const int64_t per = (r1 - r0 + groups - 1) / groups;
    const int64_t a = min(r1, r0 + g * per), b = min(r1, a + per);
    for (int base = c_first; base < c_end; base += width) {
        const int c = base + c0;
        if (g < groups) {
            double acc = 0.0;
            if (c < c_end) {
                const double *p = in + a * cols + c;
                int64_t r = a;
                for (; r + 8 <= b; r += 8) {
                    double v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = p[static_cast<int64_t>(i) * cols];
#pragma unroll
                    for (int i = 0; i < 8; ++i) acc += v[i];
                    p += static_cast<int64_t>(8) * cols;
                }
                for (; r < b; ++r, p += cols) acc += *p;
            }
            part[threadIdx.x] = acc;
        }
        __syncthreads();
        if (g == 0 && c < c_end) {
            double acc = part[c0];
            for (int i = 1; i < groups; ++i) acc += part[i * width + c0];
            out[c] = acc;
        }
        __syncthreads();
    }
}

// Pass 1: block b sums the wave partials' rows [b*256, (b+1)*256) of the 256
// columns of blockIdx.z.
__global__ void __launch_bounds__(kReduceBlock) reduce_rows_kernel(
    PassArgs one, const PassArgs *__restrict__ many, int64_t rows) {
    __shared__ double part[kReduceBlock];
    PassArgs a = one;
    if (many) a = many[blockIdx.y];
    const int cols = a.N * (3 * a.S + 2);
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kChunkRows;
    const int c0 = blockIdx.z * kChunkCols;
    if (c0 >= cols) return;
    sum_rows(a.partials, r0, min(rows, r0 + kChunkRows), cols, c0, min(cols, c0 + kChunkCols), part,
             a.chunks + static_cast<int64_t>(blockIdx.x) * cols);
}

// Pass 2: one block sums the chunk rows (or the few wave partials themselves), then prices, standard errors and martingale residuals from
// the sums (eq. (caplet)): price = delta_i B(0, T_*) mean(p), B(0, T_*) =
// B(0, T_1) / prod_l (1 + delta_l L_l(0)).
__global__ void __launch_bounds__(kReduceBlock) finalize_kernel(PassArgs one,
                                                                const PassArgs *__restrict__ many,
                                                                int64_t rows, int from_partials,
                                                                int64_t n_paths) {
    __shared__ double part[kReduceBlock], sums[kMaxCols], fac[LLL_N_MAX_MP];
    PassArgs a = one;
    if (many) a = many[blockIdx.y];
    const int N = a.N, S = a.S, nstat = 3 * S + 2, cols = N * nstat;
    const int t = threadIdx.x;
    if (t < N) fac[t] = 1.0 + a.delta[t] * a.L0[t];
    sum_rows(from_partials ? a.partials : a.chunks, 0, rows, cols, 0, cols, part, sums);
    for (int i = t; i < cols; i += kReduceBlock) a.sums[i] = sums[i];
    // inputs set from device memory that fail the checks of Section 2 give NaN
    const double poison = (a.lam_pm[2] != 0.0 || a.lam_pm[3] != 0.0) ? __builtin_nan("") : 0.0;
    double prod_all = 1.0;
    for (int l = 0; l < N; ++l) prod_all *= fac[l];
    const double B0T = a.B0_T1 / prod_all;
    const double n = static_cast<double>(n_paths);
    const double nm1 = n > 1.0 ? n - 1.0 : 1.0;
    double *res = a.results;
    double *price = res, *se = res + N * S, *itm = res + 2 * N * S;
    double *mart = res + 3 * N * S, *mart_se = res + 3 * N * S + N;
    for (int i = t; i < N * S; i += kReduceBlock) {
        const int r = i / S, k = i % S;
        const double *sr = sums + r * nstat;
        // caplets pay delta_r (L - K)^+; swaption payoffs are already amounts
        const double scale = a.product == LLL_SWAPTIONS ? B0T : a.delta[r] * B0T;
        const double mean = sr[k] / n;
        const double var = fmax(sr[S + k] / n - mean * mean, 0.0);
        price[i] = scale * mean + poison;
        se[i] = scale * sqrt(var / nm1) + poison;
        itm[i] = sr[2 * S + k];
    }
    if (t < N) {
        const double *sr = sums + t * nstat;
        double fwd = 1.0;
        for (int l = t; l < N; ++l) fwd *= fac[l];
        const double mm = sr[3 * S] / n;
        const double mv = fmax(sr[3 * S + 1] / n - mm * mm, 0.0);
        mart[t] = mm - fwd;
        mart_se[t] = sqrt(mv / nm1);
    }
}

// max_cols: the most columns of any structure.
hipError_t reduce(const PassArgs &one, const PassArgs *many, int structures, int max_cols,
                  int64_t n_paths, hipStream_t st) {
    const int64_t waves = (n_paths + kWave - 1) / kWave;
    const int64_t chunks = (waves + kChunkRows - 1) / kChunkRows;
    const bool direct = waves <= kDirectRows;
    if (!direct) {
        hipLaunchKernelGGL(reduce_rows_kernel,
                           dim3(static_cast<unsigned>(chunks), structures,
                                (max_cols + kChunkCols - 1) / kChunkCols),
                           dim3(kReduceBlock), 0, st, one, many, waves);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(finalize_kernel, dim3(1, structures), dim3(kReduceBlock), 0, st, one, many,
                       direct ? waves : chunks, direct ? 1 : 0, n_paths);
    return hipGetLastError();
}

}  // namespace

int bucket_for(int n_rates, bool slots20) {
    if (n_rates <= 8) return 8;
    if (n_rates <= 16) return 16;
    if (slots20 && n_rates <= 20) return 20;
    if (n_rates <= 24) return 24;
    if (n_rates <= 32) return 32;
    if (n_rates <= 40) return 40;
    return 64;  // tables only: the maturity-parallel PICARD
}

hipError_t launch_paths(const lll_plan &p, int scheme, int64_t n_paths, int64_t path_offset,
                        uint64_t seed, double *path_fix, hipStream_t st) {
    using namespace detail;
    if (p.precision == LLL_FP64) {
        switch (p.nmax) {
            case 8: return launch_bucket<double, 8>(p, scheme, n_paths, path_offset, seed, path_fix, st);
            case 16: return launch_bucket<double, 16>(p, scheme, n_paths, path_offset, seed, path_fix, st);
            case 24: return launch_bucket<double, 24>(p, scheme, n_paths, path_offset, seed, path_fix, st);
            default: return hipErrorInvalidValue;
        }
    }
    switch (p.nmax) {
        case 8: return launch_bucket<float, 8>(p, scheme, n_paths, path_offset, seed, path_fix, st);
        case 16: return launch_bucket<float, 16>(p, scheme, n_paths, path_offset, seed, path_fix, st);
        case 20: return launch_bucket<float, 20>(p, scheme, n_paths, path_offset, seed, path_fix, st);
        case 24: return launch_bucket<float, 24>(p, scheme, n_paths, path_offset, seed, path_fix, st);
        case 32: return launch_bucket<float, 32>(p, scheme, n_paths, path_offset, seed, path_fix, st);
        case 40: return launch_bucket<float, 40>(p, scheme, n_paths, path_offset, seed, path_fix, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_drift(const lll_plan &p, int k, const double *L_dev, int64_t n, double *b_dev,
                        hipStream_t st) {
    using namespace detail;
    if (p.precision == LLL_FP64) {
        switch (p.nmax) {
            case 8: return launch_drift_bucket<double, 8>(p, k, L_dev, n, b_dev, st);
            case 16: return launch_drift_bucket<double, 16>(p, k, L_dev, n, b_dev, st);
            case 24: return launch_drift_bucket<double, 24>(p, k, L_dev, n, b_dev, st);
            default: return hipErrorInvalidValue;
        }
    }
    switch (p.nmax) {
        case 8: return launch_drift_bucket<float, 8>(p, k, L_dev, n, b_dev, st);
        case 16: return launch_drift_bucket<float, 16>(p, k, L_dev, n, b_dev, st);
        case 20: return launch_drift_bucket<float, 20>(p, k, L_dev, n, b_dev, st);
        case 24: return launch_drift_bucket<float, 24>(p, k, L_dev, n, b_dev, st);
        case 32: return launch_drift_bucket<float, 32>(p, k, L_dev, n, b_dev, st);
        case 40: return launch_drift_bucket<float, 40>(p, k, L_dev, n, b_dev, st);
        default: return hipErrorInvalidValue;
    }
}

PassArgs pass_args(const lll_plan &p) {
    const DeviceTables &d = p.d;
    PassArgs a{};
    a.tenor = d.tenor;
    a.delta = d.delta;
    a.L0 = d.L0;
    a.vol = d.vol;
    a.x = d.x;
    a.w = d.w;
    a.steps = d.steps;
    a.lam_pm = d.lam_pm;
    a.L0s = d.L0s;
    a.deltas = d.deltas;
    a.gx = d.gx;
    a.gw = d.gw;
    a.kappa = d.kappa;
    a.nq = d.nq;
    a.cinv = d.cinv;
    a.ew = d.ew;
    a.lam = d.lam;
    a.drift0 = d.drift0;
    a.frozen = d.frozen;
    a.dt = d.dt;
    a.partials = d.partials;
    a.chunks = d.chunks;
    a.sums = d.sums;
    a.results = d.results;
    a.N = p.N;
    a.s = p.s;
    a.S = p.S;
    a.off = p.off;
    a.nmax = p.nmax;
    a.driver = p.driver;
    a.product = p.product;
    a.alpha = p.alpha;
    a.beta = p.beta;
    a.delta_nig = p.delta_nig;
    a.c = p.c;
    a.B0_T1 = p.B0_T1;
    return a;
}

hipError_t launch_reduce(const lll_plan &p, int64_t n_paths, hipStream_t st) {
    return reduce(pass_args(p), nullptr, 1, p.N * (3 * p.S + 2), n_paths, st);
}

hipError_t launch_reduce_batch(const PassArgs *many, int structures, int64_t n_paths,
                               hipStream_t st) {
    return reduce(PassArgs{}, many, structures, LLL_N_MAX * (3 * LLL_S_MAX + 2), n_paths, st);
}

hipError_t launch_increments(const lll_plan &p, int k, int64_t p0, int64_t n, uint64_t seed,
                             double *V_dev, double *dH_dev, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>((n + kBlock - 1) / kBlock));
    hipLaunchKernelGGL(increments_kernel, grid, dim3(kBlock), 0, st, p.d.steps, k, p.s, p0, n,
                       p.struct_id & 0xFFFFFFu, static_cast<uint32_t>(seed & 0xFFFFFFFFull),
                       static_cast<uint32_t>(seed >> 32),
                       p.driver == LLL_DRIVER_BROWNIAN ? 1 : 0, V_dev, dH_dev);
    return hipGetLastError();
}

hipError_t launch_sampler_math(int fn, const double *x_dev, int64_t n, double *out_dev,
                               hipStream_t st) {
    const dim3 grid(static_cast<unsigned>((n + kBlock - 1) / kBlock));
    hipLaunchKernelGGL(sampler_math_kernel, grid, dim3(kBlock), 0, st, fn, x_dev, n, out_dev);
    return hipGetLastError();
}

hipError_t launch_philox(const uint32_t *ctr_dev, const uint32_t *key_dev, int64_t n,
                         uint32_t *out_dev, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>((n + kBlock - 1) / kBlock));
    hipLaunchKernelGGL(philox_kernel, grid, dim3(kBlock), 0, st, ctr_dev, key_dev, n, out_dev);
    return hipGetLastError();
}

}  // namespace lll
