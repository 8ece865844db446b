// picard_mp.hip -- PICARD in a maturity-parallel layout (few paths, many rates).
//
// Paper Section 3 (eqs. (Picard-2), (bdrift)) and its parallelism remark: under
// the Picard approximation the drift of every rate at step k is evaluated at
// the predictor X1(t_k), which is a function of the driver increments alone and
// never of the other rates' main states.  So the drift integrals of different
// steps are independent given the predictor, and the main state of every rate
// at the tenor dates is a plain sum:
//
//   X_i(T_{m+1}) = sum over the windows up to period m of Z_{window,i},
//   Z_{window,i} = sum_{k in window} (lambda_{k,i} dH_k - kappa_{k,i} dt_k)
//                - sum_{k in window} dt_k C_i(ell(X1(t_k)))   (C_{N-1} = 0),
//
// a window being up to kWindow consecutive steps of one accrual period (5: with 10
// the items hold 132 registers and take 0.28 ms instead of 0.17), C_i the
// coupling of eq. (LIBOR-drift-PT) on the period's Gauss rule.  With one path per
// lane and all of its steps (the path kernel) a run of 10^4 paths fills 157
// wavefronts, a sixth of the SIMDs; here a lane holds a path and a wavefront one
// window, or a few rates, of it:
//
//   0. tables -- (lambda, -kappa dt, b0 dt) and the nodes' (E, -W E dt) of each
//      (step, rate) in one record, read as wave-uniform scalars;
//   1. increments -- one thread per (path, step);
//   2. predictor -- a wavefront per (64 paths, window): the window's move of X1; then
//      a wavefront per (64 paths, rate): running sums, X1 at each window's start;
//   3. items -- a wavefront per (64 paths, window): the suffix recursion of the
//      path kernel over the rates, the window's steps side by side (independent
//      chains) and the nodes in registers;
//   4. states -- running sums of Z per rate, the states at the windows' ends;
//   5. payoffs -- a wavefront per (64 paths, fixing): the payoff quantities, formula
//      and partial sums of the path kernel.
//
// Everything is stored per 64 paths in rows of 64 lanes.  What bounds it: the vector
// ALU in the items (per rate and step an exponential and a reciprocal, and three
// FMAs per node).  N = 60, 10^4 paths: 0.545 ms a pass, of which the items 0.167; with the
// nodes on the lanes of a wavefront (64 of them, 4 paths a wavefront, ell^ of every
// step stored by a prologue, 736 MB) they took 1.64 ms and the pass 2.1 ms.
#include <hip/hip_runtime.h>

#include "lll_device.hpp"
#include "lll_internal.hpp"
#include "path_kernel.hpp"

namespace lll {
namespace {

using detail::as_const;
using detail::cptr;

constexpr int kWindow = 5;                // steps per window at most
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kRec = 4 + 2 * kQ;          // floats per (step, rate) record

struct MpArgs {
    cptr<float> rec;                  // [K][N][kRec]: lam, -kappa dt, b0 dt, 0, (E, -W E dt)[q]
    cptr<float> lam, frozen, cinv;    // [K][nmax], [K][nmax], [nmax]
    cptr<int> nq;                     // [K]
    cptr<double> steps;               // [N][4]
    float *__restrict__ x1;           // [W][rows][64] predictor at each window's start
    float *__restrict__ z;            // [W][rows][64] state increments of each window
    float *__restrict__ dh;           // [W][K][64] driver increments
    int64_t path_base;                // global index of the chunk's first path
    int W, N, s, K, off, nmax;        // W wavefronts of 64 paths
    int windows, steps_each;          // per period
    uint32_t stream_word, key0, key1;
};

__host__ __device__ inline int windows_of(int s) { return (s + kWindow - 1) / kWindow; }
// Rows of 64 lanes per wavefront: the live rates of every window; row of rate r in
// window w of period m (r >= m).
__host__ __device__ inline int64_t window_rows(int s, int N) {
    return (int64_t)windows_of(s) * N * (N + 1) / 2;
}
__device__ __forceinline__ int64_t window_row(const MpArgs &a, int m, int w, int r) {
    return (int64_t)a.windows * (m * a.N - m * (m - 1) / 2) + w * (a.N - m) + (r - m);
}

// Records of step k, zero past the period's node count up to a multiple of 8.
// One block per step.
__global__ void __launch_bounds__(256) mp_tables_kernel(
    const double *__restrict__ tenor, const double *__restrict__ vol,
    const double *__restrict__ gx, const double *__restrict__ gw, const int *__restrict__ nq_in,
    const float *__restrict__ lam, const float *__restrict__ drift0,
    const float *__restrict__ frozen, int N, int s, int off, int nmax, float *__restrict__ rec) {
    const int k = blockIdx.x, m = k / s;
    const double dt = (tenor[m] - (m == 0 ? 0.0 : tenor[m - 1])) / s;
    const int nq = nq_in[k], n8 = (nq + 7) / 8 * 8;
    for (int i = threadIdx.x; i < N * n8; i += 256) {
        const int r = i / n8, q = i % n8;
        float e = 0.0f, we = 0.0f;
        if (q < nq && r >= m) {
            const double E = expm1(vol[(size_t)k * N + r] * gx[m * kQ + q]);
            e = static_cast<float>(E);
            we = static_cast<float>(-gw[m * kQ + q] * dt * E);
        }
        float *o = rec + ((size_t)k * N + r) * kRec + 4 + 2 * q;
        o[0] = e;
        o[1] = we;
    }
    for (int r = threadIdx.x; r < N; r += 256) {
        float *o = rec + ((size_t)k * N + r) * kRec;
        const size_t j = (size_t)k * nmax + off + r;
        o[0] = lam[j];
        o[1] = drift0[j];
        o[2] = frozen[j];
        o[3] = 0.0f;
    }
}

// Driver increments of the chunk's paths, one thread per (path, step) (the
// FP64 sampler needs the occupancy of a flat grid), FP32 as the path kernel
// uses them; a block takes 4 steps of 64 paths.
__global__ void __launch_bounds__(kBlock) mp_increments_kernel(MpArgs a) {
    const int per = (a.K + kWavesPerBlock - 1) / kWavesPerBlock;
    const int wave = blockIdx.x / per;
    const int k = blockIdx.x % per * kWavesPerBlock +
                  __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (k >= a.K) return;
    const int lane = threadIdx.x % kWave;
    const uint64_t path = static_cast<uint64_t>(a.path_base + (int64_t)wave * kWave + lane);
    const cptr<double> sc = a.steps + 4 * (k / a.s);
    const StepConsts cst{sc[0], sc[1], sc[2], sc[3]};
    const uint4 w = philox4x32_10(make_uint4(static_cast<uint32_t>(k), static_cast<uint32_t>(path),
                                             static_cast<uint32_t>(path >> 32), a.stream_word),
                                  a.key0, a.key1);
    a.dh[((int64_t)wave * a.K + k) * kWave + lane] =
        static_cast<float>(increment(w, cst, false, nullptr));
}

// A block takes one window of 4 wavefronts of paths (they read the same tables),
// windows in time order: those with the most live rates first.  Wavefront of paths,
// period and window of this wavefront; false past the last path.
__device__ __forceinline__ bool window_wave(const MpArgs &a, int &wave, int &m, int &w) {
    const int blocks = (a.W + kWavesPerBlock - 1) / kWavesPerBlock;
    const int win = blockIdx.x / blocks;
    wave = blockIdx.x % blocks * kWavesPerBlock +
           __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    m = win / a.windows;
    w = win % a.windows;
    return wave < a.W;
}

// Each window's step of the predictor, sum over its steps of lambda dH + b0 dt, by
// rate; a wavefront per (64 paths, window).
__global__ void __launch_bounds__(kBlock) mp_moves_kernel(MpArgs a) {
    int wave, m, w;
    if (!window_wave(a, wave, m, w)) return;
    const int lane = threadIdx.x % kWave, N = a.N;
    const int k0 = m * a.s + w * a.steps_each;
    const int ns = min(a.steps_each, a.s - w * a.steps_each);
    const float *dh = a.dh + ((int64_t)wave * a.K + k0) * kWave + lane;
    float *x1 = a.x1 + ((int64_t)wave * window_rows(a.s, N) + window_row(a, m, w, m)) * kWave + lane;
    float d[kWindow];
    cptr<float> lam[kWindow], frz[kWindow];
#pragma unroll
    for (int u = 0; u < kWindow; ++u) {
        const int k = k0 + min(u, ns - 1);
        d[u] = dh[(k - k0) * kWave];
        lam[u] = a.lam + (size_t)k * a.nmax + a.off;
        frz[u] = a.frozen + (size_t)k * a.nmax + a.off;
    }
#pragma unroll 4
    for (int r = m; r < N; ++r) {
        float x = 0.0f;
#pragma unroll
        for (int u = 0; u < kWindow; ++u)
            x += u < ns ? fmaf(lam[u][r], d[u], frz[u][r]) : 0.0f;
        x1[(r - m) * kWave] = x;
    }
}

// Running sums over the windows of a rate's life, in place: of the windows before
// each (the predictor at its start) or up to and including it (the states).  A
// wavefront per (64 paths, rate), eight windows' loads in flight.
template <bool kInclusive>
__global__ void __launch_bounds__(kBlock) mp_prefix_kernel(MpArgs a, float *__restrict__ v) {
    const int i = blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wave = i / a.N, r = a.N - 1 - i % a.N;  // the longest lives first
    if (wave >= a.W) return;
    float *col = v + (int64_t)wave * window_rows(a.s, a.N) * kWave + threadIdx.x % kWave;
    const int n = (r + 1) * a.windows;
    float x = 0.0f;
    for (int t0 = 0; t0 < n; t0 += 8) {
        float y[8];
        int64_t at[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int t = min(t0 + u, n - 1);
            at[u] = window_row(a, t / a.windows, t % a.windows, r) * kWave;
            y[u] = col[at[u]];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (t0 + u < n) {
                if constexpr (kInclusive) col[at[u]] = x += y[u];
                else {
                    col[at[u]] = x;
                    x += y[u];
                }
            }
    }
}

// One window of 64 paths on NG nodes a time.  R[u][q] is prod_{l>i}(1 + ell^_l E_{l,q}) - 1
// at the window's step u, advanced from the last rate down as in the path kernel.
// NS: steps of the window (the step loops carry no branches).
template <int NS, int NG>
__device__ __forceinline__ void mp_window(const MpArgs &a, int m, int k0, int nq,
                                          const float *__restrict__ x1, float *__restrict__ z,
                                          const float *__restrict__ dh) {
    const int N = a.N;
    float d[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) d[u] = dh[u * kWave];
    for (int q0 = 0; q0 < nq; q0 += NG) {
        float R[NS][NG];
#pragma unroll
        for (int u = 0; u < NS; ++u)
#pragma unroll
            for (int q = 0; q < NG; ++q) R[u][q] = 0.0f;
        float x = x1[(N - 1 - m) * kWave];
        for (int r = N - 1; r >= m; --r) {
            // the next rate's predictor, ahead of this rate's arithmetic
            const float xn = x1[max(r - 1 - m, 0) * kWave];
            float acc = q0 == 0 ? 0.0f : z[(r - m) * kWave];
            const float ci = a.cinv[a.off + r];
            cptr<float> rec = a.rec + ((size_t)k0 * N + r) * kRec;
#pragma unroll
            for (int u = 0; u < NS; ++u, rec += (size_t)N * kRec) {
                const float lam = rec[0];
                const cptr<float> e = rec + 4 + 2 * q0;
                const float ell = detail::ell_of(x, ci);
                float c = q0 == 0 ? rec[1] : 0.0f;
#pragma unroll
                for (int q = 0; q < NG; ++q) c = fmaf(e[2 * q + 1], R[u][q], c);
                acc += q0 == 0 ? fmaf(lam, d[u], c) : c;
#pragma unroll
                for (int q = 0; q < NG; ++q)
                    R[u][q] = fmaf(ell, fmaf(e[2 * q], R[u][q], e[2 * q]), R[u][q]);
                x += fmaf(lam, d[u], rec[2]);
            }
            z[(r - m) * kWave] = acc;
            x = xn;
        }
    }
}

template <int NS>
__device__ __forceinline__ void mp_window_nodes(const MpArgs &a, int m, int k0, const float *x1,
                                                float *z, const float *dh) {
    const int nq = a.nq[k0];
    // the node counts of the rules are 3, 4, 5, 6, 7, 8, 10, ...: up to 8 in one go
    if (nq <= 4) mp_window<NS, 4>(a, m, k0, nq, x1, z, dh);
    else if (nq <= 6) mp_window<NS, 6>(a, m, k0, nq, x1, z, dh);
    else mp_window<NS, 8>(a, m, k0, nq, x1, z, dh);
}

__global__ void __launch_bounds__(kBlock) mp_item_kernel(MpArgs a) {
    int wave, m, w;
    if (!window_wave(a, wave, m, w)) return;
    const int lane = threadIdx.x % kWave;
    const int k0 = m * a.s + w * a.steps_each;
    const int ns = min(a.steps_each, a.s - w * a.steps_each);
    const int64_t row = ((int64_t)wave * window_rows(a.s, a.N) + window_row(a, m, w, m)) * kWave + lane;
    const float *dh = a.dh + ((int64_t)wave * a.K + k0) * kWave + lane;
    switch (ns) {
        case 1: mp_window_nodes<1>(a, m, k0, a.x1 + row, a.z + row, dh); break;
        case 2: mp_window_nodes<2>(a, m, k0, a.x1 + row, a.z + row, dh); break;
        case 3: mp_window_nodes<3>(a, m, k0, a.x1 + row, a.z + row, dh); break;
        case 4: mp_window_nodes<4>(a, m, k0, a.x1 + row, a.z + row, dh); break;
        case 5: mp_window_nodes<5>(a, m, k0, a.x1 + row, a.z + row, dh); break;
        default: break;
    }
}

// Payoffs of the fixing of rate m for 64 paths.
__global__ void __launch_bounds__(kBlock) mp_payoff_kernel(detail::PathArgs<float> a, MpArgs mp,
                                                           int64_t chunk_first) {
    const int i = blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wave = i / a.N, m = i % a.N;
    if (wave >= mp.W) return;
    const int lane = threadIdx.x % kWave;
    const float *x = mp.z + ((int64_t)wave * window_rows(a.s, a.N) + window_row(mp, m, mp.windows - 1, m)) * kWave +
                     lane;
    double Q = 1.0, A = 0.0, D = 1.0, Lc = 0.0;
    for (int r = a.N - 1; r >= m; --r) {
        const int j = a.off + r;
        const double L = a.L0s[j] * static_cast<double>(exp(x[(r - m) * kWave]));
        if (r == m) {
            D = Q;
            Lc = L;
        }
        A = fma(a.deltas[j], Q, A);
        Q *= 1.0 + a.deltas[j] * L;
    }
    const int64_t gid = chunk_first + (int64_t)wave * kWave + lane;
    detail::fixing_sums(a, m, gid, gid < a.n_paths, a.product == LLL_SWAPTIONS, Q, A, D, Lc);
}

int blocks_for(int64_t waves) { return static_cast<int>((waves + kWavesPerBlock - 1) / kWavesPerBlock); }

}  // namespace

int64_t picard_mp_chunk(const lll_plan &p) {
    // paths per chunk: a multiple of 256 with predictor, Z and increments within
    // kMpBufferBytes (and within 2^30 wavefront items)
    const int64_t per_path = (2 * window_rows(p.s, p.N) + (int64_t)p.K) * (int64_t)sizeof(float);
    int64_t c = kMpBufferBytes / per_path;
    const int64_t items = (int64_t(1) << 30) / ((int64_t)p.K + p.N) * kWave;
    if (c > items) c = items;
    c = c / kBlock * kBlock;
    if (c < kBlock) c = kBlock;
    const int64_t need = (p.max_paths + kBlock - 1) / kBlock * kBlock;
    return c < need ? c : need;
}

hipError_t picard_mp_alloc(lll_plan &p) {
    if (p.d.mp_x1) return hipSuccess;
    const int64_t chunk = picard_mp_chunk(p);
    hipError_t e = hipMalloc(&p.d.mp_rec, (size_t)p.K * p.N * kRec * sizeof(float));
    if (e == hipSuccess)
        e = hipMalloc(&p.d.mp_x1, (size_t)chunk * (2 * window_rows(p.s, p.N) + p.K) * sizeof(float));
    if (e != hipSuccess) {
        picard_mp_free(p);
        return e;
    }
    p.mp_chunk = chunk;
    return hipSuccess;
}

void picard_mp_free(lll_plan &p) {
    (void)hipFree(p.d.mp_rec);
    (void)hipFree(p.d.mp_x1);
    p.d.mp_rec = nullptr;
    p.d.mp_x1 = nullptr;
    p.mp_chunk = 0;
}

hipError_t launch_picard_mp(const lll_plan &p, int64_t n_paths, int64_t path_offset,
                            uint64_t seed, double *path_fix, hipStream_t st) {
    const detail::PathArgs<float> pa =
        detail::make_args<float>(p, seed, n_paths, path_offset, path_fix);
    const DeviceTables &d = p.d;
    hipLaunchKernelGGL(mp_tables_kernel, dim3(p.K), dim3(256), 0, st, d.tenor, d.vol, d.gx, d.gw,
                       d.nq, static_cast<const float *>(d.lam),
                       static_cast<const float *>(d.drift0), static_cast<const float *>(d.frozen),
                       p.N, p.s, p.off, p.nmax, d.mp_rec);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t rows = window_rows(p.s, p.N);
    MpArgs a;
    a.rec = as_const<float>(d.mp_rec);
    a.lam = pa.lam;
    a.frozen = pa.frozen;
    a.cinv = pa.cinv;
    a.nq = pa.nq;
    a.steps = pa.steps;
    a.x1 = d.mp_x1;
    a.z = a.x1 + p.mp_chunk * rows;
    a.dh = a.z + p.mp_chunk * rows;
    a.N = p.N;
    a.s = p.s;
    a.K = p.K;
    a.off = p.off;
    a.nmax = p.nmax;
    a.windows = windows_of(p.s);
    a.steps_each = (p.s + a.windows - 1) / a.windows;
    a.stream_word = pa.stream_word;
    a.key0 = pa.key0;
    a.key1 = pa.key1;
    for (int64_t first = 0; first < n_paths; first += p.mp_chunk) {
        const int64_t n_chunk = n_paths - first < p.mp_chunk ? n_paths - first : p.mp_chunk;
        a.path_base = path_offset + first;
        a.W = static_cast<int>((n_chunk + kWave - 1) / kWave);
        const int rate_blocks = blocks_for((int64_t)a.W * p.N);
        const int window_blocks = blocks_for(a.W) * p.N * a.windows;
        hipLaunchKernelGGL(mp_increments_kernel, dim3(a.W * blocks_for(p.K)), dim3(kBlock), 0, st, a);
        hipLaunchKernelGGL(mp_moves_kernel, dim3(window_blocks), dim3(kBlock), 0, st, a);
        hipLaunchKernelGGL(mp_prefix_kernel<false>, dim3(rate_blocks), dim3(kBlock), 0, st, a, a.x1);
        hipLaunchKernelGGL(mp_item_kernel, dim3(window_blocks), dim3(kBlock), 0, st, a);
        hipLaunchKernelGGL(mp_prefix_kernel<true>, dim3(rate_blocks), dim3(kBlock), 0, st, a, a.z);
        hipLaunchKernelGGL(mp_payoff_kernel, dim3(blocks_for((int64_t)a.W * p.N)), dim3(kBlock), 0,
                           st, pa, a, first);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lll
