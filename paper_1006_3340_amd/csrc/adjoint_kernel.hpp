// adjoint_kernel.hpp -- pathwise adjoint of the caplet prices (FULL scheme, FP32).
//
// Caplet i's price is delta_i B(0, T_*) E[f_i], f_i = D_i (L_i(T_i) - K)^+,
// D_i = prod_{l>i}(1 + delta_l L_l(T_i)) (paper Section 3.3, eq. (caplet)).
// For every path the kernel differentiates f_i with respect to the initial
// forwards L(0, T_l) and to a parallel shift of each rate's volatility curve
// lambda(., T_l), by reverse-mode differentiation of the Euler recursion
//     X_l <- X_l - kappa(lambda_l) dt - C_l dt + lambda_l dH,
//     C_l = sum_q W_q E_{l,q} (P_{l,q} - 1),  P_{l,q} = prod_{m>l} (1 + ell_m E_{m,q}),
// (eq. (LIBOR-drift-PT) with the quadrature rule), E_{l,q} = e^{lambda_l x_q} - 1,
// ell_l = delta_l L_l / (1 + delta_l L_l), L_l = L(0, T_l) e^{X_l}.
//
// Rate i depends only on rates l >= i, so the sweep of caplet i carries only
// those.  Memory: the forward pass keeps the live rates at the start of every step
// (packed, s N (N+1) / 2 floats per path), the increments and the fixing of every
// rate, and the sweeps read them back, a step ahead of their use; paths go in
// chunks (state_chunk.hpp).  Recomputing each period from a checkpoint at its tenor date
// instead (an increment, a FULL step and the same traffic through a scratch, per step)
// and three table entries per rate and node took price and gradient of 40 rates from
// 12.4 to 15.5 ms at 2^18 paths, the Jacobian from 33 to 66 ms at 2^17.  What bounds it
// now is the vector ALU at the two wavefronts per SIMD that 9 registers per rate leave the
// wide sweeps: 0.41 of the FP32 peak.
//
// Reverse of one step, per node q (the suffix products less one, R_l = P_l - 1, by a
// downward pass, then an upward pass with F_l = sum_{i<l} Cbar_i W E_{i,q}
// prod_{i<m<l} beta_m):
//     R_{l-1}   = R_l + ell_l E_{l,q} (1 + R_l),
//     ellbar_l += E_{l,q} P_l F_l,    P_l F_l = R_l F_l + F_l,
//     Ebar_l    = Cbar_l W_q R_l + ell_l P_l F_l,  lambdabar_l += x_q e^{lambda_l x_q} Ebar_l
//     F_{l+1}   = (1 + ell_l E_{l,q}) F_l + Cbar_l W_q E_{l,q},     Cbar_l = -dt Xbar_l,
// with W_q taken into Xbar, so that E is the only table entry per rate and
// node: a node's row then fits the scalar registers in one batch of loads
// (gradient kernels 10.2 -> 8.1 ms at 2^18 paths),
// then Xbar_l += ellbar_l ell_l (1 - ell_l), L0bar_l += ellbar_l ell_l (1 - ell_l) / L(0, T_l),
// lambdabar_l += Xbar_l (dH - kappa'(lambda_l) dt).  L0bar_l L(0, T_l) collects the
// same terms as Xbar_l, from the payoff's adjoint down to step 0, and its wavefront sum
// is scaled by 1 / L(0, T_l) once.  It has an accumulator of its own: a step moves Xbar
// by about dt times the drift's derivative, which the rounding of Xbar itself swallows when
// the steps are many (taken from Xbar at the start, vector-Jacobian products were 1e-5
// off FP64 at 400 steps a period; 1e-8 to 2e-8 with the accumulators).
// The products are carried less one because a node of a period's rule can lie next to the
// origin and hold most of the coupling: P - 1 formed from P is then P's FP32 rounding, and
// the vol adjoints of 12 rates were 2e-3 to 3e-3 of their norm off FP64 with a node within
// 1e-5 of it; 1e-7 to 4e-7 this way, at the same operation count.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "lll_device.hpp"
#include "lll_internal.hpp"
#include "path_kernel.hpp"

namespace lll {
namespace adj {

using detail::cptr;
using detail::PathArgs;

constexpr int kAdjBlock = 64;  // one wavefront per block: per-lane accumulators in LDS

struct AdjArgs {
    cptr<float> E;         // [K][Q][nmax]  e^{lambda x_q} - 1
    cptr<float> dkap;      // [K][nmax]     kappa'(lambda) dt
    cptr<float> xw;        // [N][Q][2]     nodes and weights of each period
    cptr<double> inv_L0;   // [nmax]        1 / L(0, T)
    // per wavefront, rows of 64 lanes (a rate's row is a constant distance from the
    // next one's, so a step's loads share one address): s N (N+1) / 2 rows of states
    // (live rates at the start of each step), K of increments, N of fixings, N of
    // the state adjoint carried between the periods of a vector-Jacobian product
    float *rows;
    int64_t n_rows;        // rows per wavefront
    double *gpart;         // [waves][N][2N] per-wave sums of L0bar (first N) and vbar
};

// This lane's column of its wavefront's rows.
__device__ __forceinline__ float *lane_rows(const AdjArgs &g, int64_t gid) {
    return g.rows + (gid / kWave) * g.n_rows * kWave + gid % kWave;
}

// Offsets in a lane's column: rate r at the start of step js of period m (r >= m),
// the increment of step k, the fixing of rate r, its carried adjoint.
__device__ __forceinline__ int64_t at_state(const PathArgs<float> &a, int m, int js, int r) {
    return kWave * (static_cast<int64_t>(a.s) * (m * a.N - (m * (m - 1)) / 2) + js * (a.N - m) +
                    (r - m));
}
__device__ __forceinline__ int64_t at_dh(const PathArgs<float> &a, int k) {
    return kWave * (static_cast<int64_t>(a.s) * (a.N * (a.N + 1) / 2) + k);
}
__device__ __forceinline__ int64_t at_fix(const PathArgs<float> &a, int r) {
    return at_dh(a, a.N * a.s) + kWave * r;
}
__device__ __forceinline__ int64_t at_xb(const PathArgs<float> &a, int r) {
    return at_fix(a, a.N) + kWave * r;
}

__device__ __forceinline__ float increment_f(const PathArgs<float> &a, int k, int m, uint32_t p_lo,
                                             uint32_t p_hi) {
    const cptr<double> sc = a.steps + 4 * m;
    const StepConsts cst{sc[0], sc[1], sc[2], sc[3]};
    const uint4 w = philox4x32_10(make_uint4(static_cast<uint32_t>(k), p_lo, p_hi, a.stream_word),
                                  a.key0, a.key1);
    return static_cast<float>(increment(w, cst, a.brownian != 0, nullptr));
}

template <int NMAX, int J0>
__device__ __forceinline__ void store_state(const PathArgs<float> &a, int m, int js, float *d,
                                            const float (&X)[NMAX]) {
    float *row = d + at_state(a, m, js, J0 - a.off);
#pragma unroll
    for (int j = J0; j < NMAX; ++j) row[(j - J0) * kWave] = X[j];
}

template <int NMAX, int... Js>
__device__ __forceinline__ void dispatch_store(std::integer_sequence<int, Js...>, int j0,
                                               const PathArgs<float> &a, int m, int js, float *d,
                                               const float (&X)[NMAX]) {
    (void)((j0 == Js ? (store_state<NMAX, Js>(a, m, js, d, X), 0) : 0) + ...);
}

// Forward FULL pass that keeps its states; also the price partials of PRODUCT
// (LLL_CAPLETS or LLL_SWAPTIONS, fixed at compile time: the product's payoff
// code is inlined at every fixing date).
template <int NMAX, int PRODUCT>
__device__ void forward(const PathArgs<float> &a, const AdjArgs &g, int64_t gid, bool active) {
    const int64_t p = a.path_offset + gid;
    const uint32_t p_lo = static_cast<uint32_t>(p);
    const uint32_t p_hi = static_cast<uint32_t>(static_cast<uint64_t>(p) >> 32);
    float X[NMAX], X1[NMAX];
    float *d = lane_rows(g, gid);
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
        X[j] = 0.0f;
        X1[j] = 0.0f;
    }
    for (int m = 0; m < a.N; ++m) {
        const int j0 = a.off + m;
        for (int js = 0; js < a.s; ++js) {
            const int k = m * a.s + js;
            const float dH = increment_f(a, k, m, p_lo, p_hi);
            dispatch_store<NMAX>(std::make_integer_sequence<int, NMAX>{}, j0, a, m, js, d, X);
            d[at_dh(a, k)] = dH;
            detail::dispatch_step<float, NMAX, kFull>(std::make_integer_sequence<int, NMAX>{}, j0,
                                                      a, k, dH, X, X1);
        }
        // X of the rate that fixes now (slot j0), selected from registers
        float xf = 0.0f;
#pragma unroll
        for (int j = 0; j < NMAX; ++j) xf = (j == j0) ? X[j] : xf;
        d[at_fix(a, m)] = xf;
        detail::dispatch_payoff<float, NMAX, PRODUCT>(std::make_integer_sequence<int, NMAX>{}, j0,
                                                      a, m, gid, active, X);
    }
}

// The same forward pass with the state in the block's LDS columns, as the
// plain FP32 FULL path kernels of the 24- to 40-slot buckets run it (same
// step and payoff code, so the same prices bit for bit): X, ell and the
// coupling sums do not all fit the registers of two wavefronts per SIMD.
template <int NMAX, int PRODUCT>
__device__ void forward_lds(const PathArgs<float> &a, const AdjArgs &g, int64_t gid, bool active) {
    float *xs = detail::state_lds<float, NMAX>() + threadIdx.x;
    const int64_t p = a.path_offset + gid;
    const uint32_t p_lo = static_cast<uint32_t>(p);
    const uint32_t p_hi = static_cast<uint32_t>(static_cast<uint64_t>(p) >> 32);
    float X1[NMAX];
    float *d = lane_rows(g, gid);
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
        xs[j * kBlock] = 0.0f;
        X1[j] = 0.0f;
    }
    for (int m = 0; m < a.N; ++m) {
        const int j0 = a.off + m;
        for (int js = 0; js < a.s; ++js) {
            const int k = m * a.s + js;
            const float dH = increment_f(a, k, m, p_lo, p_hi);
            float *row = d + at_state(a, m, js, m);
            for (int j = j0; j < NMAX; ++j, row += kWave) *row = xs[j * kBlock];
            d[at_dh(a, k)] = dH;
            detail::dispatch_step_lds<float, NMAX, kFull>(std::make_integer_sequence<int, NMAX>{}, j0,
                                                          a, k, dH, xs, X1);
        }
        d[at_fix(a, m)] = xs[j0 * kBlock];
        detail::payoff_lds<float, NMAX, PRODUCT>(a, m, gid, active, xs, j0);
    }
}

// X of the slots JC .. NMAX-1 at the start of step js of period m.
template <int NMAX, int JC>
__device__ __forceinline__ void load_state(const PathArgs<float> &a, int m, int js, const float *d,
                                           float (&X)[NMAX]) {
    const float *row = d + at_state(a, m, js, JC - a.off);
#pragma unroll
    for (int j = JC; j < NMAX; ++j) X[j] = row[(j - JC) * kWave];
}

// X at the start of the step before step js of period m.
template <int NMAX, int JC>
__device__ __forceinline__ void load_before(const PathArgs<float> &a, int m, int js,
                                            const float *d, float (&X)[NMAX]) {
    if (js > 0) load_state<NMAX, JC>(a, m, js - 1, d, X);
    else load_state<NMAX, JC>(a, m - 1, a.s - 1, d, X);
}

// A reverse step holds X (loaded ahead), ell, Xb, R, lb, vb, a temporary and the two
// accumulators per rate: 9 registers, two wavefronts per SIMD up to 26 rates.  Beyond,
// the accumulators stay in LDS; beyond 34 rates, X is loaded after the node loop instead of
// ahead of it.
template <int NMAX, int JC>
constexpr bool kAccInLds = NMAX - JC > 26;
template <int NMAX, int JC>
constexpr bool kLoadAhead = NMAX - JC <= 34;

// Reverse of step js of period m for the slots JC .. NMAX-1, given the state X
// at the start of the step and Xb = adjoint of the state at its end (updated in
// place to the adjoint at the start); X is then loaded with the state of the step
// before.  The adjoints of L0 (times L0) and of the vol go to the lane's accumulators
// acc[2 i] and acc[2 i + 1] of slot JC + i, in rows of kAdjBlock.
template <int NMAX, int JC>
__device__ __forceinline__ void reverse_step(const PathArgs<float> &a, const AdjArgs &g, int m,
                                             int js, const float *d, float (&X)[NMAX],
                                             float (&Xb)[NMAX], float *__restrict__ acc) {
    // Cbar = -dt Xbar: the factor -dt is applied to lb after the node loop and to
    // the node x in the vol adjoints
    const int k = m * a.s + js;
    const float dH = d[at_dh(a, k)];
    const float mdt = -a.dt[k];
    const cptr<float> dk = g.dkap + (size_t)k * NMAX;
    if constexpr (kAccInLds<NMAX, JC>) __asm__ volatile("" ::: "memory");
    float ell[NMAX], lb[NMAX], vb[NMAX], R[NMAX];
#pragma unroll
    for (int j = JC; j < NMAX; ++j) {
        ell[j] = detail::ell_of(X[j], a.cinv[j]);
        lb[j] = 0.0f;
        vb[j] = 0.0f;
    }
    if (kLoadAhead<NMAX, JC> && k > 0) load_before<NMAX, JC>(a, m, js, d, X);
    cptr<float> row = g.E + (size_t)k * kQ * NMAX;
    const int nq = a.nq[k];
#pragma unroll 1
    for (int q = 0; q < nq; ++q, row += NMAX) {
        const float x = g.xw[2 * (m * kQ + q)] * mdt, W = g.xw[2 * (m * kQ + q) + 1];
        R[NMAX - 1] = 0.0f;  // suffix products less one
#pragma unroll
        for (int j = NMAX - 2; j >= JC; --j)
            R[j] = fmaf(ell[j + 1], fmaf(row[j + 1], R[j + 1], row[j + 1]), R[j + 1]);
        float F = 0.0f;  // F of the header / -dt
#pragma unroll
        for (int j = JC; j < NMAX; ++j) {
            const float E = row[j];
            const float WX = W * Xb[j];
            const float G = fmaf(R[j], F, F);
            lb[j] = fmaf(E, G, lb[j]);
            const float xEb = x * fmaf(WX, R[j], ell[j] * G);
            vb[j] = fmaf(E, xEb, vb[j] + xEb);  // x e^{lambda x} Ebar = x (1 + E) Ebar
            F = fmaf(E, fmaf(ell[j], F, WX), F);
        }
    }
#pragma unroll
    for (int j = JC; j < NMAX; ++j) {
        acc[(2 * (j - JC) + 1) * kAdjBlock] += fmaf(Xb[j], dH - dk[j], vb[j]);
        const float move = lb[j] * mdt * ell[j] * (1.0f - ell[j]);
        acc[2 * (j - JC) * kAdjBlock] += move;
        Xb[j] += move;
    }
    if (!kLoadAhead<NMAX, JC> && k > 0) {
        __asm__ volatile("" ::: "memory");
        load_before<NMAX, JC>(a, m, js, d, X);
    }
}

// Xb = w times the payoff adjoint of product c (strike 0; slot JC = off + c)
// at its fixing date T_{c+1}, and X = the fixing state.
//   caplet:   f = D (L_c - K)^+, D = prod_{l>c}(1 + delta_l L_l);
//   swaption: f = (Q - 1 - K A)^+, Q = prod_{l>=c} b_l, b_l = 1 + delta_l L_l,
//             A = sum_{l>=c} delta_l prod_{j>l} b_j, so that with
//             S_l = sum_{c<=m<l} delta_m prod_{j>m} b_j = sum_{c<=m<l} delta_m Q / prod_{c<=j<=m} b_j
//             df/dX_l = ell_l (Q - K S_l) where the payoff is positive.
// The direct L0 terms are df/dX_l / L(0, T_l) (L = L(0,T) e^X at fixed X).  The
// scheduling barriers keep the FP64 quantities of one rate at a time in registers:
// interleaved over the rates they set the register count of the whole sweep (330
// at 40 rates, one wavefront per SIMD).
template <int NMAX, int JC>
__device__ __forceinline__ void seed_caplet(const PathArgs<float> &a, const float *d,
                                            bool active, float w, float (&X)[NMAX],
                                            float (&Xb)[NMAX]) {
    const int c = JC - a.off;
    X[JC] = d[at_fix(a, c)];
    if constexpr (JC + 1 < NMAX) load_state<NMAX, JC + 1>(a, c + 1, 0, d, X);
    if (a.product == LLL_SWAPTIONS) {
        double Q = 1.0, A = 0.0;
#pragma unroll
        for (int j = NMAX - 1; j >= JC; --j) {
            const double b = 1.0 + a.deltas[j] * (a.L0s[j] * static_cast<double>(expf(X[j])));
            A = fma(a.deltas[j], Q, A);
            Q *= b;
            __builtin_amdgcn_sched_barrier(0);
        }
        const double K = a.strikes[c * a.S];
        const bool itm = active && ((Q - 1.0) - K * A > 0.0);
        double pre = 1.0, S = 0.0;
#pragma unroll
        for (int j = JC; j < NMAX; ++j) {
            const double L = a.L0s[j] * static_cast<double>(expf(X[j]));
            const double b = 1.0 + a.deltas[j] * L;
            Xb[j] = itm ? w * static_cast<float>(a.deltas[j] * L / b * (Q - K * S)) : 0.0f;
            pre *= b;
            S = fma(a.deltas[j], Q / pre, S);
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
    double D = 1.0;
    float ellf[NMAX];
#pragma unroll
    for (int j = JC + 1; j < NMAX; ++j) {
        const double L = a.L0s[j] * static_cast<double>(expf(X[j]));
        D *= 1.0 + a.deltas[j] * L;
        ellf[j] = static_cast<float>(a.deltas[j] * L / (1.0 + a.deltas[j] * L));
        __builtin_amdgcn_sched_barrier(0);
    }
    const double Lc = a.L0s[JC] * static_cast<double>(expf(X[JC]));
    const double K = a.strikes[c * a.S];
    const bool itm = active && (Lc > K);
    const float dXc = itm ? w * static_cast<float>(D * Lc) : 0.0f;
    const float dD = itm ? w * static_cast<float>(Lc - K) : 0.0f;
    const float Df = static_cast<float>(D);
    Xb[JC] = dXc;
#pragma unroll
    for (int j = JC + 1; j < NMAX; ++j) Xb[j] = dD * Df * ellf[j];
}

// The accumulators of a sweep or period: the L0 adjoints start at the payoff's.
template <int NMAX, int JC>
__device__ __forceinline__ void start_sums(const float (&Xb)[NMAX], float *__restrict__ acc) {
#pragma unroll
    for (int j = JC; j < NMAX; ++j) {
        acc[2 * (j - JC) * kAdjBlock] = Xb[j];
        acc[(2 * (j - JC) + 1) * kAdjBlock] = 0.0f;
    }
}

// Sweep of the caplet fixing in slot JC (rate c = JC - off, period c).
template <int NMAX, int JC>
__device__ __forceinline__ void sweep(const PathArgs<float> &a, const AdjArgs &g, int64_t gid,
                                      bool active, float *__restrict__ acc) {
    const int lane = threadIdx.x;
    const int c = JC - a.off;
    const int N = a.N;
    const float *d = lane_rows(g, gid);
    acc += lane;
    float X[NMAX], Xb[NMAX];
    seed_caplet<NMAX, JC>(a, d, active, 1.0f, X, Xb);
    start_sums<NMAX, JC>(Xb, acc);
    // skip the sweep when no lane of the wavefront has a nonzero adjoint
    bool any = false;
#pragma unroll
    for (int j = JC; j < NMAX; ++j) any = any || (Xb[j] != 0.0f);
    if (__any(any)) {
        load_state<NMAX, JC>(a, c, a.s - 1, d, X);
        for (int m = c; m >= 0; --m)
            for (int js = a.s - 1; js >= 0; --js)
                reverse_step<NMAX, JC>(a, g, m, js, d, X, Xb, acc);
    }
    // wavefront sums of this caplet's adjoints
    const int64_t wave = gid / kWave;
    double *out = g.gpart + (static_cast<int64_t>(wave) * N + c) * 2 * N;
#pragma unroll
    for (int j = JC; j < NMAX; ++j) {
        const double l0 =
            detail::wave_sum(active ? acc[2 * (j - JC) * kAdjBlock] : 0.0f) * g.inv_L0[j];
        const double vv = detail::wave_sum(active ? acc[(2 * (j - JC) + 1) * kAdjBlock] : 0.0f);
        if (lane == 0) {
            out[j - a.off] = l0;
            out[N + j - a.off] = vv;
        }
    }
    if (lane == 0)
        for (int r = 0; r < c; ++r) {
            out[r] = 0.0;
            out[N + r] = 0.0;
        }
}

// Vector-Jacobian product: one reverse sweep for sum_c g_c f_c.  The kernel of
// period m (slot JC = off + m) continues the sweep from the end of period m:
// it takes the state adjoint carried from period m+1 (xb, by rate), adds the
// seed of caplet m (weight w_m = g_m delta_m) at its fixing, reverses the
// period and stores the adjoint at the period's start; the wavefront sums of
// the period's L0 and vol adjoints are added to the per-wave partials (periods in
// launch order, so the sums are deterministic).
struct VjpArgs {
    double *part;   // [waves][2N] sums of L0bar (first N) and vbar
    detail::cptr<float> w;  // [N] seeds g_m s_m of the products (device memory)
};

template <int NMAX, int JC>
__device__ __forceinline__ void vjp_period(const PathArgs<float> &a, const AdjArgs &g,
                                           const VjpArgs &v, int64_t gid, bool active,
                                           float *__restrict__ acc) {
    const int lane = threadIdx.x;
    const int m = JC - a.off;
    const float w = v.w[m];
    const int N = a.N;
    float *d = lane_rows(g, gid);
    float *xb = d + at_xb(a, m);
    acc += lane;
    float X[NMAX], Xb[NMAX];
    seed_caplet<NMAX, JC>(a, d, active, w, X, Xb);
    start_sums<NMAX, JC>(Xb, acc);
    // rate m is fixed after period m: only the later rates carry an adjoint
    if (m < N - 1) {
#pragma unroll
        for (int j = JC + 1; j < NMAX; ++j) Xb[j] += xb[(j - JC) * kWave];
    }
    bool any = false;
#pragma unroll
    for (int j = JC; j < NMAX; ++j) any = any || (Xb[j] != 0.0f);
    if (__any(any)) {
        load_state<NMAX, JC>(a, m, a.s - 1, d, X);
        for (int js = a.s - 1; js >= 0; --js) reverse_step<NMAX, JC>(a, g, m, js, d, X, Xb, acc);
    }
    if (m > 0) {
#pragma unroll
        for (int j = JC; j < NMAX; ++j) xb[(j - JC) * kWave] = Xb[j];
    }
    double *out = v.part + (gid / kWave) * 2 * N;
#pragma unroll
    for (int j = JC; j < NMAX; ++j) {
        const double l0 =
            detail::wave_sum(active ? acc[2 * (j - JC) * kAdjBlock] : 0.0f) * g.inv_L0[j];
        const double vv = detail::wave_sum(active ? acc[(2 * (j - JC) + 1) * kAdjBlock] : 0.0f);
        if (lane == 0) {
            out[j - a.off] += l0;
            out[N + j - a.off] += vv;
        }
    }
}

// One launch per caplet (slot JC): each sweep is its own kernel so that its
// register allocation covers only its own live set.
template <int NMAX, int JC>
__global__ void __launch_bounds__(kAdjBlock, (kAccInLds<NMAX, JC> ? 2 : 1)) sweep_kernel(PathArgs<float> a, AdjArgs g) {
    // per-lane accumulators of the carried slots JC..NMAX-1 only (LDS bounds
    // the resident wavefronts of the long sweeps)
    __shared__ float acc[2 * (NMAX - JC) * kAdjBlock];
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kAdjBlock + threadIdx.x;
    const int64_t wave_first = gid - threadIdx.x;
    if (wave_first >= a.n_paths) return;
    sweep<NMAX, JC>(a, g, gid, gid < a.n_paths, acc);
}

template <int NMAX, int JC>
__global__ void __launch_bounds__(kAdjBlock, (kAccInLds<NMAX, JC> ? 2 : 1))
    vjp_period_kernel(PathArgs<float> a, AdjArgs g, VjpArgs v) {
    __shared__ float acc[2 * (NMAX - JC) * kAdjBlock];
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kAdjBlock + threadIdx.x;
    const int64_t wave_first = gid - threadIdx.x;
    if (wave_first >= a.n_paths) return;
    vjp_period<NMAX, JC>(a, g, v, gid, gid < a.n_paths, acc);
}

template <int NMAX, int PRODUCT>
__global__ void __launch_bounds__(kAdjBlock) forward_kernel(PathArgs<float> a, AdjArgs g) {
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kAdjBlock + threadIdx.x;
    const int64_t wave_first = gid - threadIdx.x;
    if (wave_first >= a.n_paths) return;
    forward<NMAX, PRODUCT>(a, g, gid, gid < a.n_paths);
}

template <int NMAX, int JC>
hipError_t launch_one_sweep(dim3 grid, const PathArgs<float> &a, const AdjArgs &g, hipStream_t st) {
    hipLaunchKernelGGL((sweep_kernel<NMAX, JC>), grid, dim3(kAdjBlock), 0, st, a, g);
    return hipGetLastError();
}

template <int NMAX, int... Js>
hipError_t launch_sweep(std::integer_sequence<int, Js...>, int jc, dim3 grid,
                        const PathArgs<float> &a, const AdjArgs &g, hipStream_t st) {
    hipError_t e = hipErrorInvalidValue;
    (void)((jc == Js ? (e = launch_one_sweep<NMAX, Js>(grid, a, g, st), 0) : 0) + ...);
    return e;
}

template <int NMAX, int JC>
hipError_t launch_one_vjp(dim3 grid, const PathArgs<float> &a, const AdjArgs &g, const VjpArgs &v,
                          hipStream_t st) {
    hipLaunchKernelGGL((vjp_period_kernel<NMAX, JC>), grid, dim3(kAdjBlock), 0, st, a, g, v);
    return hipGetLastError();
}

template <int NMAX, int... Js>
hipError_t launch_vjp(std::integer_sequence<int, Js...>, int jc, dim3 grid, const PathArgs<float> &a,
                      const AdjArgs &g, const VjpArgs &v, hipStream_t st) {
    hipError_t e = hipErrorInvalidValue;
    (void)((jc == Js ? (e = launch_one_vjp<NMAX, Js>(grid, a, g, v, st), 0) : 0) + ...);
    return e;
}

template <int NMAX, int PRODUCT>
__global__ void __launch_bounds__(kBlock) forward_lds_kernel(PathArgs<float> a, AdjArgs g) {
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const int64_t wave_first = gid - (threadIdx.x % kWave);
    if (wave_first >= a.n_paths) return;
    forward_lds<NMAX, PRODUCT>(a, g, gid, gid < a.n_paths);
}

template <int NMAX>
hipError_t launch_forward(dim3 grid, const PathArgs<float> &a, const AdjArgs &g, hipStream_t st) {
    if constexpr (detail::kStateInLds<float, NMAX, kFull>) {
        const dim3 lgrid(static_cast<unsigned>((a.n_paths + kBlock - 1) / kBlock));
        if (a.product == LLL_SWAPTIONS)
            hipLaunchKernelGGL((forward_lds_kernel<NMAX, LLL_SWAPTIONS>), lgrid, dim3(kBlock), 0, st,
                               a, g);
        else
            hipLaunchKernelGGL((forward_lds_kernel<NMAX, LLL_CAPLETS>), lgrid, dim3(kBlock), 0, st, a,
                               g);
    } else {
        if (a.product == LLL_SWAPTIONS)
            hipLaunchKernelGGL((forward_kernel<NMAX, LLL_SWAPTIONS>), grid, dim3(kAdjBlock), 0, st, a,
                               g);
        else
            hipLaunchKernelGGL((forward_kernel<NMAX, LLL_CAPLETS>), grid, dim3(kAdjBlock), 0, st, a, g);
    }
    return hipGetLastError();
}

// Forward pass, then the periods from the last to the first
// (v.w[m] = weight of product m times its price scale; v.part must be zero).
template <int NMAX>
hipError_t launch_vjp_bucket(const PathArgs<float> &a, const AdjArgs &g, const VjpArgs &v,
                             hipStream_t st) {
    const dim3 grid(static_cast<unsigned>((a.n_paths + kAdjBlock - 1) / kAdjBlock));
    hipError_t e = launch_forward<NMAX>(grid, a, g, st);
    for (int m = a.N - 1; m >= 0 && e == hipSuccess; --m)
        e = launch_vjp<NMAX>(std::make_integer_sequence<int, NMAX>{}, a.off + m, grid, a, g, v, st);
    return e;
}

// Forward pass, then one sweep launch per caplet.  The sweeps are independent and
// write their own rows of the partials: they go round the caller's stream and the
// side streams, so that the many of them that leave the SIMDs short of wavefronts
// (2^17 paths: two per SIMD and launch) run beside each other.
template <int NMAX>
hipError_t launch_adjoint_bucket(const PathArgs<float> &a, const AdjArgs &g, const SideStreams &ss,
                                 hipStream_t st) {
    const dim3 grid(static_cast<unsigned>((a.n_paths + kAdjBlock - 1) / kAdjBlock));
    hipError_t e = launch_forward<NMAX>(grid, a, g, st);
    if (e != hipSuccess) return e;
    return run_beside(ss, st, a.N, [&](int c, hipStream_t s) {
        return launch_sweep<NMAX>(std::make_integer_sequence<int, NMAX>{}, a.off + c, grid, a, g, s);
    });
}

}  // namespace adj
}  // namespace lll
