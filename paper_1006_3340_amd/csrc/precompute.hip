// precompute.hip -- FP64 precompute on the device, once per pricing pass.
//
// Paper Section 2, eq. (LIBOR-drift-PT): for the pure-jump NIG driver the
// drift of rate i at step k is
//     b_i = -kappa(lambda_i) - int (e^{lambda_i x} - 1)(prod_{l>i} beta_l(x) - 1) F(dx).
// The cumulant is closed form (Section 4 NIG cumulant, generalised to beta != 0
// with the martingale drift).  The coupling integral uses a fixed 64-node rule:
// 32 Gauss-Legendre points v_j on [0, 1] mapped by x = +-X_pm v^2 on each side,
// weights W = w_j 2 X_pm v_j f(x) with the NIG Lévy density
// f(x) = (delta alpha / pi) e^{beta x} K_1(alpha |x|) / |x|, and truncation
// X_+ = min(36 / (alpha - beta - Lambda_+), 40), X_- = min(36 / (alpha + beta - Lambda_-), 40)
// where Lambda_pm bounds the sum of the live vols' positive / negative parts.
//
// Tables (per step k and live rate slot j), at the nodes x_q of the period's
// Gauss rule (see setup_rule_kernel):
//   E[k][q][j]  = e^{lambda_{k,j} x_q} - 1 and W_q E   (path kernel, interleaved)
//   drift0      = -kappa(lambda_{k,j}) dt_k
//   frozen      = b0 dt_k, b0 the drift at the initial rates (eq. (Picard-2))
// all computed in FP64 and stored in the plan's precision.
#include <hip/hip_runtime.h>

#include "lll_device.hpp"
#include "lll_internal.hpp"

namespace lll {
namespace {

// Positive points (descending) and weights of the 32-point Gauss-Legendre rule
// on [-1, 1] (roots of P_32 and 2 / ((1 - x^2) P_32'(x)^2), from 40-digit
// arithmetic).
__device__ const double kGLx[kGL / 2] = {
    0.9972638618494815635, 0.9856115115452683354, 0.9647622555875064308, 0.9349060759377396892,
    0.896321155766052124, 0.8493676137325699701, 0.794483795967942407, 0.7321821187402896804,
    0.663044266930215201, 0.587715757240762329, 0.50689990893222939, 0.4213512761306353454,
    0.3318686022821276498, 0.2392873622521370745, 0.1444719615827964935, 0.04830766568773831623};
__device__ const double kGLw[kGL / 2] = {
    0.0070186100094700966, 0.01627439473090567061, 0.02539206530926205946, 0.0342738629130214331,
    0.04283589802222668066, 0.0509980592623761762, 0.05868409347853554715, 0.06582222277636184684,
    0.07234579410884850623, 0.07819389578707030647, 0.08331192422694675522, 0.08765209300440381114,
    0.09117387869576388471, 0.09384439908080456564, 0.09563872007927485942, 0.09654008851472780057};

// v of lane i + its DPP image, for the FP64 wavefront sum below.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0u, static_cast<uint32_t>(u), CTRL, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0u, static_cast<uint32_t>(u >> 32), CTRL, 0xF, 0xF, true);
    return v + __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

__device__ __forceinline__ double lane_of(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(u), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(u >> 32), lane);
    return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// Wavefront sum in every lane: within each row of 16 lanes by DPP (quad
// permutes, half-row and row mirror), then the four rows through scalar
// registers.  The rule's set-up is a chain of such sums, and a DPP step takes a
// tenth of a cross-lane LDS permute's latency.
__device__ __forceinline__ double wave_sum_dpp(double v) {
    v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);  // row_half_mirror
    v = dpp_add<0x140>(v);  // row_mirror
    return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}

// The step tables do not hold the 64-node rule itself but, per period, the
// n-point Gauss rule of the same discrete measure, n as small as the plan's
// precision allows.  With p_U the probability that independent Bernoulli(ell_l)
// variables select the subset U of the later rates,
//     prod_{l>i} (1 + ell_l E_l) = sum_U p_U e^{lambda_U x},   lambda_U = sum_{l in U} lambda_l,
// so the coupling is an average of the functions
//     f_{lambda,a}(x) = (e^{lambda x} - 1)(e^{a x} - 1),   lambda = lambda_i, a = lambda_U,
// with a between -Lambda_- and Lambda_+ of the live rates: x^2 e^{theta x} times
// an entire function of exponential type at most about (Lambda_+ + Lambda_-) / 2
// for a tilt theta near (Lambda_+ - Lambda_-) / 2, and the Gauss rule of the tilted
// measure sum_q W_q x_q^2 e^{theta x_q} delta_{x_q} converges geometrically on them
// (error down 50 to 500 times per added node at the light-tailed structures; a
// factor of 0.45 instead of 0.5 balances its ends, halving the largest error).
// f keeps one sign in x, so an error relative to the 64-node sum of f that holds
// at every a bounds the error of every coupling, whatever the state: relative to the
// coupling itself with vols of one sign; with both signs the terms of the average
// cancel, and it is relative to sum_q W |E_i| (prod_{l>i} (1 + ell_l |E_l|) - 1), at whose
// rounding the 64 nodes' own sum stands.  The error is largest at the ends of the range of a:
// each candidate is checked against the 64-node sums at a = Lambda_+, at -Lambda_- and in
// the limit a -> 0 (f / a -> (e^{lambda x} - 1) x), for the smallest and largest live vol
// (the vols between them are not checked one by one), before it is taken:
//   FP32 plans: 2^-30, a 64th of a unit in the last place of the tables;
//   FP64 plans: 2^-47, the rounding of the 64-term sums.
// At 64 nodes FULL spent 15.3 of its 19.1 ms (20 rates, 2^20 paths) in the
// recursion; 4 to 6 nodes suffice there (6 at 40 rates, 8 at 60), 8 to 16 with
// the tails of alpha = 1.5, and near the moment limit, where none of the
// candidates passes, the period keeps the 64 nodes.
constexpr int kCand[] = {3, 4, 5, 6, 7, 8, 10, 12, 16, 24};
constexpr int kNCand = sizeof(kCand) / sizeof(kCand[0]);
constexpr int kFirstCand = 8;    // the candidates of the first round, one per wavefront
constexpr int kGaussFirst = 12;  // their largest node count
constexpr int kGaussMax = 24;
constexpr int kRuleBlock = 64 * kFirstCand;
constexpr double kTolF32 = 9.3132257461547852e-10;   // 2^-30
constexpr double kTolF64 = 7.1054273576010019e-15;   // 2^-47

// The test functions of the acceptance check at one point, times the weight:
// lambda the smallest (l0) and the largest (l1) live vol of the period, a the
// largest positive (ap) and negative (am) subset sum and the limit a -> 0.
struct TestVols {
    double l0, l1, ap, am;
};
constexpr int kTests = 6;
__device__ __forceinline__ void add_tests(const TestVols &t, double x, double w,
                                          double (&f)[kTests]) {
    const double e0 = w * expm1(t.l0 * x), e1 = w * expm1(t.l1 * x);
    const double gp = expm1(t.ap * x), gm = t.am < 0.0 ? expm1(t.am * x) : 0.0;
    f[0] = e0 * gp;
    f[1] = e1 * gp;
    f[2] = e0 * gm;
    f[3] = e1 * gm;
    f[4] = e0 * x;
    f[5] = e1 * x;
}

// One block per accrual period m (blockIdx.x) and structure (blockIdx.y), one
// wavefront per candidate node count.  Every block forms the 64-node rule (block 0
// also writes it, with Lambda_pm and the per-period and per-slot constants), then
// its period's Gauss rule.  Latency-bound: one launch of N blocks.  The 64 Bessel
// values are summed by several lanes each and Lambda_pm by 8 lanes a step, the
// Gauss-Legendre points are tabulated, the nodes found by multisection over the
// wavefront, and the candidates above 12 nodes run only where none below passes:
// 30 to 55 us; one wavefront iterating for the 64 nodes alone took 85 to 220 us of
// every pass.
template <typename Real>
__global__ void __launch_bounds__(kRuleBlock) setup_rule_kernel(PassArgs one,
                                                                const PassArgs *__restrict__ many) {
    PassArgs pa = one;
    if (many) pa = many[blockIdx.y];
    const int N = pa.N, s = pa.s, off = pa.off, driver = pa.driver, nmax = pa.nmax;
    if (static_cast<int>(blockIdx.x) >= N) return;
    const double alpha = pa.alpha, beta = pa.beta, delta_nig = pa.delta_nig, c = pa.c;
    const double *__restrict__ tenor = pa.tenor, *__restrict__ delta = pa.delta;
    const double *__restrict__ L0 = pa.L0, *__restrict__ vol = pa.vol;
    double *__restrict__ x_out = pa.x, *__restrict__ w_out = pa.w, *__restrict__ steps = pa.steps;
    double *__restrict__ lam_pm = pa.lam_pm, *__restrict__ L0s = pa.L0s;
    double *__restrict__ deltas = pa.deltas, *__restrict__ gx = pa.gx, *__restrict__ gw = pa.gw;
    Real *__restrict__ cinv = static_cast<Real *>(pa.cinv);
    int *__restrict__ nq = pa.nq;
    constexpr int kWaves = kRuleBlock / 64;
    __shared__ double red[6][kWaves];
    __shared__ double xs[kQ], ws[kQ];
    __shared__ double ja[kGaussMax], jb[kGaussMax];
    __shared__ int ok[kNCand];
    const int t = threadIdx.x, lane = t % 64, wave = t / 64;
    const int K = N * s;
    const int m = blockIdx.x;

    // Lambda_pm over all steps, and over this period with its extreme live vols
    double lp = 0.0, lm = 0.0, mp = 0.0, mm = 0.0, vmin = 1e300, vmax = -1e300;
    int bad = 0;  // inputs the host could not check (set from device memory)
    const int sub = t % 8;
    for (int k0 = 0; k0 < K; k0 += kRuleBlock / 8) {
        const int k = k0 + t / 8;
        const int first = k / s;
        double sp = 0.0, sm = 0.0;
        if (k < K)
            for (int r = sub; r < N; r += 8) {
                if (r < first) continue;
                const double v = vol[(size_t)k * N + r];
                bad |= !isfinite(v);
                sp += fmax(v, 0.0);
                sm += fmax(-v, 0.0);
                if (first == m) {
                    vmin = fmin(vmin, v);
                    vmax = fmax(vmax, v);
                }
            }
        sp = dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(sp)));
        sm = dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(sm)));
        lp = fmax(lp, sp);
        lm = fmax(lm, sm);
        if (first == m) {
            mp = fmax(mp, sp);
            mm = fmax(mm, sm);
        }
    }
    for (int r = t; r < N; r += kRuleBlock) bad |= !(L0[r] > 0.0) || !isfinite(L0[r]);
    bad = __syncthreads_or(bad);
    double v6[6] = {lp, lm, mp, mm, -vmin, vmax};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v6[i] = fmax(v6[i], __shfl_xor(v6[i], o, 64));
        if (lane == 0) red[i][wave] = v6[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        v6[i] = red[i][0];
        for (int w = 1; w < kWaves; ++w) v6[i] = fmax(v6[i], red[i][w]);
    }
    const double Lp = v6[0], Lm = v6[1];

    if (blockIdx.x == 0) {
        if (t == 0) {
            lam_pm[0] = Lp;
            lam_pm[1] = Lm;
            // (LR1): the drift integral is finite iff Lambda_+ < alpha - beta and
            // Lambda_- < alpha + beta; the pricing pass returns NaN otherwise
            lam_pm[2] = (driver == kNig && !(Lp < alpha - beta && Lm < alpha + beta)) ? 1.0 : 0.0;
            lam_pm[3] = bad ? 1.0 : 0.0;
        }
        if (t < N) {
            const double Ta = (t == 0) ? 0.0 : tenor[t - 1];
            const double dt = (tenor[t] - Ta) / s;
            double *sc = steps + 4 * t;
            if (driver == kNig) {
                const double gamma = sqrt(alpha * alpha - beta * beta);
                const double mean = delta_nig * dt / gamma;
                sc[0] = 0.5 * sqrt(mean) / (delta_nig * dt);  // IG shape (delta dt)^2
                sc[1] = beta * mean;
                sc[2] = sqrt(mean);
                sc[3] = -delta_nig * beta / gamma * dt;       // mu_H dt
            } else {
                sc[0] = sc[1] = sc[3] = 0.0;
                sc[2] = sqrt(c * dt);
            }
        }
        if (t < nmax) {
            const int r = t - off;
            if (r >= 0) {
                cinv[t] = static_cast<Real>(1.0 / (delta[r] * L0[r]));
                L0s[t] = L0[r];
                deltas[t] = delta[r];
            } else {
                cinv[t] = Real(0);
                L0s[t] = 0.0;
                deltas[t] = 0.0;
            }
        }
    }
    if (driver != kNig) {  // the Brownian coupling is closed form: no nodes
        if (t < kQ) {
            gx[m * kQ + t] = gw[m * kQ + t] = 0.0;
            if (m == 0) x_out[t] = w_out[t] = 0.0;
        }
        for (int i = t; i < s; i += kRuleBlock) nq[m * s + i] = kQ;
        return;
    }

    // The 64-node rule; 8 lanes share each node's Bessel sum
    // K_1(z) e^z = int_0^inf e^{-z (cosh u - 1)} cosh u du (Abramowitz & Stegun
    // 9.6.24) by the trapezoidal rule, which converges geometrically for this
    // analytic integrand: step h = min(1/8, 1 / (2 sqrt z)), error below e^{-60}
    // for all z > 0, cut where z (cosh u - 1) > 50.
    const double xp = fmin(kTailExponent / (alpha - beta - Lp), kXCap);
    const double xm = fmin(kTailExponent / (alpha + beta - Lm), kXCap);
    if (t < 8 * kQ) {
        const int q = t / 8, j = q % kGL;
        const bool right = q < kGL;
        const double g = j < kGL / 2 ? -kGLx[j] : kGLx[kGL - 1 - j];
        const double wg = kGLw[j < kGL / 2 ? j : kGL - 1 - j];
        const double v = 0.5 * (g + 1.0);
        const double X = right ? xp : xm;
        const double xq = right ? X * v * v : -X * v * v;
        const double ax = fabs(xq), z = alpha * ax;
        const double h = fmin(0.125, 0.5 / sqrt(z));
        double sum = sub == 0 ? 0.5 : 0.0;  // the u = 0 term counts half
        // em = e^{u/2} - 1 and inv = e^{-u/2} along u = i h, eight points a time
        const int i0 = sub == 0 ? 8 : sub;
        double em = expm1(0.5 * i0 * h), inv = 1.0 / (1.0 + em);
        const double f = expm1(4.0 * h), finv = 1.0 / (1.0 + f);
        for (int i = i0; i < 4000; i += 8) {
            const double sh = 0.5 * fma(em, inv, em);  // sinh(u / 2)
            const double e = 2.0 * sh * sh;            // cosh u - 1
            if (!(z * e <= 50.0)) break;
            sum += exp(-z * e) * (1.0 + e);
            em = fma(em, f, em) + f;
            inv *= finv;
        }
        sum = dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(sum)));
        if (sub == 0) {
            const double pi = 3.141592653589793238462643383279502884;
            xs[q] = xq;
            ws[q] = 0.5 * wg * 2.0 * X * v *
                    (delta_nig * alpha / pi * exp(beta * xq - z) * (h * sum) / ax);
        }
    }
    __syncthreads();
    const double xq = xs[lane], wq = ws[lane];
    if (m == 0 && wave == 0) {
        x_out[lane] = xq;
        w_out[lane] = wq;
    }

    // Jacobi matrix (ja diagonal, jb squared off-diagonal) of the tilted measure
    // by the Stieltjes procedure, lane = node
    const double Mp = v6[2], Mm = v6[3];
    const double theta = 0.45 * (Mp - Mm);
    const double tilt = exp(theta * xq);
    const double nu = wq * xq * xq * tilt;
    const double mu0 = wave_sum_dpp(nu);
    double prev = 0.0, cur = sqrt(nu / mu0), b = 0.0;  // orthonormal polynomials, wavefront 0
    const TestVols tv{-v6[4], v6[5], Mp, -Mm};
    double ref[kTests];
    add_tests(tv, xq, wq, ref);
#pragma unroll
    for (int i = 0; i < kTests; ++i) ref[i] = wave_sum_dpp(ref[i]);
    int pick = kNCand;
    for (int round = 0; round < 2 && pick == kNCand; ++round) {
        __syncthreads();
        if (wave == 0)
            for (int j = round ? kGaussFirst : 0; j < (round ? kGaussMax : kGaussFirst); ++j) {
                const double a = wave_sum_dpp(cur * cur * xq);
                const double r = (xq - a) * cur - b * prev;
                const double b2 = wave_sum_dpp(r * r);
                if (lane == 0) {
                    ja[j] = a;
                    jb[j] = b2;
                }
                b = sqrt(b2);
                prev = cur;
                cur = b > 0.0 ? r / b : 0.0;
            }
        if (t < kNCand) ok[t] = 0;
        __syncthreads();
        const int cand = round * kFirstCand + wave;
        const int n = cand < kNCand ? kCand[cand] : 0;
        double x = 0.0, wt = 0.0;
        if (n) {
            // The nodes: 64 / n lanes a node, multisection on the sign changes of the
            // monic polynomials p_{j+1} = (x - a_j) p_j - b_j^2 p_{j-1} (their number
            // is the number of nodes above x), down to 2^-26 of the range
            const int per = 64 / n, node = min(lane / per, n - 1), part = lane % per;
            const double width = 1.0 / (per + 1);
            double lo = -xm, hi = xp;
            const int its = static_cast<int>(ceil(26.0 / log2(per + 1.0)));
            for (int it = 0; it < its; ++it) {
                const double step = (hi - lo) * width;
                const double at = fma(step, part + 1.0, lo);
                double p0 = 1.0, p1 = at - ja[0];
                int above = p1 < 0.0;
                for (int j = 1; j < n; ++j) {
                    const double p2 = fma(at - ja[j], p1, -jb[j - 1] * p0);
                    above += (p2 < 0.0) != (p1 < 0.0);
                    p0 = p1;
                    p1 = p2;
                }
                // points of this lane's node that lie above it
                const uint64_t vote = __ballot(lane < n * per && n - above > node);
                const int below = per - __popcll((vote >> (node * per)) & ((uint64_t(1) << per) - 1));
                lo = fma(step, static_cast<double>(below), lo);
                hi = lo + step;
            }
            // lane i < n takes node i: Newton steps, then the weight
            // mu_0 / sum_j p_j(x)^2 / |p_j|^2 back from the tilted measure; a node at
            // the origin itself (where x^2 vanishes) moves off it
            const int src = min(lane, n - 1) * per;
            lo = __shfl(lo, src, 64);
            hi = __shfl(hi, src, 64);
            x = 0.5 * (lo + hi);
            for (int it = 0; it < 3; ++it) {
                double p0 = 1.0, p1 = x - ja[0], d0 = 0.0, d1 = 1.0;
                for (int j = 1; j < n; ++j) {
                    const double p2 = fma(x - ja[j], p1, -jb[j - 1] * p0);
                    const double d2 = fma(x - ja[j], d1, fma(-jb[j - 1], d0, p1));
                    p0 = p1;
                    p1 = p2;
                    d0 = d1;
                    d1 = d2;
                }
                const double step = p1 / d1;
                if (fabs(step) <= hi - lo) x -= step;
            }
            double p0 = 0.0, p1 = 1.0, nrm = 1.0, sum = 1.0;
            for (int j = 0; j + 1 < n; ++j) {
                const double p2 = fma(x - ja[j], p1, -(j ? jb[j - 1] : 0.0) * p0);
                p0 = p1;
                p1 = p2;
                nrm *= jb[j];
                sum += p1 * p1 / nrm;
            }
            if (fabs(x) < 1e-12) x = 1e-12;
            wt = mu0 / sum / (x * x * exp(theta * x));
            double got[kTests] = {};
            if (lane < n) add_tests(tv, x, wt, got);
            bool pass = lane >= n || isfinite(wt);
            const double tol = sizeof(Real) == 4 ? kTolF32 : kTolF64;
#pragma unroll
            for (int i = 0; i < kTests; ++i)
                pass = pass && fabs(wave_sum_dpp(got[i]) - ref[i]) <= tol * fabs(ref[i]);
            pass = __all(pass);
            if (lane == 0) ok[cand] = pass;
        }
        __syncthreads();
        pick = 0;
        while (pick < kNCand && !ok[pick]) ++pick;
        if (pick == cand && lane < n) {
            gx[m * kQ + lane] = x;
            gw[m * kQ + lane] = wt;
        }
    }
    if (pick == kNCand && wave == 0) {
        gx[m * kQ + lane] = xq;
        gw[m * kQ + lane] = wq;
    }
    for (int i = t; i < s; i += kRuleBlock) nq[m * s + i] = pick < kNCand ? kCand[pick] : kQ;
}

// One block of 256 threads per Euler step k (blockIdx.x) and structure: the cumulants, the tables
// (E, W E) at the period's nodes, and the frozen drift.
template <typename Real>
__global__ void __launch_bounds__(256) setup_tables_kernel(PassArgs one,
                                                           const PassArgs *__restrict__ many) {
    PassArgs pa = one;
    if (many) pa = many[blockIdx.y];
    const int N = pa.N, s = pa.s, off = pa.off, nmax = pa.nmax, driver = pa.driver;
    if (static_cast<int>(blockIdx.x) >= N * s) return;
    const double alpha = pa.alpha, beta = pa.beta, delta_nig = pa.delta_nig, c = pa.c;
    const double *__restrict__ tenor = pa.tenor, *__restrict__ delta = pa.delta;
    const double *__restrict__ L0 = pa.L0, *__restrict__ vol = pa.vol;
    const double *__restrict__ gx = pa.gx, *__restrict__ gw = pa.gw;
    const int *__restrict__ nq_in = pa.nq;
    double *__restrict__ kappa_out = pa.kappa;
    Real *__restrict__ ew = static_cast<Real *>(pa.ew), *__restrict__ lam_t = static_cast<Real *>(pa.lam);
    Real *__restrict__ drift0 = static_cast<Real *>(pa.drift0);
    Real *__restrict__ frozen = static_cast<Real *>(pa.frozen);
    Real *__restrict__ dt_t = static_cast<Real *>(pa.dt);
    __shared__ double es[LLL_N_MAX_MP * kQ];   // E, then W E R, by [rate][node]
    __shared__ double kap[LLL_N_MAX_MP];
    const int k = blockIdx.x, t = threadIdx.x;
    const int m = k / s;
    const double Ta = (m == 0) ? 0.0 : tenor[m - 1];
    const double dt = (tenor[m] - Ta) / s;
    const double *lam = vol + (size_t)k * N;
    const bool nig = (driver == kNig);
    const int nq = nq_in[k];
    const double *x = gx + m * kQ, *w = gw + m * kQ;

    if (t < N) {  // cumulant of every live rate
        double kv = 0.0;
        if (t >= m) {
            const double u = lam[t];
            kv = nig ? nig_cumulant(u, alpha, beta, delta_nig) : 0.5 * c * u * u;
        }
        kap[t] = kv;
        kappa_out[(size_t)k * N + t] = kv;
    }
    for (int i = t; i < nmax * ((nq + 3) / 4 * 4); i += 256) {  // zero rows to a multiple of 4
        const int q = i / nmax, j = i % nmax, r = j - off;
        const double E = (r >= m && nig && q < nq) ? expm1(lam[r] * x[q]) : 0.0;
        Real *row = ew + (((size_t)k * kQ + q) * nmax + j) * 2;
        row[0] = static_cast<Real>(E);
        row[1] = static_cast<Real>(q < nq ? w[q] * E : 0.0);
        if (r >= 0) es[r * kQ + q] = E;
    }
    __syncthreads();
    // suffix recursion at the initial rates: R <- R + ell0_l E_l (1 + R) from the
    // last rate down, C_i = sum_q W E_i R_q
    if (t < nq) {
        double R = 0.0;
        for (int r = N - 1; r >= m; --r) {
            const double E = es[r * kQ + t];
            const double ell0 = delta[r] * L0[r] / (1.0 + delta[r] * L0[r]);
            es[r * kQ + t] = w[t] * E * R;
            R = R + ell0 * E * (1.0 + R);
        }
    }
    __syncthreads();
    if (t == 0) dt_t[k] = static_cast<Real>(dt);
    if (t < nmax) {
        const int j = t, r = j - off;
        double b0 = 0.0, kv = 0.0, lv = 0.0;
        if (r >= m) {
            kv = kap[r];
            lv = lam[r];
            double C = 0.0;
            if (nig) {
                for (int q = 0; q < nq; ++q) C += es[r * kQ + q];
            } else {
                double S = 0.0;
                for (int l = r + 1; l < N; ++l)
                    S += delta[l] * L0[l] / (1.0 + delta[l] * L0[l]) * lam[l];
                C = c * lv * S;
            }
            b0 = -kv - C;
        }
        lam_t[(size_t)k * nmax + j] = static_cast<Real>(lv);
        drift0[(size_t)k * nmax + j] = static_cast<Real>(-kv * dt);
        frozen[(size_t)k * nmax + j] = static_cast<Real>(b0 * dt);
    }
}

// E at the 64 nodes and the frozen drift on them, [K][N][Q] and [K][N] FP64:
// what lll_plan_tables shows and the training labels integrate on (made for those
// calls only).  One block of 64 threads (node q) per step.
__global__ void __launch_bounds__(64) full_tables_kernel(
    const double *__restrict__ delta, const double *__restrict__ L0,
    const double *__restrict__ vol, const double *__restrict__ x_in,
    const double *__restrict__ w_in, const double *__restrict__ kappa, int N, int s, int driver,
    double c, double *__restrict__ E_out, double *__restrict__ b0_out) {
    __shared__ double cq[LLL_N_MAX_MP][kQ];    // W E_q R_q contributions per rate
    const int k = blockIdx.x;
    const int q = threadIdx.x;
    const int m = k / s;
    const double *lam = vol + (size_t)k * N;
    const double xq = x_in[q], wq = w_in[q];
    const bool nig = (driver == kNig);
    double R = 0.0;
    for (int r = N - 1; r >= 0; --r) {
        double E = 0.0;
        if (r >= m && nig) {
            E = expm1(lam[r] * xq);
            cq[r][q] = wq * E * R;
            const double ell0 = delta[r] * L0[r] / (1.0 + delta[r] * L0[r]);
            R = R + ell0 * E * (1.0 + R);
        }
        E_out[((size_t)k * N + r) * kQ + q] = E;
    }
    __syncthreads();
    if (q < N) {
        double b0 = 0.0;
        if (q >= m) {
            double C = 0.0, S = 0.0;
            if (nig) {
                for (int i = 0; i < kQ; ++i) C += cq[q][i];
            } else {
                for (int l = q + 1; l < N; ++l)
                    S += delta[l] * L0[l] / (1.0 + delta[l] * L0[l]) * lam[l];
                C = c * lam[q] * S;
            }
            b0 = -kappa[(size_t)k * N + q] - C;
        }
        b0_out[(size_t)k * N + q] = b0;
    }
}

template <typename Real>
hipError_t launch_setup(const PassArgs &one, const PassArgs *many, int structures, int max_N,
                        int max_K, hipStream_t st) {
    hipLaunchKernelGGL(setup_rule_kernel<Real>, dim3(max_N, structures), dim3(kRuleBlock), 0, st,
                       one, many);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(setup_tables_kernel<Real>, dim3(max_K, structures), dim3(256), 0, st, one,
                       many);
    return hipGetLastError();
}

// First-order expansion of the coupling (paper Section 3.2, eq. (drifta)):
// K2[k][j][l] = kappa(lambda_j + lambda_l) - kappa(lambda_j) - kappa(lambda_l)
// for live slots j < l at step k, 0 elsewhere; FP64, stored in the plan
// precision.  One block per step.
template <typename Real>
__global__ void __launch_bounds__(64) setup_first_order_kernel(
    const double *__restrict__ vol, int N, int s, int off, int nmax, int driver, double alpha,
    double beta, double delta_nig, double c, Real *__restrict__ k2) {
    const int k = blockIdx.x;
    const int m = k / s;
    const double *lam = vol + (size_t)k * N;
    const bool nig = driver == LLL_DRIVER_NIG;
    for (int e = threadIdx.x; e < nmax * nmax; e += 64) {
        const int j = e / nmax, l = e % nmax;
        const int rj = j - off, rl = l - off;
        double v = 0.0;
        if (rj >= m && rl > rj) {
            const double a = lam[rj], b = lam[rl];
            v = nig ? nig_cumulant(a + b, alpha, beta, delta_nig) -
                          nig_cumulant(a, alpha, beta, delta_nig) -
                          nig_cumulant(b, alpha, beta, delta_nig)
                    : c * a * b;  // c (a + b)^2 / 2 - c a^2 / 2 - c b^2 / 2
        }
        k2[(size_t)k * nmax * nmax + e] = static_cast<Real>(v);
    }
}

template <typename Real>
hipError_t launch_first_order_t(const lll_plan &p, hipStream_t st) {
    hipLaunchKernelGGL(setup_first_order_kernel<Real>, dim3(p.K), dim3(64), 0, st, p.d.vol, p.N,
                       p.s, p.off, p.nmax, p.driver, p.alpha, p.beta, p.delta_nig, p.c,
                       static_cast<Real *>(p.d.k2));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_first_order_tables(const lll_plan &p, hipStream_t st) {
    if (!p.d.k2) return hipErrorInvalidValue;
    return p.precision == LLL_FP64 ? launch_first_order_t<double>(p, st)
                                   : launch_first_order_t<float>(p, st);
}

namespace {

// New initial forwards and a parallel shift of each rate's vol curve:
// vol[k][r] = vol_base[k][r] + shift[r] for the live rates r >= k / s.
__global__ void __launch_bounds__(256) set_inputs_kernel(const double *__restrict__ L0_in,
                                                         const double *__restrict__ shift,
                                                         const double *__restrict__ vol_base,
                                                         double *__restrict__ L0,
                                                         double *__restrict__ vol, int N, int s) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (L0_in && i < N) L0[i] = L0_in[i];
    if (shift && i < N * s * N) {
        const int k = i / N, r = i % N;
        vol[i] = vol_base[i] + (r >= k / s ? shift[r] : 0.0);
    }
}

}  // namespace

hipError_t launch_set_inputs(const lll_plan &p, const double *L0_dev, const double *shift_dev,
                             hipStream_t st) {
    const int n = shift_dev ? p.K * p.N : p.N;
    hipLaunchKernelGGL(set_inputs_kernel, dim3((n + 255) / 256), dim3(256), 0, st, L0_dev,
                       shift_dev, p.d.vol_base, p.d.L0, p.d.vol, p.N, p.s);
    return hipGetLastError();
}

hipError_t launch_precompute(const lll_plan &p, hipStream_t st) {
    const PassArgs a = pass_args(p);
    return p.precision == LLL_FP64 ? launch_setup<double>(a, nullptr, 1, p.N, p.K, st)
                                   : launch_setup<float>(a, nullptr, 1, p.N, p.K, st);
}

hipError_t launch_full_tables(const lll_plan &p, double *E, hipStream_t st) {
    const DeviceTables &d = p.d;
    hipLaunchKernelGGL(full_tables_kernel, dim3(p.K), dim3(64), 0, st, d.delta, d.L0, d.vol, d.x,
                       d.w, d.kappa, p.N, p.s, p.driver, p.c, E, d.b0);
    return hipGetLastError();
}

hipError_t launch_precompute_batch(const PassArgs *many, int structures, int max_N, int max_K,
                                   hipStream_t st) {
    return launch_setup<float>(PassArgs{}, many, structures, max_N, max_K, st);
}

}  // namespace lll
