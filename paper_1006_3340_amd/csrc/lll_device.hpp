// lll_device.hpp -- device-side building blocks shared by the kernels:
// the counter-based generator, the driver increment and the NIG cumulant.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lll {

constexpr int kQ = 64;          // quadrature nodes of the coupling integral
constexpr int kGL = 32;         // Gauss-Legendre points per half line
constexpr int kWave = 64;       // CDNA wavefront
constexpr int kBlock = 256;     // threads per path block (4 wavefronts)
constexpr double kTailExponent = 36.0;  // truncate the Lévy integral where e^{-36}
constexpr double kXCap = 40.0;          // ... but never beyond |x| = 40

enum { kFull = 0, kPicard = 1, kFrozen = 2, kFirst = 3, kSecond = 4 };
enum { kNig = 0, kBrownian = 1 };

// Philox-4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11): ten rounds of two
// 32x32->64 multiplications with the Weyl key schedule.
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32x32->64 product each (v_mad_u64_u32) rather than separate
        // low and high halves
        const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c.x;
        const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c.z;
        const uint32_t lo0 = static_cast<uint32_t>(p0), hi0 = static_cast<uint32_t>(p0 >> 32);
        const uint32_t lo1 = static_cast<uint32_t>(p1), hi1 = static_cast<uint32_t>(p1 >> 32);
        // three-input XORs as one v_bitop3_b32 each (truth table 0x96)
        c = make_uint4(__builtin_amdgcn_bitop3_b32(hi1, c.y, k0, 0x96), lo1,
                       __builtin_amdgcn_bitop3_b32(hi0, c.w, k1, 0x96), lo0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// 24-bit uniform on (0, 1), exact in FP64: (k + 1/2) 2^-24 = k 2^-24 + 2^-25
// for the top 24 bits k of the word, one FMA with no rounding.
__device__ __forceinline__ double uniform24(uint32_t w) {
    return fma(static_cast<double>(w >> 8), 1.0 / 16777216.0, 1.0 / 33554432.0);
}

// FP64 arithmetic of the increment on its own argument ranges (all operands
// positive and normal), each a textbook construction with at most 2 ulp of
// error against the correctly rounded result -- a third of the instructions
// of the general-purpose library routines, whose double-double steps and
// special-value paths the sampler does not need.  The hardware reciprocal and
// reciprocal square root are good to 2^-24 (measured over 2^22 arguments), so one
// Newton step (2^-48) and one residual correction reach the last bit.

// A polynomial coefficient as a scalar-register operand: left to itself the
// compiler copies each FP64 constant into a vector register pair in front of its
// FMA (55 vector instructions of the increment).
__device__ __forceinline__ double scalar_const(double c) {
#if defined(__HIP_DEVICE_COMPILE__)
    __asm__ volatile("" : "+s"(c));
#endif
    return c;
}

template <int N>
__device__ __forceinline__ double horner(double x, const double (&c)[N]) {
    double s = scalar_const(c[N - 1]);
#pragma unroll
    for (int i = N - 2; i >= 0; --i) s = fma(s, x, scalar_const(c[i]));
    return s;
}

// a / b for b > 0 normal: Newton step r <- r + r (1 - b r), then the residual
// correction q <- q + r (a - b q) (each residual exact by FMA).
__device__ __forceinline__ double div_pos(double a, double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(fma(-b, r, 1.0), r, r);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}

// sqrt(x) for x > 0 normal: from the hardware 1/sqrt estimate y, g = x y and
// h = y / 2 refined by one coupled Newton (Goldschmidt) step, then
// g <- g + h (x - g^2).
__device__ __forceinline__ double sqrt_pos(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, x), h, g);
}

// log(x) for 0 < x <= 1 normal: x = f 2^e with f in [1/sqrt 2, sqrt 2),
// log f = 2 atanh(z) = 2 z + 2 z w p(w), z = (f - 1) / (f + 1), w = z^2, |z| <=
// 0.172, p the minimax polynomial of (atanh(z) / z - 1) / w (Remez exchange in
// 50-digit arithmetic, error 1.6e-16, i.e. 5e-18 of log f), and e log 2 with
// log 2 split into 32 leading bits (e times it is exact) and the FP64 rest.
__device__ __forceinline__ double log_unit(double x) {
    constexpr double kLn2Hi = 0x1.62e42ffp-1;             // log 2 to 32 bits
    constexpr double kLn2Lo = -4.2009150726810846e-11;    // log 2 - kLn2Hi
    constexpr double kP[] = {0.3333333333333334865, 0.1999999999994922219, 0.1428571431319969345,
                             0.1111110553641115111, 0.09091446609892922211, 0.07665798466224352336,
                             0.07308936476253457391};
    double f = __builtin_amdgcn_frexp_mant(x);             // [1/2, 1)
    int e = __builtin_amdgcn_frexp_exp(x);
    if (f < 0.7071067811865476) {
        f *= 2.0;
        --e;
    }
    const double z = div_pos(f - 1.0, f + 1.0);
    const double w = z * z;
    const double tz = 2.0 * z;
    const double lf = fma(tz * w, horner(w, kP), tz);
    const double de = static_cast<double>(e);
    return fma(de, scalar_const(kLn2Hi), fma(de, scalar_const(kLn2Lo), lf));
}

// sin(pi/2 v) and cos(pi/2 v) for v = q + 2 r, integer q, |r| <= 1/4 (exact):
// sin(pi r) / r and cos(pi r) by minimax polynomials in r^2 (Remez exchange in
// 50-digit arithmetic; errors 1e-17 and 3e-20), then the quadrant q mod 4.
__device__ __forceinline__ void sincos_quadrant(int q, double r, double &sn, double &cs) {
    constexpr double kS[] = {3.141592653589793229, -5.167712780049954539, 2.550164039873378514,
                             -0.5992645289398096045, 0.08214586918508168636,
                             -0.007370021659139428769, 0.0004615322405479640474};
    constexpr double kC[] = {1.0, -4.934802200544679247, 4.058712126416747358,
                             -1.335262768851918561, 0.2353306301909417545, -0.0258068856542158721,
                             0.001929465758794343034, -0.0001035675398146088982};
    const double x = r * r;
    const double s = r * horner(x, kS);
    const double c = horner(x, kC);
    const int qi = q & 3;
    const bool odd = (qi & 1) != 0;
    sn = odd ? c : s;
    cs = odd ? s : c;
    if (qi & 2) sn = -sn;
    if (qi == 1 || qi == 2) cs = -cs;
}

// sin(pi t) and cos(pi t) for 0 <= t <= 2 with t a multiple of 2^-24: v = 2 t,
// q = rint(v) and r = (v - q) / 2 (both steps exact).
__device__ __forceinline__ void sincospi_unit(double t, double &sn, double &cs) {
    const double v = 2.0 * t;
    const double q = __builtin_rint(v);
    sincos_quadrant(static_cast<int>(q), (v - q) * 0.5, sn, cs);
}

// The same for the angle 2 pi u, u = uniform24(word): with k the top 24 bits,
// 4 u = (k + 1/2) 2^-22, so q and r come from integer arithmetic.
__device__ __forceinline__ void sincos_uniform(uint32_t word, double &sn, double &cs) {
    const uint32_t k = (word >> 8) + (1u << 21);
    const int j = static_cast<int>(k & ((1u << 22) - 1)) - (1 << 21);
    sincos_quadrant(static_cast<int>(k >> 22),
                    fma(static_cast<double>(j), 1.0 / 8388608.0, 1.0 / 16777216.0), sn, cs);
}

// Per-period constants of the increment, from the IG mean m = delta dt / gamma
// and shape lam = (delta dt)^2: sqrt(m / lam) / 2, beta m, sqrt(m) and the drift
// mu_H dt; the Brownian driver has only the scale sqrt(c dt), in place of sqrt(m).
struct StepConsts {
    double a, bm, sm, mu_dt;
};

// Driver increment of one Euler step from four Philox words (FP64).
// NIG(alpha, beta, delta dt, mu_H dt) as a normal variance-mean mixture over an
// inverse-Gaussian subordinator: Box-Muller normals (z1, z2) and the IG draw by
// Michael-Schucany-Haas.  With y = z1^2 its smaller root, written without
// cancellation, is x = 4 m^2 lam y / (m y + sqrt(m^2 y^2 + 4 m lam y))^2; in
// h = |z1| sqrt(m / lam) / 2 and g = h + sqrt(h^2 + 1) it is m / g^2, the other
// root m g^2, and the acceptance u2 <= m / (m + x) reads u2 (g^2 + 1) <= g^2.  So
// one square root and one reciprocal give V = m rho^2 and sqrt(V) = sqrt(m) rho with
// rho = 1/g or g, and dH = mu_H dt + beta V + sqrt(V) z2.  Brownian: sqrt(c dt) z1.
// 120 vector instructions instead of 220 (with Philox 165 instead of 270 a step): the
// scheme that does little else, FROZEN, takes 2.5 ms instead of 3.3 (N = 20, 2^20 paths,
// 400 steps).
__device__ __forceinline__ double increment(uint4 w, const StepConsts& sc, bool brownian,
                                            double* V_out) {
    const double r = sqrt_pos(-2.0 * log_unit(uniform24(w.x)));
    double sn, cs;
    sincos_uniform(w.y, sn, cs);
    const double z1 = r * cs;
    if (brownian) {
        if (V_out) *V_out = 0.0;
        return sc.sm * z1;
    }
    const double z2 = r * sn;
    const double h = sc.a * fabs(z1);
    const double g = h + sqrt_pos(fma(h, h, 1.0));
    const double g2 = g * g;
    const bool small = uniform24(w.z) * (g2 + 1.0) <= g2;
    double inv = __builtin_amdgcn_rcp(g);
    inv = fma(fma(-g, inv, 1.0), inv, inv);
    inv = fma(fma(-g, inv, 1.0), inv, inv);
    const double rho = small ? inv : g;
    if (V_out) *V_out = (sc.sm * rho) * (sc.sm * rho);
    return fma(rho, fma(sc.bm, rho, sc.sm * z2), sc.mu_dt);
}

// NIG cumulant kappa(u) = mu_H u + delta (gamma - sqrt(alpha^2 - (beta+u)^2)),
// mu_H = -delta beta / gamma, rearranged so that no two large terms cancel:
// kappa(u) = delta u^2 (gamma + beta (2 beta + u) / (gamma + s)) / (gamma (gamma + s)),
// s = sqrt(alpha^2 - (beta + u)^2).
__device__ __forceinline__ double nig_cumulant(double u, double alpha, double beta, double delta) {
    const double gamma = sqrt(alpha * alpha - beta * beta);
    const double bu = beta + u;
    const double s = sqrt(alpha * alpha - bu * bu);
    const double gs = gamma + s;
    return delta * u * u * (gamma + beta * (2.0 * beta + u) / gs) / (gamma * gs);
}

}  // namespace lll
