// mlp_train.hip -- data generation, BF16-MFMA forward/backward and Adam for
// the drift surrogate (layout and target in mlp.hpp).
//
// Training data: FULL paths (their own random stream, Philox tag 1) record
// their state at a staggered set of steps; for every recorded state and live
// rate i an FP64 kernel forms the features and the label
//     (C_i - C'_i), C_i = sum_q W_q E_{i,q} (prod_{l>i}(1 + ell_l E_{l,q}) - 1)
// (the quadrature coupling of eq. (LIBOR-drift-PT)) and C'_i its first-order
// expansion (eq. (drifta)).  Training: minibatches drawn with replacement by
// Philox (tag 2); one block of eight wavefronts per 64 samples draws its rows, runs
// the three hidden layers forward and backward on v_mfma_f32_16x16x32_bf16 and
// writes its gradient; a second kernel sums the block gradients in a fixed order and
// applies Adam to the FP32 master weights, refreshing their BF16 copies.
#include <hip/hip_runtime.h>

#include <utility>

#include "lll_device.hpp"
#include "lll_internal.hpp"
#include "mlp.hpp"
#define LLL_BUCKET_TU
#include "path_kernel.hpp"

namespace lll {
namespace mlp {
namespace {

using detail::cptr;
using detail::PathArgs;

constexpr int kTile = 64;         // samples per block
constexpr int kTrainBlock = 512;  // eight wavefronts

// ---------------------------------------------------------------- data ----

// FULL paths recording their state (all NMAX slots; fixed rates 0) at steps
// k_r = r * (K / R) + (p mod (K / R)), r = 0..R-1.
template <int NMAX>
__global__ void __launch_bounds__(kBlock) record_kernel(PathArgs<float> a, int R,
                                                        float *__restrict__ states,
                                                        int *__restrict__ kidx) {
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const int64_t wave_first = gid - (threadIdx.x % kWave);
    if (wave_first >= a.n_paths) return;
    const bool active = gid < a.n_paths;
    const int64_t p = a.path_offset + gid;
    const uint32_t p_lo = static_cast<uint32_t>(p);
    const uint32_t p_hi = static_cast<uint32_t>(static_cast<uint64_t>(p) >> 32);
    const int K = a.N * a.s;
    const int stride = K / R;
    const int phase = static_cast<int>(gid % stride);
    float X[NMAX], X1[NMAX];
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
        X[j] = 0.0f;
        X1[j] = 0.0f;
    }
    int r = 0;
    for (int k = 0; k < K; ++k) {
        const int m = k / a.s;
        const int j0 = a.off + m;
        if (r < R && k == r * stride + phase) {   // divergent: per-lane phase
            if (active) {
                float *dst = states + (gid * R + r) * NMAX;
#pragma unroll
                for (int j = 0; j < NMAX; ++j) dst[j] = (j >= j0) ? X[j] : 0.0f;
                kidx[gid * R + r] = k;
            }
            ++r;
        }
        const cptr<double> sc = a.steps + 4 * m;
        const StepConsts cst{sc[0], sc[1], sc[2], sc[3]};
        const uint4 w = philox4x32_10(
            make_uint4(static_cast<uint32_t>(k), p_lo, p_hi, a.stream_word), a.key0, a.key1);
        const float dH = static_cast<float>(increment(w, cst, false, nullptr));
        detail::dispatch_step<float, NMAX, kFull>(std::make_integer_sequence<int, NMAX>{}, j0, a,
                                                  k, dH, X, X1);
    }
}

// FP64 labels and BF16 features of every live rate of one recorded state.
__global__ void __launch_bounds__(64) label_kernel(
    const float *__restrict__ states, const int *__restrict__ kidx, const int64_t *__restrict__ poff,
    int64_t n_states, int nmax, int off, int N, int s, const double *__restrict__ tenor,
    const double *__restrict__ delta, const double *__restrict__ L0, const double *__restrict__ vol,
    const double *__restrict__ E, const double *__restrict__ w, double alpha, double beta,
    double delta_nig, __bf16 *__restrict__ feat, float *__restrict__ label) {
    const int64_t st = static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x;
    if (st >= n_states) return;
    const int k = kidx[st];
    const int first = k / s;
    const float *X = states + st * nmax;
    const double *lam = vol + (size_t)k * N;
    const double t = (first == 0 ? 0.0 : tenor[first - 1]) +
                     (k - first * s) * (tenor[first] - (first == 0 ? 0.0 : tenor[first - 1])) / s;
    const double tn = t / tenor[N - 1];
    double ell[kRates], C[kRates];
    for (int r = first; r < N; ++r) {
        const double L = L0[r] * exp(static_cast<double>(X[r + off]));
        ell[r] = delta[r] * L / (1.0 + delta[r] * L);
        C[r] = 0.0;
    }
    for (int q = 0; q < kQ; ++q) {
        double R = 0.0;
        for (int r = N - 1; r >= first; --r) {
            const double e = E[((size_t)k * N + r) * kQ + q];
            C[r] += w[q] * e * R;
            R += ell[r] * e * (1.0 + R);
        }
    }
    int64_t pi = poff[st];
    for (int i = first; i < N; ++i, ++pi) {
        double c1 = 0.0;
        const double ki = nig_cumulant(lam[i], alpha, beta, delta_nig);
        for (int l = i + 1; l < N; ++l)
            c1 += ell[l] * (nig_cumulant(lam[i] + lam[l], alpha, beta, delta_nig) - ki -
                            nig_cumulant(lam[l], alpha, beta, delta_nig));
        label[pi] = static_cast<float>(C[i] - c1);
        __bf16 *f = feat + pi * kIn;
        for (int c = 0; c < kIn; ++c) f[c] = static_cast<__bf16>(0.0f);
        f[0] = static_cast<__bf16>(static_cast<float>(tn));
        for (int l = i + 1; l < N; ++l) f[1 + l] = static_cast<__bf16>(X[l + off]);
        f[1 + kRates + i] = static_cast<__bf16>(1.0f);
    }
}

// Per-slot range of the state over the data (the surrogate's trust box) and
// the root mean square of the labels; one block, fixed reduction order.
__global__ void __launch_bounds__(256) stats_kernel(const float *__restrict__ states,
                                                    const int *__restrict__ kidx, int64_t n_states,
                                                    int nmax, int off, int s,
                                                    const float *__restrict__ label,
                                                    int64_t n_pairs, float *__restrict__ out) {
    __shared__ float lo[256], hi[256];
    __shared__ double ss[256];
    const int t = threadIdx.x;
    for (int r = 0; r < kRates; ++r) {
        const int j = r + off;
        float l = 3.0e38f, h = -3.0e38f;
        if (j < nmax)
            for (int64_t st = t; st < n_states; st += 256) {
                if (kidx[st] / s > r) continue;  // rate already fixed in this state
                const float v = states[st * nmax + j];
                l = fminf(l, v);
                h = fmaxf(h, v);
            }
        lo[t] = l;
        hi[t] = h;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if (t < o) {
                lo[t] = fminf(lo[t], lo[t + o]);
                hi[t] = fmaxf(hi[t], hi[t + o]);
            }
            __syncthreads();
        }
        if (t == 0) {
            out[r] = lo[0];
            out[kRates + r] = hi[0];
        }
        __syncthreads();
    }
    double acc = 0.0;
    for (int64_t p = t; p < n_pairs; p += 256) acc += static_cast<double>(label[p]) * label[p];
    ss[t] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (t < o) ss[t] += ss[t + o];
        __syncthreads();
    }
    if (t == 0) out[2 * kRates] = static_cast<float>(sqrt(ss[0] / static_cast<double>(n_pairs)));
}

// ------------------------------------------------------------ training ----

__global__ void __launch_bounds__(256) init_kernel(float *__restrict__ wts, __bf16 *__restrict__ wbf,
                                                   float *__restrict__ adam, uint32_t key0,
                                                   uint32_t key1) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= kParams) return;
    float a = 0.0f;
    if (p < kOffB1) a = sqrtf(6.0f / (kIn + kHid));
    else if (p >= kOffW2 && p < kOffB2) a = sqrtf(6.0f / (2 * kHid));
    else if (p >= kOffW3 && p < kOffB3) a = sqrtf(6.0f / (2 * kHid));
    else if (p >= kOffW4 && p < kOffB4) a = sqrtf(6.0f / (kHid + 1));
    const uint4 r = philox4x32_10(make_uint4(static_cast<uint32_t>(p), 0u, 0u, 2u << 24), key0, key1);
    const float u = static_cast<float>(uniform24(r.x));
    const float v = a * (2.0f * u - 1.0f);
    wts[p] = v;
    wbf[p] = static_cast<__bf16>(v);
    adam[p] = 0.0f;
    adam[kParams + p] = 0.0f;
}

struct TileArgs {
    const __bf16 *feat;   // [P][96]
    const float *target;  // [P] raw labels (scaled by inv_sigma here)
    int B;
    uint64_t n_pairs;     // rows drawn with replacement among these, or 0: rows 0..B-1
    uint64_t n_inv;       // floor((2^64 - 1) / n_pairs)
    uint32_t step, key0, key1;
    float inv_sigma;
    float inv_B;
    const __bf16 *wbf;    // BF16 copy of the parameter vector
    const float *wf;      // FP32 parameter vector
    float *gpart;         // [tiles][kGradRow] or null (forward only)
    float *lpart;         // [tiles] loss partials or null
    float *yout;          // [B] outputs (normalised units) or null
};

// Row of the batch's sample r: x mod n_pairs for 64 Philox bits x, the quotient from
// one high product (n_inv x >> 64 is at most 2 below it).
__device__ __forceinline__ int64_t sample_row(const TileArgs &t, int64_t r) {
    if (t.n_pairs == 0) return r;
    const uint4 w = philox4x32_10(make_uint4(t.step, static_cast<uint32_t>(r), 1u, 2u << 24),
                                  t.key0, t.key1);
    const uint64_t x = (static_cast<uint64_t>(w.x) << 32) | w.y;
    uint64_t m = x - __umul64hi(x, t.n_inv) * t.n_pairs;
    if (m >= t.n_pairs) m -= t.n_pairs;
    if (m >= t.n_pairs) m -= t.n_pairs;
    return static_cast<int64_t>(m);
}

// LDS rows: 8 elements of padding behind 64 or 96 BF16 (4 behind 64 floats) keep 16-byte
// alignment and spread 16 consecutive rows over the banks.
constexpr int kLd = kHid + 8, kLdX = kIn + 8, kLdF = kHid + 4;

// Every matrix is kept in the order in which the product that takes it reads 8
// contraction indices at once (16 bytes a lane): the activations and dZ by sample (for
// the next layer and for dH) and by unit (for dW), W2 and W3 transposed for dH.
struct TileLds {
    union {
        struct {
            __bf16 X[kTile * kLdX];         // [m][i]
            __bf16 H[2][kTile * kLd];       // [m][o], layers 1 and 2
        } fwd;
        float dZ[3][kTile * kLdF];          // [m][o], layers 1..3 (after the forward pass)
    };
    __bf16 XT[kIn * kLd];                   // [i][m]
    __bf16 HT[2][kHid * kLd];               // [o][m]
    __bf16 H3[kTile * kLd];                 // [m][o]
    __bf16 WT[2][kHid * kLd];               // [i][o], layers 2 and 3
    __bf16 dZb[2][kTile * kLd];             // [m][o], layers 2 and 3
    __bf16 dZT[2][kHid * kLd];              // [o][m], layer l in slot l % 2
    float dy[kTile], loss[kTile];
};

// 16 bytes of BF16 data with the alignment of the caller's features.
struct __attribute__((packed, aligned(2))) Chunk {
    uint32_t d[4];
};
__device__ __forceinline__ bf16x8 load_chunk(const __bf16 *p) {
    const Chunk c = *reinterpret_cast<const Chunk *>(p);
    return __builtin_bit_cast(bf16x8, c.d);
}
__device__ __forceinline__ bf16x8 frag(const __bf16 *p) {
    return *reinterpret_cast<const bf16x8 *>(p);
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Wave w holds units 16 (w % 4) + 4 (lane / 16) + e of samples 32 (w / 4) + 16 j +
// lane % 16, j = 0, 1, of every layer's Z, H, dH and dZ: what the matrix instruction
// returns for Z^T = W H^T and dH^T = W^T dZ^T alike, so that Z stays in registers.
struct Lane {
    int ob, nb, lr, lk;  // 16 (w % 4), 32 (w / 4), lane % 16, lane / 16
    __device__ int unit() const { return ob + 4 * lk; }
    __device__ int sample(int j) const { return nb + 16 * j + lr; }
};

// Z^T = W . H^T + b for the wave's units and samples, W's rows in registers.
template <int KT, int LD>
__device__ __forceinline__ void layer_fwd(const Lane &l, const bf16x8 (&W)[KT], const __bf16 *Hin,
                                          const floatx4 &bias, floatx4 (&Z)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        floatx4 acc{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
            acc = mfma16(W[kt], frag(Hin + l.sample(j) * LD + 32 * kt + 8 * l.lk), acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) Z[j][e] = acc[e] + bias[e];
    }
}

// One wave's tile to its [m][o] and / or [o][m] copy.
__device__ __forceinline__ void put(const Lane &l, int j, const floatx4 &v, __bf16 *rows,
                                    __bf16 *cols) {
    bf16x4 b;
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = static_cast<__bf16>(v[e]);
    if (rows) *reinterpret_cast<bf16x4 *>(rows + l.sample(j) * kLd + l.unit()) = b;
    if (cols)
#pragma unroll
        for (int e = 0; e < 4; ++e) cols[(l.unit() + e) * kLd + l.sample(j)] = b[e];
}

// dW[o][i] = sum_m dZ[m][o] Hin[m][i] for the block: the wave's 16 rows o and half of
// the NT column tiles of 16, written to the block's gradient slice.
template <int NT, int STRIDE>
__device__ __forceinline__ void weight_grad(const Lane &l, const __bf16 *dZT, const __bf16 *HT,
                                            float *g) {
    const int first = l.nb / 32 * (NT / 2);
#pragma unroll
    for (int j = 0; j < NT / 2; ++j) {
        floatx4 acc{0.0f, 0.0f, 0.0f, 0.0f};
        const int i = 16 * (first + j) + l.lr;
#pragma unroll
        for (int kt = 0; kt < kTile / 32; ++kt)
            acc = mfma16(frag(dZT + (l.ob + l.lr) * kLd + 32 * kt + 8 * l.lk),
                         frag(HT + i * kLd + 32 * kt + 8 * l.lk), acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) g[(l.unit() + e) * STRIDE + i] = acc[e];
    }
}

// dZ of the layer below: (dH^T = W^T dZ^T) gelu'(Z).
__device__ __forceinline__ void input_grad(const Lane &l, const __bf16 *WT, const __bf16 *dZb,
                                           const floatx4 (&Z)[2], floatx4 (&dZ)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        floatx4 acc{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kt = 0; kt < kHid / 32; ++kt)
            acc = mfma16(frag(WT + (l.ob + l.lr) * kLd + 32 * kt + 8 * l.lk),
                         frag(dZb + l.sample(j) * kLd + 32 * kt + 8 * l.lk), acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) dZ[j][e] = acc[e] * gelu_grad(Z[j][e]);
    }
}

// Column sums over the block's samples, in sample order: one lane a unit.
__device__ __forceinline__ float column_sum(const float *dZ, int o) {
    float s = 0.0f;
#pragma unroll 16
    for (int m = 0; m < kTile; ++m) s += dZ[m * kLdF + o];
    return s;
}

// A batch of 16384 is 256 blocks, one a compute unit: what bounds the kernel is the time
// of one block, a chain of gathers, products and barriers.  So the rows are drawn here,
// all loads are 16 bytes a lane and issued at once, W1..W3 go to registers as
// fragments, eight wavefronts share the elementwise work, and the bias sums wait for
// the end, one wavefront each.  At a batch of 16384: 16 us; with 2-byte loads, unpadded
// rows read across, Z in LDS and four wavefronts 38 us and 4.6 us for the rows' own launch.
__global__ void __launch_bounds__(kTrainBlock) tile_kernel(TileArgs t) {
    __shared__ TileLds S;
    const int lane = threadIdx.x % 64, w = threadIdx.x / 64;
    const Lane l{16 * (w % 4), 32 * (w / 4), lane % 16, lane / 16};
    const __bf16 *wbf = t.wbf;
    const float *wf = t.wf;
    bf16x8 W1[kIn / 32], W2[kHid / 32], W3[kHid / 32], wt[2];
#pragma unroll
    for (int kt = 0; kt < kIn / 32; ++kt)
        W1[kt] = load_chunk(wbf + kOffW1 + (l.ob + l.lr) * kIn + 32 * kt + 8 * l.lk);
#pragma unroll
    for (int kt = 0; kt < kHid / 32; ++kt) {
        W2[kt] = load_chunk(wbf + kOffW2 + (l.ob + l.lr) * kHid + 32 * kt + 8 * l.lk);
        W3[kt] = load_chunk(wbf + kOffW3 + (l.ob + l.lr) * kHid + 32 * kt + 8 * l.lk);
    }
    wt[0] = load_chunk(wbf + kOffW2 + lane * kHid + 8 * w);
    wt[1] = load_chunk(wbf + kOffW3 + lane * kHid + 8 * w);
    floatx4 b1, b2, b3, w4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        b1[e] = wf[kOffB1 + l.unit() + e];
        b2[e] = wf[kOffB2 + l.unit() + e];
        b3[e] = wf[kOffB3 + l.unit() + e];
        w4[e] = wf[kOffW4 + l.unit() + e];
    }
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kTile + lane;
    const bool valid = r < t.B;
    float target = 0.0f;
    bf16x8 x[2] = {};
    if (valid) {
        const int64_t smp = sample_row(t, r);
        const __bf16 *row = t.feat + smp * kIn;
        x[0] = load_chunk(row + 8 * w);
        if (w < kIn / 8 - 8) x[1] = load_chunk(row + 64 + 8 * w);
        if (w == 0) target = t.target[smp] * t.inv_sigma;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        if (c == 1 && w >= kIn / 8 - 8) break;
        const int i = 64 * c + 8 * w;
        *reinterpret_cast<bf16x8 *>(S.fwd.X + lane * kLdX + i) = x[c];
#pragma unroll
        for (int e = 0; e < 8; ++e) S.XT[(i + e) * kLd + lane] = x[c][e];
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) S.WT[c][(8 * w + e) * kLd + lane] = wt[c][e];
    __syncthreads();
    floatx4 Z1[2], Z2[2], Z3[2], v;
    auto activate = [&](const floatx4 &z) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu(z[e]);
    };
    layer_fwd<kIn / 32, kLdX>(l, W1, S.fwd.X, b1, Z1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        activate(Z1[j]);
        put(l, j, v, S.fwd.H[0], S.HT[0]);
    }
    __syncthreads();
    layer_fwd<kHid / 32, kLd>(l, W2, S.fwd.H[0], b2, Z2);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        activate(Z2[j]);
        put(l, j, v, S.fwd.H[1], S.HT[1]);
    }
    __syncthreads();
    layer_fwd<kHid / 32, kLd>(l, W3, S.fwd.H[1], b3, Z3);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        activate(Z3[j]);
        put(l, j, v, S.H3, nullptr);
    }
    __syncthreads();
    if (w == 0) {
        float y = wf[kOffB4];
#pragma unroll
        for (int c = 0; c < kHid / 8; ++c) {
            const bf16x8 h = frag(S.H3 + lane * kLd + 8 * c);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                y = fmaf(wf[kOffW4 + 8 * c + e], static_cast<float>(h[e]), y);
        }
        if (valid && t.yout) t.yout[r] = y;
        const float d = valid ? (y - target) : 0.0f;
        S.dy[lane] = d * t.inv_B;
        S.loss[lane] = 0.5f * d * d * t.inv_B;
    }
    __syncthreads();
    if (t.lpart && w == 7 && lane == 0) {
        float s = 0.0f;
        for (int m = 0; m < kTile; ++m) s += S.loss[m];
        t.lpart[blockIdx.x] = s;
    }
    if (!t.gpart) return;
    float *g = t.gpart + static_cast<int64_t>(blockIdx.x) * kGradRow;
    floatx4 dZ[2];
    auto put_f32 = [&](float *out) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            *reinterpret_cast<floatx4 *>(out + l.sample(j) * kLdF + l.unit()) = dZ[j];
    };
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float dy = S.dy[l.sample(j)];
#pragma unroll
        for (int e = 0; e < 4; ++e) dZ[j][e] = dy * w4[e] * gelu_grad(Z3[j][e]);
        put(l, j, dZ[j], S.dZb[1], S.dZT[1]);
    }
    put_f32(S.dZ[2]);
    __syncthreads();
    input_grad(l, S.WT[1], S.dZb[1], Z2, dZ);
#pragma unroll
    for (int j = 0; j < 2; ++j) put(l, j, dZ[j], S.dZb[0], S.dZT[0]);
    put_f32(S.dZ[1]);
    weight_grad<kHid / 16, kHid>(l, S.dZT[1], S.HT[1], g + kOffW3);
    __syncthreads();
    input_grad(l, S.WT[0], S.dZb[0], Z1, dZ);
#pragma unroll
    for (int j = 0; j < 2; ++j) put(l, j, dZ[j], nullptr, S.dZT[1]);
    put_f32(S.dZ[0]);
    weight_grad<kHid / 16, kHid>(l, S.dZT[0], S.HT[0], g + kOffW2);
    __syncthreads();
    weight_grad<kIn / 16, kIn>(l, S.dZT[1], S.XT, g + kOffW1);
    if (w == 0) {
        g[kOffB1 + lane] = column_sum(S.dZ[0], lane);
    } else if (w == 1) {
        g[kOffB2 + lane] = column_sum(S.dZ[1], lane);
    } else if (w == 2) {
        g[kOffB3 + lane] = column_sum(S.dZ[2], lane);
    } else if (w == 3) {
        float s = 0.0f;
#pragma unroll 16
        for (int m = 0; m < kTile; ++m)
            s = fmaf(S.dy[m], static_cast<float>(S.H3[m * kLd + lane]), s);
        g[kOffW4 + lane] = s;
    } else if (w == 4 && lane == 0) {
        float s = 0.0f;
        for (int m = 0; m < kTile; ++m) s += S.dy[m];
        g[kOffB4] = s;
    }
}

// Sum of the tile gradients and, with lr > 0, an Adam step of the FP32 master
// weights (and a refresh of the BF16 copy).  A block takes 32 parameters; each
// parameter's tiles are split into 8 contiguous slices summed by 8 threads at
// once (coalesced rows of 32 parameters), then the slices in slice order: a
// fixed summation order, the same in every call.  Block 0 sums the tile losses
// the same way.  256 tiles are 15 MB: 4.5 us with 16 loads of a slice in flight on whole
// cache lines, 13.7 us with rows of an odd number of floats and few in flight.
constexpr int kSlices = 8;
constexpr int kParamsPerBlock = 256 / kSlices;

__global__ void __launch_bounds__(256) reduce_adam_kernel(const float *__restrict__ gpart,
                                                          int tiles, const float *__restrict__ lpart,
                                                          float *__restrict__ loss_out,
                                                          float *__restrict__ wts,
                                                          __bf16 *__restrict__ wbf,
                                                          float *__restrict__ adam,
                                                          float *__restrict__ grad_out, float lr,
                                                          float bc1, float bc2) {
    __shared__ float part[kSlices][kParamsPerBlock];
    __shared__ float lsum[kSlices];
    const int pl = threadIdx.x % kParamsPerBlock, sl = threadIdx.x / kParamsPerBlock;
    const int p = blockIdx.x * kParamsPerBlock + pl;
    const int per = (tiles + kSlices - 1) / kSlices;
    const int t0 = sl * per, t1 = min(tiles, t0 + per);
    float s = 0.0f;
    if (p < kParams)
#pragma unroll 16
        for (int i = t0; i < t1; ++i) s += gpart[static_cast<int64_t>(i) * kGradRow + p];
    part[sl][pl] = s;
    if (blockIdx.x == 0 && loss_out && pl == 0) {
        float l = 0.0f;
#pragma unroll 16
        for (int i = t0; i < t1; ++i) l += lpart[i];
        lsum[sl] = l;
    }
    __syncthreads();
    if (blockIdx.x == 0 && loss_out && threadIdx.x == 0) {
        float l = lsum[0];
        for (int k = 1; k < kSlices; ++k) l += lsum[k];
        *loss_out = l;
    }
    if (sl != 0 || p >= kParams) return;
    float gsum = part[0][pl];
#pragma unroll
    for (int k = 1; k < kSlices; ++k) gsum += part[k][pl];
    if (grad_out) grad_out[p] = gsum;
    if (lr > 0.0f) {
        const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
        const float m = b1 * adam[p] + (1.0f - b1) * gsum;
        const float v = b2 * adam[kParams + p] + (1.0f - b2) * gsum * gsum;
        adam[p] = m;
        adam[kParams + p] = v;
        const float wv = wts[p] - lr * (m * bc1) / (sqrtf(v * bc2) + eps);
        wts[p] = wv;
        wbf[p] = static_cast<__bf16>(wv);
    }
}

__global__ void refresh_bf16_kernel(const float *__restrict__ wts, __bf16 *__restrict__ wbf) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < kParams) wbf[p] = static_cast<__bf16>(wts[p]);
}

}  // namespace

// ----------------------------------------------------------- launchers ----

hipError_t launch_record(const lll_plan &p, int64_t n_paths, int R, uint64_t seed, float *states,
                         int *kidx, hipStream_t st) {
    PathArgs<float> a = detail::make_args<float>(p, seed, n_paths, 0, nullptr);
    a.stream_word = (p.struct_id & 0xFFFFFFu) | (1u << 24);  // tag 1: training data
    const dim3 grid(static_cast<unsigned>((n_paths + kBlock - 1) / kBlock));
    if (p.nmax != kRates) return hipErrorInvalidValue;
    hipLaunchKernelGGL(record_kernel<kRates>, grid, dim3(kBlock), 0, st, a, R, states, kidx);
    return hipGetLastError();
}

hipError_t launch_labels(const lll_plan &p, const double *E, const float *states, const int *kidx,
                         const int64_t *poff, int64_t n_states, __bf16 *feat, float *label,
                         hipStream_t st) {
    const dim3 grid(static_cast<unsigned>((n_states + 63) / 64));
    hipLaunchKernelGGL(label_kernel, grid, dim3(64), 0, st, states, kidx, poff, n_states, p.nmax,
                       p.off, p.N, p.s, p.d.tenor, p.d.delta, p.d.L0, p.d.vol, E, p.d.w,
                       p.alpha, p.beta, p.delta_nig, feat, label);
    return hipGetLastError();
}

hipError_t launch_stats(const lll_plan &p, const float *states, const int *kidx, int64_t n_states,
                        const float *label, int64_t n_pairs, float *out, hipStream_t st) {
    hipLaunchKernelGGL(stats_kernel, dim3(1), dim3(256), 0, st, states, kidx, n_states, p.nmax,
                       p.off, p.s, label, n_pairs, out);
    return hipGetLastError();
}

hipError_t launch_init(float *wts, __bf16 *wbf, float *adam, uint64_t seed, hipStream_t st) {
    hipLaunchKernelGGL(init_kernel, dim3((kParams + 255) / 256), dim3(256), 0, st, wts, wbf, adam,
                       static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32));
    return hipGetLastError();
}

hipError_t launch_refresh(const float *wts, __bf16 *wbf, hipStream_t st) {
    hipLaunchKernelGGL(refresh_bf16_kernel, dim3((kParams + 255) / 256), dim3(256), 0, st, wts, wbf);
    return hipGetLastError();
}

// One pass over B samples (drawn among n_pairs rows by (seed, step), or rows 0..B-1
// with n_pairs = 0): forward (and backward when gpart != null), then the fixed-order
// reduction (and an Adam step when lr > 0).
hipError_t launch_tiles(const __bf16 *feat, const float *target, int64_t n_pairs, uint32_t step,
                        uint64_t seed, int B, float inv_sigma, const float *wts, const __bf16 *wbf, float *gpart,
                        float *lpart, float *yout, float *loss_out, float *wts_mut,
                        __bf16 *wbf_mut, float *adam, float *grad_out, float lr, float bc1,
                        float bc2, hipStream_t st) {
    const int tiles = (B + kTile - 1) / kTile;
    const uint64_t n = static_cast<uint64_t>(n_pairs);
    TileArgs t{feat, target, B, n, n ? ~uint64_t{0} / n : 0, step, static_cast<uint32_t>(seed),
               static_cast<uint32_t>(seed >> 32), inv_sigma, 1.0f / static_cast<float>(B), wbf,
               wts, gpart, lpart, yout};
    hipLaunchKernelGGL(tile_kernel, dim3(tiles), dim3(kTrainBlock), 0, st, t);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !gpart) return e;
    hipLaunchKernelGGL(reduce_adam_kernel, dim3((kParams + kParamsPerBlock - 1) / kParamsPerBlock),
                       dim3(256), 0, st, gpart,
                       tiles, lpart, loss_out, wts_mut, wbf_mut, adam, grad_out, lr, bc1, bc2);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace lll
