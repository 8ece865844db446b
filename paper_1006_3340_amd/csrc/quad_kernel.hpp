// quad_kernel.hpp -- the path kernel of small passes: four lanes a path.
//
// A pass of few paths leaves most SIMDs of the chip with one wavefront or none, and one
// wavefront runs the step of path_kernel.hpp at its latency: every step's table rows come
// from beyond the XCD's L2 on first touch, node by node (6,700 cycles a step at 20 rates).
// Here a quad of lanes shares one path (16 paths a wavefront, 64 a block), so the same
// pass has four times the wavefronts and a quarter of the serial work in each:
//   - lane c of the quad draws the increments of steps 4 i + c, eight steps at a time;
//   - it owns the slots j = 4 g + c: their state, ell, update and rates at a fixing;
//   - it runs the coupling recursion over all rates for the nodes q = 4 i + c (rules are
//     padded to a multiple of four nodes with zero rows); a 4 x 4 transpose within the
//     quad brings the four nodes' R of a slot to its owner, which adds them in node order;
//   - at a fixing it takes the strikes t = 4 i + c.
// Every path's state sees the operations of path_kernel.hpp in the same order and the
// sums over a block's 64 paths are taken in wave_sum's order, so which of the two
// kernels ran cannot be told from FP32 results.
// Exchanges within a quad are DPP operands.  The block streams the tables through LDS
// in chunks of units (four node rows and the step's lambda and drifts each); the next chunk
// is in flight in registers while one is used.  The fixed slots are left out in eights:
// straight-line code over the rest, so that its LDS reads go out together (a guard per four
// slots left each read's latency exposed), and few enough bodies to stay in the instruction
// cache.  4,000 paths, FULL, against path_kernel.hpp: 277 against 637 us (FP32, 20 rates, 200
// steps), 968 against 1,970 (40 rates, 400 steps), 227 against 402 (FP64, 10 rates,
// 100 steps), of which 60 to 80 us are the set-up and the reduction.
#pragma once

namespace lll {
namespace detail {

template <int CTRL>
__device__ __forceinline__ float quad_dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                                0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double quad_dpp(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0u, static_cast<uint32_t>(u), CTRL, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0u, static_cast<uint32_t>(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E;  // quad_perm [1,0,3,2] and [2,3,0,1]
constexpr int kQuadPaths = kBlock / 4;     // paths per block

// The values of slots 4 g .. 4 g + 3 from their owners.
template <typename Real>
__device__ __forceinline__ void quad_spread(Real own, Real *v) {
    v[0] = quad_dpp<0x00>(own);
    v[1] = quad_dpp<0x55>(own);
    v[2] = quad_dpp<0xAA>(own);
    v[3] = quad_dpp<0xFF>(own);
}

// v[i] of lane c becomes v[c] of lane i.
template <typename Real>
__device__ __forceinline__ void quad_transpose(Real (&v)[4], int c) {
    const bool odd = c & 1, high = c & 2;
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const Real t = quad_dpp<kXor1>(odd ? v[i] : v[i + 1]);
        v[i] = odd ? t : v[i];
        v[i + 1] = odd ? v[i + 1] : t;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const Real t = quad_dpp<kXor2>(high ? v[i] : v[i + 2]);
        v[i] = high ? t : v[i];
        v[i + 2] = high ? v[i + 2] : t;
    }
}

// The table stream of a block.  A unit holds, of one step, four node rows (E by node and
// slot, W E by slot and node; FIRST: the step's K2 rows; FROZEN: nothing) and per slot
// (lambda, -kappa dt, b0 dt).
template <typename Real, int NMAX, int SCHEME>
struct QuadStream {
    static constexpr int V = 16 / sizeof(Real);  // reals per 16-byte piece
    typedef Real Vec __attribute__((ext_vector_type(V)));
    static constexpr bool kTable = SCHEME == kFull || SCHEME == kPicard || SCHEME == kSecond;
    static constexpr int kPieces = (kTable ? 8 * NMAX : SCHEME == kFirst ? NMAX * NMAX : 0) / V;
    static constexpr int kUnitPieces = kPieces + 3 * NMAX / V;
    static constexpr int kLoads = 4;             // pieces per thread and chunk
    static constexpr int kUnits =
        kLoads * kBlock / kUnitPieces < 32 ? kLoads * kBlock / kUnitPieces : 32;
    static constexpr int kRow = NMAX + V;        // LDS row of E or K2
    static constexpr int kWE = 4 * kRow;         // offsets in a unit
    static constexpr int kHead = kTable ? kWE + 4 * NMAX : SCHEME == kFirst ? NMAX * kRow : 0;
    static constexpr int kUnit = kHead + 4 * NMAX;
    static_assert(kUnits >= 1, "a unit has to fit a chunk");

    Vec piece[kLoads];

    // the chunk's pieces to registers; cum[m]: units before period m, inv[m] = 2^32 / (its
    // units a step) rounded up, 0 for one unit (the quotient is exact: units a period times
    // units a step < 2^32), m0: a period at or before the chunk's first unit
    __device__ __forceinline__ void load(const PathArgs<Real> &a, const int *cum,
                                         const uint32_t *inv, int first, int total, int m0) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int e = threadIdx.x + kBlock * i, r = e % kUnitPieces;
            const int unit = min(first + e / kUnitPieces, total - 1);
            int m = m0;
            while (unit >= cum[m + 1]) ++m;
            const int in = unit - cum[m];
            int k = m * a.s, group = 0;
            if (kTable && inv[m]) {
                const int step = __umulhi(in, inv[m]);
                group = in - step * ((cum[m + 1] - cum[m]) / a.s);
                k += step;
            } else {
                k += in;
            }
            const Real *src;
            if (r < kPieces) {
                src = kTable ? (const Real *)a.ew + ((size_t)k * kQ + 4 * group) * (NMAX * 2) + r * V
                             : (const Real *)a.k2 + (size_t)k * (NMAX * NMAX) + r * V;
            } else {
                const int h = r - kPieces, which = h / (NMAX / V);
                src = which == 0 ? (const Real *)a.lam
                                 : which == 1 ? (const Real *)a.drift0 : (const Real *)a.frozen;
                src += (size_t)k * NMAX + h % (NMAX / V) * V;
            }
            piece[i] = *reinterpret_cast<const Vec *>(src);
        }
    }
    __device__ __forceinline__ void store(Real *lds) const {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int e = threadIdx.x + kBlock * i, u = e / kUnitPieces, r = e % kUnitPieces;
            if (u >= kUnits) continue;
            Real *unit = lds + u * kUnit;
            if (r < kPieces) {
                if constexpr (kTable) {
                    const int node = r / (2 * NMAX / V), j = r % (2 * NMAX / V) * V / 2;
#pragma unroll
                    for (int b = 0; b < V / 2; ++b) {
                        unit[node * kRow + j + b] = piece[i][2 * b];
                        unit[kWE + 4 * (j + b) + node] = piece[i][2 * b + 1];
                    }
                } else {
                    const int j = r * V / NMAX, l = r * V % NMAX;
                    *reinterpret_cast<Vec *>(unit + j * kRow + l) = piece[i];
                }
            } else {
                const int h = r - kPieces, which = h / (NMAX / V), j = h % (NMAX / V) * V;
#pragma unroll
                for (int b = 0; b < V; ++b) unit[kHead + 4 * (j + b) + which] = piece[i][b];
            }
        }
    }
};

// Four consecutive reals from LDS, 16 bytes a read.
template <typename Real>
__device__ __forceinline__ void read4(const Real *p, Real (&v)[4]) {
    constexpr int V = 16 / sizeof(Real);
    typedef Real Vec __attribute__((ext_vector_type(V)));
#pragma unroll
    for (int i = 0; i < 4 / V; ++i) {
        const Vec x = *reinterpret_cast<const Vec *>(p + V * i);
#pragma unroll
        for (int b = 0; b < V; ++b) v[V * i + b] = x[b];
    }
}

// f(LO) with the largest even LO <= g0, LO < G.
template <int G, int LO = 0, typename F>
__device__ __forceinline__ void from_group(int g0, F &&f) {
    if constexpr (LO + 2 < G) {
        if (g0 >= LO + 2) {
            from_group<G, LO + 2>(g0, f);
            return;
        }
    }
    f(std::integral_constant<int, LO>{});
}

template <typename Real, int NMAX, int SCHEME>
__global__ void __launch_bounds__(kBlock) quad_kernel(PathArgs<Real> a) {
    typedef QuadStream<Real, NMAX, SCHEME> Stream;
    constexpr int G = NMAX / 4;
    __shared__ __attribute__((aligned(16))) Real units[Stream::kUnits * Stream::kUnit];
    __shared__ double pays[2][LLL_S_MAX + 1][kQuadPaths];
    __shared__ double steps[NMAX * 4], deltas[NMAX], L0s[NMAX], strikes[NMAX * LLL_S_MAX];
    __shared__ Real dts[NMAX];
    __shared__ int cum[NMAX + 1];
    __shared__ uint32_t inv[NMAX];
    const int tid = threadIdx.x, lane = tid % kWave, c = lane % 4;
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kQuadPaths + tid / 4;
    const bool active = gid < a.n_paths;
    const int64_t p = a.path_offset + gid;
    const uint32_t p_lo = static_cast<uint32_t>(p);
    const uint32_t p_hi = static_cast<uint32_t>(static_cast<uint64_t>(p) >> 32);
    const bool brownian = a.brownian != 0, nodes = Stream::kTable && !brownian;
    const int N = a.N, K = a.N * a.s, S = a.S;
    for (int i = tid; i < 4 * N; i += kBlock) steps[i] = a.steps[i];
    for (int i = tid; i < N * S; i += kBlock) strikes[i] = a.strikes[i];
    if (tid < NMAX) {
        deltas[tid] = a.deltas[tid];
        L0s[tid] = a.L0s[tid];
    }
    if (tid < N) {
        dts[tid] = a.dt[tid * a.s];
        const uint32_t per = nodes ? (a.nq[tid * a.s] + 3) / 4 : 1;  // units a step
        cum[tid + 1] = a.s * per;
        inv[tid] = per == 1 ? 0u : ~0u / per + 1u;
    }
    if (tid == 0) cum[0] = 0;
    __syncthreads();
    if (tid == 0)
        for (int m = 0; m < N; ++m) cum[m + 1] += cum[m];
    __syncthreads();
    const int total = cum[N];

    Real X[G], pred[G], cinv[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        X[g] = Real(0);
        cinv[g] = ((const Real *)a.cinv)[4 * g + c];
        pred[g] = SCHEME == kPicard ? ell_of(Real(0), cinv[g]) : Real(0);
    }
    Stream stream;
    stream.load(a, cum, inv, 0, total, 0);
    int first = 0, used = Stream::kUnits;  // the chunk's first unit, its units used up
    Real dHs[2] = {}, dt = Real(0);
    int m = 0, js = 0, groups = 0;
    for (int k = 0; k < K; ++k) {
        const int j0 = a.off + m, g0 = j0 / 4;
        if (js == 0) {
            groups = (cum[m + 1] - cum[m]) / a.s;
            dt = dts[m];
        }
        if (k % 8 == 0) {  // two chains at once: one alone runs at its latency
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int kc = k + 4 * h + c;
                const double *sc = steps + 4 * min(kc / a.s, N - 1);
                const StepConsts cst{sc[0], sc[1], sc[2], sc[3]};
                const uint4 w = philox4x32_10(
                    make_uint4(static_cast<uint32_t>(kc), p_lo, p_hi, a.stream_word), a.key0, a.key1);
                dHs[h] = static_cast<Real>(increment(w, cst, brownian, nullptr));
            }
        }
        const Real dH = __shfl(k & 4 ? dHs[1] : dHs[0], (lane & ~3) | (k & 3), kWave);
        Real ell[NMAX], C[G];
        if constexpr (SCHEME != kFrozen)
            from_group<G>(g0, [&](auto lo) {
#pragma unroll
                for (int g = lo; g < G; ++g) {
                    C[g] = Real(0);
                    quad_spread(SCHEME == kPicard ? pred[g] : ell_of(X[g], cinv[g]), ell + 4 * g);
                }
            });
        const Real *unit = nullptr;
        for (int q = 0; q < groups; ++q) {
            if (used == Stream::kUnits) {  // the same for the whole block
                __syncthreads();
                stream.store(units);
                __syncthreads();
                first += used;
                used = 0;
                stream.load(a, cum, inv, min(first, total - 1), total, m);
            }
            unit = units + used++ * Stream::kUnit;
            if constexpr (Stream::kTable) {
                if (!nodes) break;
                const Real *Es = unit + c * Stream::kRow, *WEs = unit + Stream::kWE + 4 * c;
                from_group<G>(g0, [&](auto lo) {
                    Real R = Real(0), u = Real(1);  // SECOND_ORDER: R = e1 + e2, u = 1 + e1
#pragma unroll
                    for (int g = G - 1; g >= lo; --g) {
                        Real E[4], WE[4], Rs[4];
                        read4(Es + 4 * g, E);
                        read4(WEs + 16 * g, WE);
#pragma unroll
                        for (int i = 3; i >= 0; --i) {
                            Rs[i] = R;
                            if constexpr (SCHEME == kSecond) {
                                const Real t = ell[4 * g + i] * E[i];
                                R = fma(t, u, R);
                                u = fma(ell[4 * g + i], E[i], u);
                            } else {
                                R = fma(ell[4 * g + i], fma(E[i], R, E[i]), R);
                            }
                        }
                        quad_transpose(Rs, c);
#pragma unroll
                        for (int i = 0; i < 4; ++i) C[g] = fma(WE[i], Rs[i], C[g]);
                    }
                });
            }
        }
        const Real *head = unit + Stream::kHead + 4 * c;
        from_group<G>(g0, [&](auto lo) {
            Real h[G][4];
#pragma unroll
            for (int g = lo; g < G; ++g) read4(head + 16 * g, h[g]);
            if constexpr (Stream::kTable) {
                if (brownian) {  // C_i = c lambda_i sum_{l>i} ell_l lambda_l
                    Real T = Real(0);
#pragma unroll
                    for (int g = G - 1; g >= lo; --g) {
                        Real l4[4], above[4];
                        quad_spread(h[g][0], l4);
#pragma unroll
                        for (int i = 3; i >= 0; --i) {
                            above[i] = T;
                            T = fma(ell[4 * g + i], l4[i], T);
                        }
                        C[g] = static_cast<Real>(a.c) * h[g][0] *
                               (c & 2 ? (c & 1 ? above[3] : above[2]) : (c & 1 ? above[1] : above[0]));
                    }
                }
            }
            if constexpr (SCHEME == kFirst) {
                const Real *rows = unit + c * Stream::kRow;
#pragma unroll
                for (int g = lo; g < G; ++g)
#pragma unroll
                    for (int i = g; i < G; ++i) {
                        Real v[4];
                        read4(rows + 4 * g * Stream::kRow + 4 * i, v);
#pragma unroll
                        for (int b = 0; b < 4; ++b) C[g] = fma(ell[4 * i + b], v[b], C[g]);
                    }
            }
#pragma unroll
            for (int g = lo; g < G; ++g) {
                if constexpr (SCHEME == kFrozen) {
                    X[g] += fma(h[g][0], dH, h[g][2]);
                } else {
                    X[g] += fma(h[g][0], dH, fma(-C[g], dt, h[g][1]));
                    if constexpr (SCHEME == kPicard)
                        pred[g] = ell_advance(pred[g], static_cast<Real>(fma(h[g][0], dH, h[g][2])));
                }
            }
        });
        if (++js < a.s) continue;

        // fixing of rate m: Q, A, D and L_m as in fixing_quantities_lds, in every lane
        const bool swaption = a.product == LLL_SWAPTIONS;
        double Q = 1.0, A = 0.0, D = 1.0, Lown = 0.0;
        from_group<G>(g0, [&](auto lo) {
            double f[G], d[G];  // 1 + delta L and delta of the lane's slots, 1 and 0 below j0
#pragma unroll
            for (int g = lo; g < G; ++g) {
                const int j = 4 * g + c;
                const double L = L0s[j] * static_cast<double>(exp(X[g]));
                d[g] = j >= j0 ? deltas[j] : 0.0;
                f[g] = j >= j0 ? 1.0 + deltas[j] * L : 1.0;
                if (g == g0) Lown = L;
            }
#pragma unroll
            for (int g = G - 1; g >= lo; --g) {
                double f4[4], d4[4];
                quad_spread(f[g], f4);
                quad_spread(d[g], d4);
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    D = 4 * g + i == j0 ? Q : D;
                    A = fma(d4[i], Q, A);
                    Q *= f4[i];
                }
            }
        });
        const double Lc = __shfl(Lown, (lane & ~3) | (j0 & 3), kWave);
        if (!swaption && a.path_fix != nullptr && active && c == 0) {
            a.path_fix[gid * 2 * N + 2 * m] = Lc;
            a.path_fix[gid * 2 * N + 2 * m + 1] = D;
        }
        double (*pay)[kQuadPaths] = pays[m & 1];
        for (int t = c; t < S; t += 4) {
            const double v = payoff_value(swaption, strikes[m * S + t], Q, A, D, Lc);
            pay[t][tid / 4] = active ? fmax(v, 0.0) : 0.0;
        }
        if (c == 3) pay[S][tid / 4] = active ? Q : 0.0;
        __syncthreads();
        // 16 lanes a row of 64, in wave_sum's order: lanes 32, 16, 8, 4, 2, 1 apart
        const int t = tid / 16;
        if (t <= S) {
            const double *v = pay[t] + tid % 16;
            const double v0 = v[0], v1 = v[16], v2 = v[32], v3 = v[48];
            auto row_sum = [](double x) {
                x += quad_dpp<0x128>(x);  // row_ror:8
                x += quad_dpp<0x124>(x);  // row_ror:4
                x += quad_dpp<kXor2>(x);
                return x + quad_dpp<kXor1>(x);
            };
            auto itm = [](double x) { return x > 0.0 ? 1.0 : 0.0; };
            const double s1 = row_sum((v0 + v2) + (v1 + v3));
            const double s2 = row_sum(fma(v0, v0, v2 * v2) + fma(v1, v1, v3 * v3));
            const double ni = row_sum((itm(v0) + itm(v2)) + (itm(v1) + itm(v3)));
            double *out = a.partials + ((size_t)blockIdx.x * N + m) * (3 * S + 2);
            if (tid % 16 == 0) {
                if (t < S) {
                    out[t] = s1;
                    out[S + t] = s2;
                    out[2 * S + t] = ni;
                } else {
                    out[3 * S] = s1;
                    out[3 * S + 1] = s2;
                }
            }
        }
        js = 0;
        ++m;
    }
}

}  // namespace detail
}  // namespace lll
