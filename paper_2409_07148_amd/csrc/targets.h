// Target densities p and regeneration densities u evaluated per lane.
//
// The Gaussian mixtures are evaluated in log space, in base 2 (log2 e is
// folded into the packed parameters on the host), with a blocked online
// log-sum-exp: a block of components' terms, one maximum over them and the
// running maximum, one exponential per term and one per block.  Neither far
// tails nor sharp peaks leave the float32 range.  Parameters are read from
// a packed slab whose addresses are wave-uniform: from global memory they
// become scalar loads (SGPR operands of the FMAs); with LDS staging they
// are broadcast reads.
#pragma once

#include <type_traits>

#include "../../include/restore.h"
#include "device_common.h"

namespace restore {

// Parameters read through the constant address space: wave-uniform loads
// from it always become scalar (SMEM) loads feeding SGPR operands, even
// when the kernel also writes global memory (image splats) that the
// compiler cannot prove disjoint from the slab.
typedef const __attribute__((address_space(4))) float *const_fptr;
// An LDS copy of read-only parameters (per-lane indexed reads are ds_reads).
typedef const __attribute__((address_space(3))) float *lds_fptr;

// A packed full-covariance slab read both ways at once: the scalar cache,
// and an LDS copy of the last rows of every component's factor (see
// GmmFull; one 16-byte aligned block of MixRows<D>::STRIDE floats each).
struct MixPtr {
    const_fptr P;
    lds_fptr L;
};

// An isotropic slab whose first four components stay in vector registers
// through the step loop, for populations with a wave or less a SIMD: read at
// each step they would put a scalar load's latency (some 200 cycles) on its
// path.  A mixture of fewer is filled up with copies of its last one, which
// nothing reads.
constexpr int HELD = 4;
template <int D>
struct HeldPtr {
    static constexpr int STRIDE = comp_stride(TGT_ISO, D);
    const_fptr P;
    float q[HELD * STRIDE];
    __device__ __forceinline__ HeldPtr(const_fptr slab, int K) : P(slab) {
        int zero;   // in a vector register, and the loads with it
        asm("v_mov_b32_e32 %0, 0" : "=v"(zero));
#pragma unroll
        for (int k = 0; k < HELD; ++k)
#pragma unroll
            for (int i = 0; i < D + 2; ++i) q[k * STRIDE + i] = P[min(k, K - 1) * STRIDE + i + zero];
    }
};
template <class PT>
struct IsHeld : std::false_type {};
template <int D>
struct IsHeld<HeldPtr<D>> : std::true_type {};

// Chains spread over several lanes (small populations and the tails of
// drains, where a SIMD has a wave or two and a step costs its instruction
// stream): every lane of a group of G holds the whole chain and computes
// the same step, and the group shares out the density's components.  The
// lanes of a group take every branch together.
// A full-covariance slab in LDS, four lanes a chain:
struct QuadPtr {
    lds_fptr L;
    int role;   // the lane within its chain's four
};
// The isotropic mixture of the unadjusted jump process, sixteen lanes a
// chain (see GmmIsoInflow):
template <int D>
struct RowPtr {
    HeldPtr<D> H;
    int role;   // the lane within its chain's sixteen
    // the first pass's component of this lane: means and inflow parameters
    float m[2], c, ivar, alpha, beta;
    __device__ __forceinline__ RowPtr(const_fptr slab, int K, int lane) : H(slab, K), role(lane) { load(K, 0); }
    __device__ __forceinline__ void load(int K, int k0) {
        const int S = comp_stride(TGT_ISO, D), k = min(k0 + role / (2 * D), K - 1);
        m[0] = H.P[k * S + 1];
        m[1] = D == 2 ? H.P[k * S + 2] : 0.0f;
        const const_fptr q = H.P + K * S + k * INFLOW_STRIDE;
        c = q[0]; ivar = q[1]; alpha = q[2]; beta = q[3];
    }
};
template <class PT>
struct IsRow : std::false_type {};
template <int D>
struct IsRow<RowPtr<D>> : std::true_type {};
// lane R's x of each group of four, and of each row of sixteen
template <int R>
__device__ __forceinline__ float quad_bcast(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), R * 0x55, 0xf, 0xf, true));
}
template <int R>
__device__ __forceinline__ float row_bcast(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x150 + R, 0xf, 0xf, true));
}
// f(0), .., f(N - 1) with compile-time indices
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// Components per log-sum-exp block: four for values alone, two when the
// gradient needs each component's vector until the block's weights are
// known (fewer live registers), and fewer while the block's parameters
// (STRIDE floats per component, scalar operands of the FMAs) would take
// more than LSE_SGPR_BUDGET scalar registers at once: past that the
// compiler reloads and spills them, which costs more than the shared
// maximum saves.
// BMAX caps the block for kernels whose own state already crowds the
// scalar registers.
constexpr int LSE_SGPR_BUDGET = 96;
template <int STRIDE, bool GRAD, int BMAX = 4>
struct LseBlock {
    static constexpr int cap(int b) { return (b > 1 && b * STRIDE > LSE_SGPR_BUDGET) ? cap(b / 2) : b; }
    static constexpr int value = cap((GRAD ? 2 : 4) < BMAX ? (GRAD ? 2 : 4) : BMAX);
};

// Isotropic Gaussian mixture, slab terms in base 2 (h_k = log2 e / (2 s_k^2)):
//   a_k = c_k - h_k |y - m_k|^2 = log2(w_k N(y; m_k, s_k^2 I)),
//   grad log p = -2 ln 2 sum_k r_k h_k (y - m_k),  r = softmax of the a_k in base 2.
template <int D>
struct GmmIso {
    static constexpr int STRIDE = comp_stride(TGT_ISO, D);

    // P: the slab, or a pointer to the held components
    template <int B, bool GRAD, class PT>
    __device__ __forceinline__ static void push(PT P, int k0, const float y[D], float &M, float &S, float G[D],
                                                bool want) {
        float a[B], dx[B][D];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const auto pk = P + (k0 + b) * STRIDE;
            float q = 0.0f;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                dx[b][i] = y[i] - pk[1 + i];
                q = fmaf(dx[b][i], dx[b][i], q);
            }
            a[b] = pk[0] - pk[1 + D] * q;
        }
        float sc, w[B];
        lse2_block<B>(M, S, a, sc, w);
        if (GRAD && want) {
#pragma unroll
            for (int i = 0; i < D; ++i) G[i] *= sc;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const float wh = w[b] * P[(k0 + b) * STRIDE + 1 + D];
#pragma unroll
                for (int i = 0; i < D; ++i) G[i] = fmaf(wh, dx[b][i], G[i]);
            }
        }
    }

    template <bool GRAD, int BMAX = 4, class PT>
    __device__ __forceinline__ static float eval(PT P, int K, const float y[D], float g[D], bool want) {
        constexpr int B = LseBlock<STRIDE, GRAD, BMAX>::value;
        float M = -INFINITY, S = 0.0f;
        float G[D];
#pragma unroll
        for (int i = 0; i < D; ++i) G[i] = 0.0f;
        int k = 0;
        if constexpr (IsHeld<PT>::value) {
            const float *q = P.q;
            if (K >= HELD) {
#pragma unroll
                for (int h = 0; h < HELD; h += B) push<B, GRAD>(q, h, y, M, S, G, want);
                for (k = HELD; k + B <= K; k += B) push<B, GRAD>(P.P, k, y, M, S, G, want);
                for (; k < K; ++k) push<1, GRAD>(P.P, k, y, M, S, G, want);
            } else {
                // (blocks first, as below; B is 1, 2 or 4)
                if (B == 2 && K >= 2) push<B == 2 ? 2 : 1, GRAD>(q, 0, y, M, S, G, want);
                else push<1, GRAD>(q, 0, y, M, S, G, want);
                if (B != 2 && K >= 2) push<1, GRAD>(q, 1, y, M, S, G, want);
                if (K == 3) push<1, GRAD>(q, 2, y, M, S, G, want);
            }
        } else {
            for (; k + B <= K; k += B) push<B, GRAD>(P, k, y, M, S, G, want);
            for (; k < K; ++k) push<1, GRAD>(P, k, y, M, S, G, want);
        }
        if (GRAD && want) {
            const float f = (-2.0f * LN2) / S;
#pragma unroll
            for (int i = 0; i < D; ++i) g[i] = G[i] * f;
        }
        return lse2_ln(M, S);
    }
};

// log (Q^T p)(y) of the isotropic mixture for the unadjusted random-walk
// jump process with jump N(0, sigma^2 I): the density at y of x + sigma z
// with x ~ p on the box, (Q^T p)(y) = int_box p(x) N(y; x, sigma^2 I) dx.
// Per component and coordinate the Gaussian product identity leaves
// N(y_i; m_i, s^2 + sigma^2) times the box mass of a Gaussian centred at
// c_i = m_i + alpha (y_i - m_i) with 1 / sqrt(2 var) = beta:
//   (erf(beta (1 - c_i)) + erf(beta c_i)) / 2.
// The parameters (INFLOW_STRIDE per component) follow the K components.
//
// With sixteen lanes a chain and d <= 2, each lane takes one error function:
// 2d lanes a component, 8 / d components at a time; the lanes of a component
// share its truncation factors (a sum and a product of two, so the same bits
// in either order) and its logarithm, and every lane adds the components up
// in order.
template <int D>
struct GmmIsoInflow {
    __device__ __forceinline__ static float log_inflow_row(RowPtr<D> P, int K, const float y[D]) {
        static_assert(D <= 2, "one or two coordinates");
        constexpr int PER = 8 / D;   // components per pass
        const int i = D == 2 ? (P.role >> 1) & 1 : 0;
        const bool lower = (P.role & 1) != 0;
        float M = -INFINITY, S = 0.0f;
        for (int k0 = 0; k0 < K; k0 += PER) {
            if (k0 > 0) P.load(K, k0);
            float q = 0.0f, c = 0.0f;
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const float dx = y[j] - P.m[j];
                q = fmaf(dx, dx, q);
                const float cj = fmaf(P.alpha, dx, P.m[j]);
                c = j == i ? cj : c;
            }
            const float e = erff(P.beta * (lower ? c : 1.0f - c));
            const float other = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(e), 0xb1, 0xf, 0xf, true));
            float mass = 0.5f * (e + other);
            if (D == 2)
                mass *= __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(mass), 0x4e, 0xf, 0xf, true));
            const float ak = fmaf(-0.5f * P.ivar, q, P.c) + logf(mass);
            static_for<0, PER>([&](auto j) {
                if (k0 + j < K) {
                    float sc, w;
                    lse_push(M, S, row_bcast<j * 2 * D>(ak), sc, w);
                }
            });
        }
        return M + logf(S);
    }

    template <class PT>
    __device__ __forceinline__ static float log_inflow(PT P, int K, const float y[D]) {
        const auto A = P + K * GmmIso<D>::STRIDE;
        float M = -INFINITY, S = 0.0f;
        // unrolled by four for wide scalar loads, as in GmmIso::eval
#pragma unroll 4
        for (int k = 0; k < K; ++k) {
            const auto pk = P + k * GmmIso<D>::STRIDE;
            const auto qk = A + k * INFLOW_STRIDE;
            const float ivar = qk[1], alpha = qk[2], beta = qk[3];
            float q = 0.0f, mass = 1.0f;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const float dx = y[i] - pk[1 + i];
                q = fmaf(dx, dx, q);
                const float c = fmaf(alpha, dx, pk[1 + i]);
                mass *= 0.5f * (erff(beta * (1.0f - c)) + erff(beta * c));
            }
            const float ak = fmaf(-0.5f * ivar, q, qk[0]) + logf(mass);
            float sc, w;
            lse_push(M, S, ak, sc, w);
        }
        return M + logf(S);
    }
};

// Which part of a full-covariance component the step kernels read from LDS.
// What bounds the density is issue.  Two waves of a SIMD issue FP32
// instructions side by side (2.05 cycles each) only while at most one of
// the two reads a scalar register: with a scalar operand in each a SIMD
// issues one per 4.1 cycles.  An LDS broadcast read delivers a parameter
// to a vector register in 4.2 cycles of the SIMD's share, beside the VALU.
// So half the parameters take each way (48 parameters from the scalar cache
// alone cost 218 cycles a wave, from LDS alone 203, half and half 143;
// between a third and two thirds the choice does not matter).  The last
// rows are one contiguous run: as many whole rows as fit in half the floats.
template <int D>
struct MixRows {
    static constexpr int FIRST = mix_first_row(D);            // first row read from LDS
    static constexpr int AT = FIRST * (FIRST + 1) / 2;        // its index in the packed triangle
    static constexpr int COUNT = D * (D + 1) / 2 - AT;        // floats per component
    static constexpr int STRIDE = mix_stride(D);
};

// One component's factor entries W[i (i + 1) / 2 + j].
template <int D, class PT>
struct FactorOf {
    const PT W;
    __device__ __forceinline__ FactorOf(PT P, int k) : W(P + k * comp_stride(TGT_FULL, D) + 1 + D) {}
    __device__ __forceinline__ float operator[](int i) const { return W[i]; }
};
template <int D>
struct FactorOf<D, MixPtr> {
    using R = MixRows<D>;
    const const_fptr W;
    float v[R::STRIDE];
    __device__ __forceinline__ FactorOf(MixPtr P, int k) : W(P.P + k * comp_stride(TGT_FULL, D) + 1 + D) {
        typedef float v4f __attribute__((ext_vector_type(4)));
        typedef const __attribute__((address_space(3))) v4f *lds_v4ptr;
        const auto q = (lds_v4ptr)(P.L + k * R::STRIDE);
#pragma unroll
        for (int i = 0; i < R::STRIDE / 4; ++i) {
            const v4f t = q[i];
            v[4 * i] = t.x; v[4 * i + 1] = t.y; v[4 * i + 2] = t.z; v[4 * i + 3] = t.w;
        }
    }
    __device__ __forceinline__ float operator[](int i) const { return i >= R::AT ? v[i >= R::AT ? i - R::AT : 0] : W[i]; }
};
template <class PT>
__device__ __forceinline__ PT scalar_part(PT P) { return P; }
__device__ __forceinline__ const_fptr scalar_part(MixPtr P) { return P.P; }

// Full-covariance Gaussian mixture with scaled whitening factors
// W_k = sqrt(log2 e / 2) L_k^-1 (S_k = L_k L_k^T, W_k lower triangular),
// terms in base 2:
//   v_k = W_k (y - m_k),  a_k = c_k - |v_k|^2 = log2(w_k N(y; m_k, S_k)),
//   grad log p = -2 ln 2 sum_k r_k W_k^T v_k  (= -sum_k r_k S_k^-1 (y - m_k)).
template <int D>
struct GmmFull {
    static constexpr int STRIDE = comp_stride(TGT_FULL, D);

    template <int B, bool GRAD, class PT>
    __device__ __forceinline__ static void push(PT P, int k0, const float y[D], float &M, float &S, float G[D],
                                                bool want) {
        float a[B], v[B][D];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const auto pk = scalar_part(P) + (k0 + b) * STRIDE;
            const FactorOf<D, PT> W(P, k0 + b);
            float dx[D];
#pragma unroll
            for (int i = 0; i < D; ++i) dx[i] = y[i] - pk[1 + i];
            // -a_k accumulated from -c_k: the sign folds into the maximum
            // and the differences of lse2_block
            float t = -pk[0];
#pragma unroll
            for (int i = 0; i < D; ++i) {
                float acc = W[i * (i + 1) / 2] * dx[0];
#pragma unroll
                for (int j = 1; j <= i; ++j) acc = fmaf(W[i * (i + 1) / 2 + j], dx[j], acc);
                v[b][i] = acc;
                t = fmaf(acc, acc, t);
            }
            a[b] = -t;
        }
        float sc, w[B];
        lse2_block<B>(M, S, a, sc, w);
        if (GRAD && want) {
#pragma unroll
            for (int j = 0; j < D; ++j) G[j] *= sc;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const FactorOf<D, PT> W(P, k0 + b);
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    float u = 0.0f;
#pragma unroll
                    for (int i = j; i < D; ++i) u = fmaf(W[i * (i + 1) / 2 + j], v[b][i], u);
                    G[j] = fmaf(w[b], u, G[j]);
                }
            }
        }
    }

    // Four components at a time, one per lane of the chain's four: each lane
    // forms its component's term and W^T v, then all four run the same
    // log-sum-exp blocks and gradient sums over the broadcast results, in
    // the order of push.  What bounds it is one wave's stream: 8-D takes
    // 8 + 36 + 8 (+ 36 with the gradient) of its instructions per four
    // components instead of per one.  The next four components' parameters
    // are read while these are worked on, where two sets fit.  The LDS copy
    // is filled up to a multiple of four with components of log-weight -inf
    // and W = 0: beside a component of the mixture their weights are 0 and
    // change no sum, nor the NaN of a density whose terms are all -inf.
    // Whole passes are straight lines (a wave alone on its SIMD loses some
    // 30 cycles a branch); the last one stops at the components left.
    template <bool GRAD, int BMAX>
    __device__ __forceinline__ static float eval_quad(QuadPtr P, int K, const float y[D], float g[D], bool want) {
        constexpr int B = LseBlock<STRIDE, GRAD, BMAX>::value;
        constexpr bool AHEAD = D <= 8;
        typedef float v4f __attribute__((ext_vector_type(4)));
        typedef const __attribute__((address_space(3))) v4f *lds_v4ptr;
        float M = -INFINITY, S = 0.0f;
        float G[D];
#pragma unroll
        for (int i = 0; i < D; ++i) G[i] = 0.0f;
        v4f next[STRIDE / 4];
        auto read = [&](int k0) {
            const auto q = (lds_v4ptr)(P.L + (k0 + P.role) * STRIDE);
#pragma unroll
            for (int i = 0; i < STRIDE / 4; ++i) next[i] = q[i];
        };
        if (AHEAD) read(0);
        auto pass = [&](int k0, auto whole) __attribute__((always_inline)) {
            if (!AHEAD) read(k0);
            float q[STRIDE];
#pragma unroll
            for (int i = 0; i < STRIDE; ++i) q[i] = next[i / 4][i % 4];
            if (AHEAD && whole) read(k0 + 4 < K ? k0 + 4 : k0);
            float t = -q[0], v[D], u[D], dx[D];
#pragma unroll
            for (int i = 0; i < D; ++i) dx[i] = y[i] - q[1 + i];
            const float *W = q + 1 + D;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                float acc = W[i * (i + 1) / 2] * dx[0];
#pragma unroll
                for (int j = 1; j <= i; ++j) acc = fmaf(W[i * (i + 1) / 2 + j], dx[j], acc);
                v[i] = acc;
                t = fmaf(acc, acc, t);
            }
            if (GRAD && want) {
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    u[j] = 0.0f;
#pragma unroll
                    for (int i = j; i < D; ++i) u[j] = fmaf(W[i * (i + 1) / 2 + j], v[i], u[j]);
                }
            }
            const float a = -t;
            // lanes R .. R + N - 1 as one log-sum-exp block
            auto block = [&](auto R, auto N) __attribute__((always_inline)) {
                float ab[N], w[N], sc;
                static_for<0, N>([&](auto b) { ab[b] = quad_bcast<R + b>(a); });
                lse2_block<N, true>(M, S, ab, sc, w);
                if (GRAD && want) {
#pragma unroll
                    for (int j = 0; j < D; ++j) G[j] *= sc;
                    static_for<0, N>([&](auto b) {
#pragma unroll
                        for (int j = 0; j < D; ++j) G[j] = fmaf(w[b], quad_bcast<R + b>(u[j]), G[j]);
                    });
                }
            };
            if constexpr (whole) {
                static_for<0, 4 / B>([&](auto i) __attribute__((always_inline)) {
                    block(std::integral_constant<int, i * B>{}, std::integral_constant<int, B>{});
                });
            } else {
                // the components past a multiple of B go one by one; for B
                // = 2 a filler in the block's second place gives the same
                constexpr std::integral_constant<int, 1> ONE{};
                if constexpr (B == 2) {
                    block(std::integral_constant<int, 0>{}, std::integral_constant<int, 2>{});
                } else {
                    block(std::integral_constant<int, 0>{}, ONE);
                    if (K - k0 >= 2) block(ONE, ONE);
                }
                if (K - k0 == 3) block(std::integral_constant<int, 2>{}, ONE);
            }
        };
        int k0 = 0;
        for (; k0 + 4 <= K; k0 += 4) pass(k0, std::true_type{});
        if (k0 < K) pass(k0, std::false_type{});
        if (GRAD && want) {
            const float f = (-2.0f * LN2) / S;
#pragma unroll
            for (int i = 0; i < D; ++i) g[i] = G[i] * f;
        }
        return lse2_ln(M, S);
    }

    template <bool GRAD, int BMAX = 4, class PT>
    __device__ __forceinline__ static float eval(PT P, int K, const float y[D], float g[D], bool want) {
        if constexpr (std::is_same<PT, QuadPtr>::value) {
            return eval_quad<GRAD, BMAX>(P, K, y, g, want);
        } else {
            constexpr int B = LseBlock<STRIDE, GRAD, BMAX>::value;
            float M = -INFINITY, S = 0.0f;
            float G[D];
#pragma unroll
            for (int i = 0; i < D; ++i) G[i] = 0.0f;
            int k = 0;
            for (; k + B <= K; k += B) push<B, GRAD>(P, k, y, M, S, G, want);
            for (; k < K; ++k) push<1, GRAD>(P, k, y, M, S, G, want);
            if (GRAD && want) {
                const float f = (-2.0f * LN2) / S;
#pragma unroll
                for (int i = 0; i < D; ++i) g[i] = G[i] * f;
            }
            return lse2_ln(M, S);
        }
    }
};

// Rendering-shaped integrand on [0,1]^12 (slab layout in restore_internal.h):
//   g(x) = tA(x0,x1) tB(x6..x11) [b + sum_l w_l h_l(x_{2l}, x_{2l+1})],
//   t(y) = 1 + (1/8) sum_m a_m sin(2 pi (<n_m, y> + phi_m / 2 pi)),
//   w_l h_l(u, v) = C_l exp(-kappa_l |omega(u,v) - dir_l|^2 / 2)  (= exp(kappa (dir.omega - 1))
//   for unit vectors, without the cancellation of dir.omega - 1 near the lobe),
//   omega = (2 sqrt(u (1 - u)) cos 2 pi v, 2 sqrt(u (1 - u)) sin 2 pi v, 1 - 2u).
// Texture phases are reduced modulo one revolution term by term (the
// frequencies are integers), so the hardware sine sees arguments in [0, 1).
template <int D>
struct Pss {
    // one sinusoid per iteration (not unrolled): only that row's scalars are
    // live, which keeps the slab from overflowing the SGPR file
    template <int DIM, class PT>
    __device__ __forceinline__ static float texture(PT freq, PT amp, PT phase, const float *y) {
        float t = 1.0f;
#pragma unroll 1
        for (int m = 0; m < 8; ++m) {
            float s = phase[m];
#pragma unroll
            for (int i = 0; i < DIM; ++i) s = __builtin_amdgcn_fractf(s + __builtin_amdgcn_fractf(freq[m * DIM + i] * y[i]));
            t = fmaf(amp[m], __builtin_amdgcn_sinf(s), t);
        }
        return t;
    }

    template <bool GRAD, int BMAX = 4, class PT>
    __device__ __forceinline__ static float eval(PT P, int K, const float y[D], float g[D], bool want) {
        static_assert(D == 12, "the rendering-shaped integrand lives on [0,1]^12");
        (void)K; (void)g; (void)want;
        const float ta = texture<2>(P + 0, P + 16, P + 24, y);
        const float tb = texture<6>(P + 32, P + 80, P + 88, y + 6);
        float light = P[111];
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const float u = y[2 * l], v = y[2 * l + 1];
            const float z = 1.0f - 2.0f * u;
            const float r = 2.0f * sqrtf(fmaxf(u * (1.0f - u), 0.0f));
            const auto dir = P + 96 + 3 * l;
            // the lobe exponent amplifies direction errors by ~kappa |omega - dir|,
            // so the azimuth uses the correctly rounded sin/cos of pi (2v)
            float sv, cv;
            sincospif(2.0f * v, &sv, &cv);
            const float d0 = r * cv - dir[0];
            const float d1 = r * sv - dir[1];
            const float d2 = z - dir[2];
            const float q = fmaf(d0, d0, fmaf(d1, d1, d2 * d2));
            light += expf(fmaf(-0.5f * P[105 + l], q, P[108 + l]));
        }
        // one logarithm of the product (ta, tb in (0, 2], light >= b: no
        // overflow; the product's two roundings add 2^-23 relative)
        return logf(ta * tb * light);
    }
};

// Learned regeneration distribution: defensive mixture
//   u(y) = beta 1_box(y) + (1 - beta) sum_k pi_k N(y; m_k, diag(s_k^2))
// (slab layout in restore_internal.h).  log u by the blocked base-2
// log-sum-exp with scalar-loaded parameters; sampling picks the share by
// the cumulative weights and gathers the chosen component per lane.
template <int D>
struct MuGmm {
    static constexpr int STRIDE = mu_stride(D);

    // log u(y).  P: the slab (scalar loads); R: its component blocks, either
    // P + 4 or an LDS copy.  The score fma(y_i, r_ki, n_ki) has two
    // per-component operands and a VALU instruction reads at most one
    // scalar register, so from P alone one of them costs a VALU move; from
    // the LDS copy r_ki arrives in a vector register by a ds_read.
    template <class PT, class RT>
    __device__ __forceinline__ static float log_u(PT P, RT R, int K, const float y[D]) {
        // the defensive share as the first term of the sum: log2 beta on the
        // box (S = 1), nothing outside it (S = 0)
        const bool in = in_unit_box<D>(y);
        float M = in ? P[0] : -INFINITY, S = 1.0f;
        if (M == -INFINITY) S = 0.0f;
        constexpr int B = LseBlock<STRIDE, false>::value;
        int k = 0;
        for (; k + B <= K; k += B) push<B>(P, R, k, y, M, S);
        for (; k < K; ++k) push<1>(P, R, k, y, M, S);
        return lse2_ln(M, S);
    }

    // B components' terms a_k = c_k - |(y - m_k) r_k|^2 with the scaled
    // score fma(y_i, r_ki, -m_ki r_ki), accumulated from -c_k as in GmmFull
    template <int B, class PT, class RT>
    __device__ __forceinline__ static void push(PT P, RT R, int k0, const float y[D], float &M, float &S) {
        float a[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const auto pk = P + 4 + (k0 + b) * STRIDE;
            const auto rk = R + (k0 + b) * STRIDE;
            // from the LDS copy in 16-byte reads (component blocks are a
            // multiple of 4 floats from a 16-byte aligned start)
            float r[D];
            if constexpr (std::is_same<typename std::remove_cv<RT>::type, lds_fptr>::value && D % 4 == 0) {
                typedef float v4f __attribute__((ext_vector_type(4)));
                typedef const __attribute__((address_space(3))) v4f *lds_v4ptr;
                const auto r4 = (lds_v4ptr)rk;
#pragma unroll
                for (int i = 0; i < D / 4; ++i) {
                    const v4f v = r4[i];
                    r[4 * i] = v.x; r[4 * i + 1] = v.y; r[4 * i + 2] = v.z; r[4 * i + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < D; ++i) r[i] = rk[i];
            }
            float t = -pk[2 * D];
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const float z = fmaf(y[i], r[i], pk[D + i]);
                t = fmaf(z, z, t);
            }
            a[b] = -t;
        }
        float sc, w[B];
        lse2_block<B>(M, S, a, sc, w);
    }

    // y ~ mu from the category uniform, the candidate uniforms (uniform
    // share) and their Box-Muller normals (Gaussian components)
    // (R as in log_u: with the LDS copy, which also holds the cumulative
    // weights, the component is found by a binary search with per-lane LDS
    // reads instead of K - 1 compares; both give the largest j with
    // cum[j] <= u_cat, the cumulative weights being non-decreasing)
    template <class PT, int NC, class RT = PT>
    __device__ __forceinline__ static void sample(PT P, const float *G, int K, float u_cat, const float cand[NC],
                                                  float y[D], RT R = RT()) {
        const auto cum = P + 4 + K * STRIDE;
        if (u_cat < cum[0]) {
#pragma unroll
            for (int i = 0; i < D; ++i) y[i] = cand[i];
            return;
        }
        int pick = 0;
        if constexpr (std::is_same<typename std::remove_cv<RT>::type, lds_fptr>::value) {
            static_assert(RESTORE_MAX_COMP <= 64, "six halvings cover the components");
            const auto lcum = R + K * STRIDE;
#pragma unroll
            for (int h = 32; h > 0; h >>= 1) {
                const int j = pick + h;
                if (j < K && lcum[j] <= u_cat) pick = j;
            }
        } else {
            (void)R;
            // eight weights per scalar-load wait
#pragma unroll 8
            for (int j = 1; j < K; ++j) pick += (cum[j] <= u_cat) ? 1 : 0;
        }
        float z[D];
        box_muller<D, NC, ROOT_HW>(cand, z);
        const float *ms = G + 4 + K * STRIDE + K + pick * 2 * D;
#pragma unroll
        for (int i = 0; i < D; ++i) y[i] = fmaf(ms[D + i], z[i], ms[i]);
    }
};

template <int D, int TGT>
struct TargetOf;
template <int D>
struct TargetOf<D, TGT_ISO> { using type = GmmIso<D>; };
template <int D>
struct TargetOf<D, TGT_FULL> { using type = GmmFull<D>; };
template <int D>
struct TargetOf<D, TGT_PSS> { using type = Pss<D>; };

// log p(y) with p = 0 outside the unit box; with GRAD, lanes that `want` it
// also get grad log p(y) (the gradient work is skipped by waves where no
// lane wants it).
template <int D, int TGT, bool GRAD, int BMAX = 4, class PT>
__device__ __forceinline__ float log_target(PT P, int K, const float y[D], float g[D], bool want = true) {
    float lp;
    if constexpr (IsRow<PT>::value)
        lp = TargetOf<D, TGT>::type::template eval<GRAD, BMAX>(P.H, K, y, g, want);
    else
        lp = TargetOf<D, TGT>::type::template eval<GRAD, BMAX>(P, K, y, g, want);
    const bool in = in_unit_box<D>(y);
    if (GRAD && want) {
#pragma unroll
        for (int i = 0; i < D; ++i) g[i] = in ? g[i] : 0.0f;
    }
    return in ? lp : -INFINITY;
}

}  // namespace restore
