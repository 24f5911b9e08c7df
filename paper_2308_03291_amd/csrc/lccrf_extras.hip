// Queries derived from the partition function (paper, sections "Computing Probability of a
// Structure and Partition Function" and "Entropy and KL Divergence"): the log-probability of
// a given tag path and the entropy of the distribution.  The heavy part of both is the
// first pass of the chain kernels; what is here only finishes them.
#include "lccrf_chain_args.h"
#include "lccrf_device.h"
#include "lccrf_expect.h"
#include "lccrf_launch.h"
#include "lccrf_linear.h"

namespace lccrf {

// log p(y) = phi[0][0][y_0] + sum_i phi[i][y_{i-1}][y_i] - logZ.  One workgroup per sequence; the
// score is summed in double precision (it and logZ are both of the size of the chain's total,
// their difference is not).  A tag outside [0, T) makes the result NaN.
constexpr int kPathThreads = 512;
// logZ64 null: log Z is formed here, by one of the waves while the others gather, from the vectors a first pass has left at the
// meeting position (a launch less: the paper's shape 5 us).
template <typename TIN>
__global__ __launch_bounds__(kPathThreads) void path_log_prob_kernel(const TIN* __restrict__ phi, const int32_t* __restrict__ lengths,
                                                          const int32_t* __restrict__ tags, int N, int T,
                                                          const double* __restrict__ logZ64, MeetingVectors mv, float* __restrict__ out) {
    __shared__ double part[kPathThreads / 64], lz;
    __shared__ int part_bad[kPathThreads / 64];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int L = clamp_length(lengths, b, N);
    const int32_t* y = tags + (size_t)b * N;
    const TIN* phib = phi + (size_t)b * N * T * T;
    double acc = 0.0;
    bool bad = false;
    if (!logZ64 && wave == kPathThreads / 64 - 1 && L > 0) {
        const size_t at = (size_t)b * N + meeting_point(0, L - 1);
        const float *ua = mv.ua + at * T, *ub = mv.ub + at * T;
        float m = LCCRF_NEG_INF;
        for (int t = lane; t < T; t += 64) m = fmaxf(m, ua[t] + ub[t]);
        m = xor_max<1, 64>(m);
        float S = 0.f;
        for (int t = lane; t < T; t += 64) S += ex2(ua[t] + ub[t] - finite_or_zero(m));
        S = xor_sum<1, 64>(S);
        if (lane == 0) lz = ((double)(m + lg2(S)) + mv.Oa[at] + mv.Ob[at]) * kLn2;
    }
    for (int i = tid; i < L; i += kPathThreads) {
        const int t = y[i], s = i > 0 ? y[i - 1] : 0;
        if (t < 0 || t >= T || s < 0 || s >= T) { bad = true; continue; }
        acc += (double)Elem<TIN>::get(phib + (size_t)i * T * T + (size_t)s * T + t);
    }
    acc += lane_xor<1>(acc);
    acc += lane_xor<2>(acc);
    acc += lane_xor<4>(acc);
    acc += lane_xor<8>(acc);
    acc += lane_xor<16>(acc);
    acc += lane_xor<32>(acc);
    const bool wave_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
    if (lane == 0) {
        part[wave] = acc;
        part_bad[wave] = wave_bad ? 1 : 0;
    }
    __syncthreads();
    if (tid == 0) {
        double total = 0.0;
        int any_bad = 0;
        for (int w = 0; w < kPathThreads / 64; ++w) {
            total += part[w];
            any_bad |= part_bad[w];
        }
        out[b] = any_bad ? __builtin_nanf("") : (float)(total - (logZ64 ? logZ64[b] : L > 0 ? lz : 0.0));
    }
}

hipError_t launch_path_log_prob(int dtype, const void* phi, const int32_t* lengths, const int32_t* tags, int B, int N,
                                int T, const double* logZ64, const MeetingVectors& mv, float* out, hipStream_t st) {
    if (dtype == 0)
        hipLaunchKernelGGL(path_log_prob_kernel<float>, dim3(B), dim3(kPathThreads), 0, st, static_cast<const float*>(phi), lengths,
                           tags, N, T, logZ64, mv, out);
    else
        hipLaunchKernelGGL(path_log_prob_kernel<uint16_t>, dim3(B), dim3(kPathThreads), 0, st, static_cast<const uint16_t*>(phi),
                           lengths, tags, N, T, logZ64, mv, out);
    return hipGetLastError();
}

// Entropy from what the two half chains leave at the meeting position h.  With the Markov
// property p(y) = p(y_h) p(y_<h | y_h) p(y_>h | y_h), so
//     H = H(y_h) + sum_t p(y_h = t) [ H(y_<h | y_h = t) + H(y_>h | y_h = t) ],
// the two conditional entropies being what the chains carried along (ha, hb, base 2) and
// p(y_h = t) the softmax of alpha_h + beta_h.  One wave per sequence.  No finite path: NaN.
__global__ __launch_bounds__(64) void entropy_combine_kernel(ChainArgs a, float* __restrict__ H) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int N = a.N, T = a.T;
    const int L = clamp_length(a.lengths, b, N);
    if (L == 0) {
        if (lane == 0) H[b] = 0.f;
        return;
    }
    const int h = meeting_point(0, L - 1);
    const size_t vb = (size_t)b * N;
    const float* ua = a.ua + (vb + h) * T;
    const float* ub = a.ub + (vb + h) * T;
    float m = LCCRF_NEG_INF;
    for (int t = lane; t < T; t += 64) m = fmaxf(m, ua[t] + ub[t]);
    m = xor_max<1, 64>(m);
    if (m == LCCRF_NEG_INF) {
        if (lane == 0) H[b] = __builtin_nanf("");
        return;
    }
    float S = 0.f;
    for (int t = lane; t < T; t += 64) S += ex2(ua[t] + ub[t] - m);
    S = xor_sum<1, 64>(S);
    const float lS = lg2(S);
    float acc = 0.f;
    for (int t = lane; t < T; t += 64) {
        const float z = ua[t] + ub[t] - m;  // log2 of p(y_h = t) S
        const float p = ex2(z) / S;
        if (p > 0.f) acc += p * (a.ha[(size_t)b * T + t] + a.hb[(size_t)b * T + t] - (z - lS));
    }
    acc = xor_sum<1, 64>(acc);
    if (lane == 0) H[b] = (float)(((double)acc + (a.hoff ? a.hoff[2 * b] + a.hoff[2 * b + 1] : 0.0)) * kLn2);
}

static hipError_t launch_entropy_combine(const ChainArgs& a, float* H, hipStream_t st) {
    hipLaunchKernelGGL(entropy_combine_kernel, dim3(a.B), dim3(64), 0, st, a, H);
    return hipGetLastError();
}


// ---------------------------------------------------------------------------------------
// Expectations carried along the half chains: entropy first pass for T > 32 (the one-wave
// kernels carry it themselves for T <= 32), and the expected score difference behind the
// cross-entropy and the Kullback-Leibler divergence of two chains (any T).
//
// The same two half chains as chain_half_kernel, each carrying besides its normalised vector a
// second vector h: the conditional expectation, given the current tag, of a quantity summed over
// the path behind it.  With q(s|t) = 2^(ua(s) + phi2(s,t)) / S(t) on the forward chain
// (q(t|s) = 2^(phi2(s,t) + ub(t)) / S(s) on the backward chain):
//     MODE 0, entropy (base 2):   h_i(t) = sum_s q(s|t) [h_{i-1}(s) - log2 q(s|t)],
//                                 evaluated as U / S + log2 S with U = sum e (h - log2 e);
//     MODE 1, cross-entropy:      h_i(t) = sum_s q(s|t) [h_{i-1}(s) + psi_i(s,t)],
//     MODE 2, KL divergence:      h_i(t) = sum_s q(s|t) [h_{i-1}(s) + phi_i(s,t) - psi_i(s,t)],
// psi being the potentials of the second chain (natural units), read beside phi; an edge of
// weight zero contributes nothing whatever psi holds there.  In modes 1 and 2 a common shift of
// h (its largest finite entry) moves into a double-precision offset at every step, so the vector
// stays small however long the chain is.
// At 33 .. 64 tags the steps of lccrf_expect.h come first, these ones follow where they give up.  At 33 .. 128 tags
// every mode first tries every step with one shift for the whole matrix, the normaliser of the vector it
// starts from, as the chain kernels do (lccrf_chain.hip): U / S (+ log2 S) does not depend
// on the shift as long as no term that matters is flushed, which holds if every sum lies in
// [2^-60, 2^60]; otherwise the step is replayed exactly on the same registers.  The other geometries take
// plain exact steps (every sum against its own maximum): the forward step takes the column maxima
// through LDS first, then the sums.
template <typename G>
struct EntropySmem {
    alignas(16) float pmax[G::WAVES][G::TCAP];
    alignas(16) float psum[G::WAVES][G::TCAP];
    alignas(16) float pU[G::WAVES][G::TCAP];
    alignas(16) float rvec[2][G::TCAP];
    alignas(16) float hvec[2][G::TCAP];
    alignas(16) float wmax[2][16];
    int bad[4];  // "speculative step n rejected", indexed by n & 3
};

template <typename TIN, bool ALIGNED>
__device__ __forceinline__ void load_row4(const TIN* __restrict__ mat, int T, int c4, int s, float (&o)[4]) {
    const TIN* row = mat + (size_t)(s < T ? s : T - 1) * T;
    if (ALIGNED) {
        Elem<TIN>::get4(row + (c4 < T ? c4 : T - 4), o);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = Elem<TIN>::get(row + (c4 + j < T ? c4 + j : T - 1));
    }
}

__device__ __forceinline__ float expectation_of(float U, float S) { return S > 0.f ? U / S : 0.f; }

// PLAIN: the chain alone, no expectation (the chains of the second sequence potentials, see entropy_half_kernel); `row` says
// in which row of ua / ub / Oa / Ob its vector of the meeting position goes.
// The first `from` steps are taken already: rv, hv are thread tid's entries of the vectors behind them, O and Hoff their offsets.
template <typename G, typename TIN, bool ALIGNED, int MODE, bool PLAIN>
__device__ __forceinline__ void expect_half(EntropySmem<G>& sm, const ChainArgs& a, int v, const void* phi, const void* psi, int row, int from,
                                            float rv, float hv, double O, double Hoff) {
    constexpr int ITEMS = G::ITEMS, PF = 2;
    constexpr bool CROSS = MODE != 0 && !PLAIN;
    // the second tile travels through a ring of its own where registers allow (QRING); the
    // sixteen-wave geometries have 128 registers a thread: there its rows are fetched where they
    // are used
    constexpr bool LATE_PSI = CROSS && G::WAVES >= 16;
    constexpr bool QRING = CROSS && !LATE_PSI;
    constexpr int QITEMS = QRING ? ITEMS : 1, QPF = QRING ? PF : 1;
    constexpr bool SPEC = (ITEMS == 2 || ITEMS == 4 || ITEMS == 8) && G::LPR >= 16;  // speculative step first
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = v >> 1, dir = v & 1;
    const int N = a.N, T = a.T;
    const int L = clamp_length(a.lengths, b, N);
    if (L == 0) return;
    const int e = L - 1, h = meeting_point(0, e);
    const int c4 = 4 * (tid % G::LPR), r0 = tid / G::LPR;
    const size_t TT = (size_t)T * T, vb = (size_t)b * N;
    const TIN* phib = static_cast<const TIN*>(phi) + (size_t)b * N * TT;
    const TIN* psib = CROSS ? static_cast<const TIN*>(psi) + (size_t)b * N * TT : phib;

    for (int k = tid; k < 2 * G::TCAP; k += G::W) {
        (&sm.rvec[0][0])[k] = LCCRF_NEG_INF;
        (&sm.hvec[0][0])[k] = 0.f;
    }
    if (tid < 32) (&sm.wmax[0][0])[tid] = LCCRF_NEG_INF;
    if (tid < 4) sm.bad[tid] = 0;
    int nstep = 0;
    __syncthreads();
    if (tid < T) {
        sm.rvec[0][tid] = rv;
        sm.hvec[0][tid] = hv;
    }
    __syncthreads();

    float ring[PF][ITEMS][4];
    float qring[QPF][QITEMS][4];
    auto load = [&](int i, int slot) {
        load_tile<G, TIN, ALIGNED>(phib + (size_t)i * TT, T, c4, r0, ring[slot], b != a.B - 1 || i != N - 1);
        if constexpr (QRING) load_tile<G, TIN, ALIGNED>(psib + (size_t)i * TT, T, c4, r0, qring[slot], b != a.B - 1 || i != N - 1);
    };
    // what an edge adds to the carried expectation (modes 1 and 2)
    auto edge_term = [&](int i, int slot, int k, const float (&x)[4], float (&f)[4]) {
        float qv[4];
        if constexpr (LATE_PSI) {
            load_row4<TIN, ALIGNED>(psib + (size_t)i * TT, T, c4, r0 + k * G::RPP, qv);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) qv[j] = qring[QRING ? slot : 0][QRING ? k : 0][j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = MODE == 1 ? qv[j] : x[j] - qv[j];
    };
    int buf = 0;
    auto shift = [&]() {  // normaliser of the vector in rvec[buf]: its maximum, by every thread
        float d = LCCRF_NEG_INF;
        for (int t = lane; t < T; t += 64) d = fmaxf(d, sm.rvec[buf][t]);
        return finite_or_zero(xor_max<1, 64>(d));
    };
    auto hshift = [&]() {  // largest finite entry of hvec[buf] (0 if there is none), by every thread
        float d = LCCRF_NEG_INF;
        for (int t = lane; t < T; t += 64) {
            const float g = sm.hvec[buf][t];
            if (fabsf(g) < __builtin_huge_valf()) d = fmaxf(d, g);
        }
        return finite_or_zero(xor_max<1, 64>(d));
    };

    if (dir == 0) {
        walk<PF>(1 + from, h, +1, load, [&](int i, int slot) {
            float (&x)[ITEMS][4] = ring[slot];
            settle_tile<G, ALIGNED>(x, T, c4);
            if constexpr (QRING) settle_tile<G, ALIGNED>(qring[slot], T, c4);
            const float d = shift();
            O += (double)d;
            float c = 0.f;
            if (CROSS) {
                c = hshift();
                Hoff += (double)c;
            }
            float ua[ITEMS], hin[ITEMS], lm[4] = {LCCRF_NEG_INF, LCCRF_NEG_INF, LCCRF_NEG_INF, LCCRF_NEG_INF};
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int s = r0 + k * G::RPP;
                ua[k] = (s < T) ? sm.rvec[buf][s] - d : LCCRF_NEG_INF;
                hin[k] = (s < T) ? sm.hvec[buf][s] - c : 0.f;
            }
            if constexpr (SPEC) {
                // one shift for the whole matrix: the normaliser d predicts this step's growth
                const int flag = nstep & 3;
                if (tid == 0) sm.bad[(nstep + 1) & 3] = 0;
                float ls[4] = {0.f, 0.f, 0.f, 0.f}, lu[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < ITEMS; ++k) {
                    const float uac = ua[k] - d;
                    float f[4] = {0.f, 0.f, 0.f, 0.f};
                    if constexpr (CROSS) edge_term(i, slot, k, x[k], f);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float arg = __builtin_fmaf(x[k][j], kLog2e, uac);
                        const float ex = ex2(arg);
                        ls[j] += ex;
                        if (CROSS) lu[j] += ex > 0.f ? ex * (hin[k] + f[j]) : 0.f;
                        else if (!PLAIN) lu[j] = __builtin_fmaf(ex, hin[k] - log2_term(arg), lu[j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    ls[j] = xor_sum<G::LPR, 64>(ls[j]);
                    if (!PLAIN) lu[j] = xor_sum<G::LPR, 64>(lu[j]);
                }
                if (lane < G::LPR) {
                    *reinterpret_cast<float4*>(&sm.psum[wave][c4]) = make_float4(ls[0], ls[1], ls[2], ls[3]);
                    if (!PLAIN) *reinterpret_cast<float4*>(&sm.pU[wave][c4]) = make_float4(lu[0], lu[1], lu[2], lu[3]);
                }
                __syncthreads();
                if (wave < G::COLWAVES) {
                    bool good = true;
                    if (tid < T) {
                        float S = 0.f, U = 0.f;
#pragma unroll
                        for (int w = 0; w < G::WAVES; ++w) {
                            S += sm.psum[w][tid];
                            if (!PLAIN) U += sm.pU[w][tid];
                        }
                        good = sum_in_range(S);
                        sm.rvec[buf ^ 1][tid] = d + lg2(S);
                        if (!PLAIN) sm.hvec[buf ^ 1][tid] = CROSS ? expectation_of(U, S) : entropy_of(U, S);
                    }
                    if (!__all(good) && lane == 0) sm.bad[flag] = 1;
                }
                __syncthreads();
                ++nstep;
                if (sm.bad[flag] == 0) {
                    buf ^= 1;
                    return;
                }
                __syncthreads();  // nobody still reads the flag or the rejected vectors
            }
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float xs = __builtin_fmaf(x[k][j], kLog2e, ua[k]);
                    if (!CROSS) x[k][j] = xs;  // the raw potential is needed again in mode 2
                    lm[j] = fmaxf(lm[j], xs);
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) lm[j] = xor_max<G::LPR, 64>(lm[j]);
            if (lane < G::LPR) *reinterpret_cast<float4*>(&sm.pmax[wave][c4]) = make_float4(lm[0], lm[1], lm[2], lm[3]);
            __syncthreads();
            float M[4], ls[4] = {0.f, 0.f, 0.f, 0.f}, lu[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                M[j] = LCCRF_NEG_INF;
#pragma unroll
                for (int w = 0; w < G::WAVES; ++w) M[j] = fmaxf(M[j], sm.pmax[w][c4 + j]);
                M[j] = finite_or_zero(M[j]);
            }
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                float f[4] = {0.f, 0.f, 0.f, 0.f};
                if constexpr (CROSS) edge_term(i, slot, k, x[k], f);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float arg = (CROSS ? __builtin_fmaf(x[k][j], kLog2e, ua[k]) : x[k][j]) - M[j];
                    const float ex = ex2(arg);
                    ls[j] += ex;
                    if (CROSS) lu[j] += ex > 0.f ? ex * (hin[k] + f[j]) : 0.f;
                    else if (!PLAIN) lu[j] = __builtin_fmaf(ex, hin[k] - log2_term(arg), lu[j]);
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ls[j] = xor_sum<G::LPR, 64>(ls[j]);
                if (!PLAIN) lu[j] = xor_sum<G::LPR, 64>(lu[j]);
            }
            if (lane < G::LPR) {
                *reinterpret_cast<float4*>(&sm.psum[wave][c4]) = make_float4(ls[0], ls[1], ls[2], ls[3]);
                if (!PLAIN) *reinterpret_cast<float4*>(&sm.pU[wave][c4]) = make_float4(lu[0], lu[1], lu[2], lu[3]);
            }
            __syncthreads();
            if (tid < T) {
                float S = 0.f, U = 0.f, Mt = LCCRF_NEG_INF;
#pragma unroll
                for (int w = 0; w < G::WAVES; ++w) {
                    S += sm.psum[w][tid];
                    if (!PLAIN) U += sm.pU[w][tid];
                    Mt = fmaxf(Mt, sm.pmax[w][tid]);
                }
                sm.rvec[buf ^ 1][tid] = Mt + lg2(S);  // Mt = -inf gives S = 0: -inf
                if (!PLAIN) sm.hvec[buf ^ 1][tid] = CROSS ? expectation_of(U, S) : entropy_of(U, S);
            }
            __syncthreads();
            buf ^= 1;
        });
    } else {
        walk<PF>(e - from, h + 1, -1, load, [&](int i, int slot) {
            float (&y)[ITEMS][4] = ring[slot];
            settle_tile<G, ALIGNED>(y, T, c4);
            if constexpr (QRING) settle_tile<G, ALIGNED>(qring[slot], T, c4);
            const float d = shift();
            O += (double)d;
            float c = 0.f;
            if (CROSS) {
                c = hshift();
                Hoff += (double)c;
            }
            float ub[4], hin[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ub[j] = (c4 + j < T) ? sm.rvec[buf][c4 + j] - d : LCCRF_NEG_INF;
                hin[j] = (c4 + j < T) ? sm.hvec[buf][c4 + j] - c : 0.f;
            }
            if constexpr (SPEC) {
                const int flag = nstep & 3;
                if (tid == 0) sm.bad[(nstep + 1) & 3] = 0;
                float Sl[ITEMS < 4 ? 4 : ITEMS] = {}, Ul[ITEMS < 4 ? 4 : ITEMS] = {};
#pragma unroll
                for (int k = 0; k < ITEMS; ++k) {
                    float f[4] = {0.f, 0.f, 0.f, 0.f};
                    if constexpr (CROSS) edge_term(i, slot, k, y[k], f);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float arg = __builtin_fmaf(y[k][j], kLog2e, ub[j] - d);
                        const float ex = ex2(arg);
                        Sl[k] += ex;
                        if (CROSS) Ul[k] += ex > 0.f ? ex * (hin[j] + f[j]) : 0.f;
                        else if (!PLAIN) Ul[k] = __builtin_fmaf(ex, hin[j] - log2_term(arg), Ul[k]);
                    }
                }
                // four rows at a time: each lane ends up with the complete sums of one of them
                const int kk = 2 * (lane & 1) + ((lane >> 1) & 1);
                bool good = true;
#pragma unroll
                for (int k0 = 0; k0 < ITEMS; k0 += 4) {
                    const float S = reduce4_over_lanes<G::LPR>(Sl[k0], Sl[k0 + 1], Sl[k0 + 2], Sl[k0 + 3], lane);
                    const float U = PLAIN ? 0.f : reduce4_over_lanes<G::LPR>(Ul[k0], Ul[k0 + 1], Ul[k0 + 2], Ul[k0 + 3], lane);
                    const int s = r0 + (k0 + kk) * G::RPP;
                    if ((tid % G::LPR) < 4 && s < T) {
                        sm.rvec[buf ^ 1][s] = d + lg2(S);
                        if (!PLAIN) sm.hvec[buf ^ 1][s] = CROSS ? expectation_of(U, S) : entropy_of(U, S);
                    }
                    good = good && (s >= T || sum_in_range(S));
                }
                if (!__all(good) && lane == 0) sm.bad[flag] = 1;
                __syncthreads();
                ++nstep;
                if (sm.bad[flag] == 0) {
                    buf ^= 1;
                    return;
                }
                __syncthreads();  // nobody still reads the flag or the rejected vectors
            }
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                float f[4] = {0.f, 0.f, 0.f, 0.f};
                if constexpr (CROSS) edge_term(i, slot, k, y[k], f);
#pragma unroll
                for (int j = 0; j < 4; ++j) y[k][j] = __builtin_fmaf(y[k][j], kLog2e, ub[j]);
                const float m = xor_max<1, G::LPR>(fmaxf(fmaxf(y[k][0], y[k][1]), fmaxf(y[k][2], y[k][3])));
                const float g = finite_or_zero(m);
                float Sl = 0.f, Ul = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float arg = y[k][j] - g;
                    const float ex = ex2(arg);
                    Sl += ex;
                    if (CROSS) Ul += ex > 0.f ? ex * (hin[j] + f[j]) : 0.f;
                    else if (!PLAIN) Ul = __builtin_fmaf(ex, hin[j] - log2_term(arg), Ul);
                }
                const float S = xor_sum<1, G::LPR>(Sl), U = PLAIN ? 0.f : xor_sum<1, G::LPR>(Ul);
                const int s = r0 + k * G::RPP;
                if (c4 == 0 && s < T) {
                    sm.rvec[buf ^ 1][s] = m + lg2(S);
                    if (!PLAIN) sm.hvec[buf ^ 1][s] = CROSS ? expectation_of(U, S) : entropy_of(U, S);
                }
            }
            __syncthreads();
            buf ^= 1;
        });
    }
    // the vectors of the meeting position
    const float d = shift();
    O += (double)d;
    if (tid < T) {
        (dir == 0 ? a.ua : a.ub)[(vb + row) * T + tid] = sm.rvec[buf][tid] - d;
        if (!PLAIN) (dir == 0 ? a.ha : a.hb)[(size_t)b * T + tid] = sm.hvec[buf][tid];
    }
    if (tid == 0) (dir == 0 ? a.Oa : a.Ob)[vb + row] = O;
    if (!PLAIN && a.hoff && tid == 0) a.hoff[2 * b + dir] = Hoff;
}

// The row of ua / ub / Oa / Ob that the chains of psi leave their vectors of the meeting position h in (N >= 2): not h, which
// holds those of phi.
__device__ __forceinline__ int psi_row(int h) { return h > 0 ? h - 1 : 1; }

// Where a chain starts: tag t's entry of its vector (base-2 logarithm), and of the expectation of the scores (MODE 0: of phi, base
// 2), the score of the first tag belonging to the forward chain.
template <int MODE, bool PLAIN, typename TIN>
__device__ __forceinline__ void expect_start(const TIN* phib, const TIN* psib, int dir, int t, float& rv, float& hv) {
    rv = hv = 0.f;
    if (dir != 0) return;
    const float p0 = Elem<TIN>::get(phib + t);
    rv = p0 * kLog2e;
    if (PLAIN || p0 == LCCRF_NEG_INF) return;
    if (MODE == 0) {
        hv = rv;
        return;
    }
    const float q0 = Elem<TIN>::get(psib + t);
    hv = MODE == 2 ? p0 - q0 : q0;
}

template <typename G, typename TIN, bool ALIGNED, int MODE, bool PLAIN>
__device__ __forceinline__ void expect_chain(EntropySmem<G>& sm, const ChainArgs& a, int v, const void* phi, const void* psi, int row) {
    const size_t at = (size_t)(v >> 1) * a.N * a.T * a.T;
    float rv = LCCRF_NEG_INF, hv = 0.f;
    if ((int)threadIdx.x < a.T && a.N > 0)
        expect_start<MODE, PLAIN>(static_cast<const TIN*>(phi) + at, static_cast<const TIN*>(psi) + at, v & 1, (int)threadIdx.x, rv, hv);
    if (MODE == 0) hv = 0.f;  // (these steps carry the entropy itself)
    expect_half<G, TIN, ALIGNED, MODE, PLAIN>(sm, a, v, phi, psi, row, 0, rv, hv, 0.0, 0.0);
}
// Workgroups 0 .. 2 B - 1: the half chains of phi with their expectations.  With a.psi_chains (cross-entropy and divergence),
// workgroups 2 B .. 4 B - 1 run the plain half chains of psi beside them, for its log-partition: as launches one after the
// other either leaves half of the chip idle (B=64, N=256, 64 tags, log-domain steps: 96 + 172 us, together 176).
template <typename G, typename TIN, bool ALIGNED, int MODE>
__global__ __launch_bounds__(G::W) void entropy_half_kernel(ChainArgs a) {
    __shared__ EntropySmem<G> sm;
    const int v = blockIdx.x;
    if (MODE == 0 || v < 2 * a.B) {
        const int L = clamp_length(a.lengths, v >> 1, a.N);
        expect_chain<G, TIN, ALIGNED, MODE, false>(sm, a, v, a.phi, a.psi, meeting_point(0, L - 1));
    } else if constexpr (MODE != 0) {
        const int L = clamp_length(a.lengths, (v - 2 * a.B) >> 1, a.N);
        expect_chain<G, TIN, ALIGNED, MODE, true>(sm, a, v - 2 * a.B, a.psi, nullptr, psi_row(meeting_point(0, L - 1)));
    }
}

// The same at 33 .. 64 tags: the steps of lccrf_expect.h as long as they are accepted, then those of expect_half.
template <int WAVES>
using ExpectGeo = Geo<16, WAVES, 16 / WAVES>;
template <int WAVES, int ITEMS, typename TIN, bool ALIGNED, int MODE, bool PLAIN>
__device__ __forceinline__ void expect_linear_chain(EntropySmem<ExpectGeo<WAVES>>& sm, ExpectSmem<WAVES>& lin, const ChainArgs& a, int v, const void* phi,
                                                    const void* psi, int row, int h, int e) {
    constexpr int RUN = PLAIN ? kExpectPlain : MODE;
    const int lane = threadIdx.x & 63, b = v >> 1, dir = v & 1, T = a.T;
    const size_t vb = (size_t)b * a.N, at = vb * T * T;
    const TIN *phib = static_cast<const TIN*>(phi) + at, *psib = RUN == 1 || RUN == 2 ? static_cast<const TIN*>(psi) + at : phib;
    const int n = dir == 0 ? h : e - h;
    ExpectState st{LCCRF_NEG_INF, 0.f, 0.0, 0.0};
    if (lane < T) expect_start<MODE, PLAIN>(phib, psib, dir, lane, st.v, st.h);
    // A tag that is forbidden everywhere is an exact zero in every vector, which no scaled step accepts: the first tag that the sequence
    // cannot start with is looked up in the chain's first matrix (B=512 N=64 T=64 with such a tag: 159 -> 150 us).
    bool hopeless = false;
    const unsigned long long suspects = __ballot(lane < T && (dir == 0 ? st.v : Elem<TIN>::get(phib + lane)) == LCCRF_NEG_INF);
    if (suspects != 0 && n > 0) {
        const int t = __builtin_ctzll(suspects);
        const TIN* mat = phib + (size_t)(dir == 0 ? 1 : e) * T * T;
        hopeless = __ballot(lane < T && st.v != LCCRF_NEG_INF && Elem<TIN>::get(mat + (dir == 0 ? lane * T + t : t * T + lane)) != LCCRF_NEG_INF) == 0;
    }
    const int done = hopeless ? 0
                     : dir == 0 ? expect_run<WAVES, ITEMS, TIN, ALIGNED, false, RUN>(lin, phib, psib, T, 1, n, st)
                                : expect_run<WAVES, ITEMS, TIN, ALIGNED, true, RUN>(lin, phib, psib, T, e, n, st);
    // Entropy of what lies behind a tag: log alpha less the expected score, base 2
    float hv = st.h;
    double Hoff = st.Hoff;
    if (RUN == 0) {
        hv = st.v > LCCRF_NEG_INF ? st.v - st.h : 0.f;
        Hoff = st.O - st.Hoff;
    }
    if (done < n) {
        if (RUN == 0) {
            hv = st.v > LCCRF_NEG_INF ? (float)((double)hv + Hoff) : 0.f;
            Hoff = 0.0;
        }
        expect_half<ExpectGeo<WAVES>, TIN, ALIGNED, MODE, PLAIN>(sm, a, v, phi, psi, row, done, st.v, hv, st.O, Hoff);
        return;
    }
    if ((int)threadIdx.x < T) {
        (dir == 0 ? a.ua : a.ub)[(vb + row) * T + lane] = st.v;
        if (!PLAIN) (dir == 0 ? a.ha : a.hb)[(size_t)b * T + lane] = hv;
    }
    if (threadIdx.x == 0) {
        (dir == 0 ? a.Oa : a.Ob)[vb + row] = st.O;
        if (!PLAIN) a.hoff[2 * b + dir] = Hoff;
    }
}
// (Three waves a SIMD: two potentials an edge off the 16-byte grid take 169 registers, and with one less a third workgroup has room:
// divergence B=300 N=64 T=57 125 -> 121 us.)
template <int WAVES, int ITEMS, typename TIN, bool ALIGNED, int MODE>
__global__ __launch_bounds__(64 * WAVES, 3) void expect_linear_kernel(ChainArgs a) {
    __shared__ EntropySmem<ExpectGeo<WAVES>> sm;
    __shared__ ExpectSmem<WAVES> lin;
    const bool plain = MODE != 0 && (int)blockIdx.x >= 2 * a.B;
    const int v = (int)blockIdx.x - (plain ? 2 * a.B : 0);
    const int L = clamp_length(a.lengths, v >> 1, a.N);
    if (L == 0) return;
    const int e = L - 1, h = meeting_point(0, e);
    if (MODE == 0 || !plain) expect_linear_chain<WAVES, ITEMS, TIN, ALIGNED, MODE, false>(sm, lin, a, v, a.phi, a.psi, h, h, e);
    else if constexpr (MODE != 0) expect_linear_chain<WAVES, ITEMS, TIN, ALIGNED, MODE, true>(sm, lin, a, v, a.psi, nullptr, psi_row(h), h, e);
}

template <typename TIN, bool ALIGNED, int MODE>
static hipError_t launch_entropy_T(const ChainArgs& a, hipStream_t st) {
    const dim3 grid((a.psi_chains ? 4 : 2) * a.B);
    if (a.T <= 16)
        hipLaunchKernelGGL((entropy_half_kernel<Geo<4, 1, 1>, TIN, ALIGNED, MODE>), grid, dim3(64), 0, st, a);
    else if (a.T <= 32)
        hipLaunchKernelGGL((entropy_half_kernel<Geo<8, 4, 1>, TIN, ALIGNED, MODE>), grid, dim3(256), 0, st, a);
    else if (a.T <= 48)
        hipLaunchKernelGGL((expect_linear_kernel<4, 3, TIN, ALIGNED, MODE>), grid, dim3(256), 0, st, a);
    else if (a.T <= 64) {
        // Eight waves where every workgroup has a compute unit to itself and an edge takes two potentials: the matrices are then most of
        // a step (divergence, us, eight waves / four: B=64 N=256 T=64 110 / 121, B=64 N=200 T=57 bfloat16 89 / 106, B=32 N=64 T=64
        // 34 / 37; B=128 N=64 T=64 60 / 49).  With fewer tags or one potential an edge it is the instructions that every wave
        // executes alike (divergence B=16 N=100 T=40 47 / 45; entropy B=64 N=128 T=64 55 / 49, B=128 N=128 T=48 56 / 45).
        if constexpr (MODE != 0) {
            if (grid.x <= 256) {
                hipLaunchKernelGGL((expect_linear_kernel<8, 2, TIN, ALIGNED, MODE>), grid, dim3(512), 0, st, a);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((expect_linear_kernel<4, 4, TIN, ALIGNED, MODE>), grid, dim3(256), 0, st, a);
    }
    else if (a.T <= 128) {
        if constexpr (MODE == 0)
            hipLaunchKernelGGL((entropy_half_kernel<Geo<32, 16, 4>, TIN, ALIGNED, MODE>), grid, dim3(1024), 0, st, a);
        else  // two tiles in flight: eight waves, so that a thread has the registers for both rings
            hipLaunchKernelGGL((entropy_half_kernel<Geo<32, 8, 8>, TIN, ALIGNED, MODE>), grid, dim3(512), 0, st, a);
    } else
        return hipErrorInvalidValue;  // larger tag sets take the row-batch kernel (launch_stream_expect)
    return hipGetLastError();
}
template <int MODE>
static hipError_t launch_entropy_mode(int dtype, const ChainArgs& a, hipStream_t st) {
    if (stream_supported(a.T)) return launch_stream_expect(MODE, dtype, a, st);
    const bool aligned = (a.T % 4) == 0;
    if (dtype == 0) return aligned ? launch_entropy_T<float, true, MODE>(a, st) : launch_entropy_T<float, false, MODE>(a, st);
    return aligned ? launch_entropy_T<uint16_t, true, MODE>(a, st) : launch_entropy_T<uint16_t, false, MODE>(a, st);
}

// H(p) [B] for every sequence: first pass in entropy mode, then the combination at the meeting point.
hipError_t launch_entropy(int dtype, const void* phi, const int32_t* lengths, int B, int N, int T, float* ua, float* ub,
                          double* Oa, double* Ob, float* ha, float* hb, double* hoff, float* H, hipStream_t st) {
    ChainArgs a{phi, lengths, B, N, T, ua, ub, Oa, Ob, nullptr, nullptr, 0, nullptr, 0, 1, nullptr, nullptr, nullptr, nullptr};
    a.ha = ha;
    a.hb = hb;
    if (T > 32 && T <= 64) a.hoff = hoff;  // (the other kernels keep the whole of it in ha / hb)
    const hipError_t e = wave_supported(T) ? launch_wave_pass(false, dtype, a, st) : launch_entropy_mode<0>(dtype, a, st);
    if (e != hipSuccess) return e;
    return launch_entropy_combine(a, H, st);
}

// Entropy from the per-wave sums of conditional edge entropies the second pass leaves in entropy
// mode (chunked schedule): H = ln 2 * sum over the chunks of the sequence, both directions.  One
// wave per sequence.  logZ: what the run has found for log Z ([B] floats): -inf means no finite
// path, the entropy is NaN then.
__global__ __launch_bounds__(64) void entropy_reduce_kernel(const float* __restrict__ ent, const int32_t* __restrict__ lengths,
                                                            const float* __restrict__ logZ, int N, int chunk, int C,
                                                            float* __restrict__ H) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int L = clamp_length(lengths, b, N);
    if (L == 0) {
        if (lane == 0) H[b] = 0.f;
        return;
    }
    const int Cb = (L + chunk - 1) / chunk;
    double acc = 0.0;
    for (int k = lane; k < 2 * Cb; k += 64) acc += (double)ent[2 * (size_t)b * C + k];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) H[b] = logZ[b] == LCCRF_NEG_INF ? __builtin_nanf("") : (float)(acc * kLn2);
}

hipError_t launch_entropy_reduce(const float* ent, const int32_t* lengths, const float* logZ, int B, int N, int chunk,
                                 float* H, hipStream_t st) {
    const int C = (N + chunk - 1) / chunk;
    hipLaunchKernelGGL(entropy_reduce_kernel, dim3(B), dim3(64), 0, st, ent, lengths, logZ, N, chunk, C, H);
    return hipGetLastError();
}

// The same sum over the chunks for the expectations of a second chain's potentials (natural units):
// cross-entropy logZq - E, or with kl the divergence logZq - logZp - E for E the expectation of the
// difference of the potentials.  No finite path under the chain itself (logZp = -inf): NaN.
__global__ __launch_bounds__(64) void cross_reduce_kernel(const float* __restrict__ ent, const int32_t* __restrict__ lengths,
                                                          const double* __restrict__ logZq, const double* __restrict__ logZp,
                                                          int N, int chunk, int C, int kl, float* __restrict__ out) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int L = clamp_length(lengths, b, N);
    if (L == 0) {
        if (lane == 0) out[b] = 0.f;
        return;
    }
    const int Cb = (L + chunk - 1) / chunk;
    double acc = 0.0;
    for (int k = lane; k < 2 * Cb; k += 64) acc += (double)ent[2 * (size_t)b * C + k];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) {
        const double lzp = logZp[b];
        out[b] = lzp == -__builtin_huge_val() ? __builtin_nanf("") : (float)(logZq[b] - (kl ? lzp : 0.0) - acc);
    }
}

hipError_t launch_cross_reduce(bool kl, const float* ent, const int32_t* lengths, const double* logZq, const double* logZp,
                               int B, int N, int chunk, float* out, hipStream_t st) {
    const int C = (N + chunk - 1) / chunk;
    hipLaunchKernelGGL(cross_reduce_kernel, dim3(B), dim3(64), 0, st, ent, lengths, logZq, logZp, N, chunk, C, kl ? 1 : 0, out);
    return hipGetLastError();
}

// Cross-entropy H(p, q) = log Z_q - E_p[score_q(y)] (kl = false) or Kullback-Leibler divergence
// KL(p || q) = E_p[score_p(y) - score_q(y)] - log Z_p + log Z_q (kl = true) of two chains over the
// same sequences: the expectation from the half chains of p at their meeting position (as the
// entropy above), log Z_p from the same vectors, log Z_q handed in (double precision, natural
// logarithm).  No finite path under p: NaN.  One wave per sequence.
__global__ __launch_bounds__(64) void cross_combine_kernel(ChainArgs a, const double* __restrict__ logZq, float* __restrict__ out,
                                                           int kl) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int N = a.N, T = a.T;
    const int L = clamp_length(a.lengths, b, N);
    if (L == 0) {
        if (lane == 0) out[b] = 0.f;
        return;
    }
    const int h = meeting_point(0, L - 1);
    const size_t vb = (size_t)b * N;
    const float* ua = a.ua + (vb + h) * T;
    const float* ub = a.ub + (vb + h) * T;
    float m = LCCRF_NEG_INF;
    for (int t = lane; t < T; t += 64) m = fmaxf(m, ua[t] + ub[t]);
    m = xor_max<1, 64>(m);
    if (m == LCCRF_NEG_INF) {
        if (lane == 0) out[b] = __builtin_nanf("");
        return;
    }
    float S = 0.f;
    for (int t = lane; t < T; t += 64) S += ex2(ua[t] + ub[t] - m);
    S = xor_sum<1, 64>(S);
    float acc = 0.f;
    for (int t = lane; t < T; t += 64) {
        const float p = ex2(ua[t] + ub[t] - m) / S;
        if (p > 0.f) acc += p * (a.ha[(size_t)b * T + t] + a.hb[(size_t)b * T + t]);
    }
    acc = xor_sum<1, 64>(acc);
    double lzq;
    if (a.psi_chains) {  // from the vectors the chains of psi have left
        const size_t r = vb + psi_row(h);
        float mq = LCCRF_NEG_INF;
        for (int t = lane; t < T; t += 64) mq = fmaxf(mq, a.ua[r * T + t] + a.ub[r * T + t]);
        mq = xor_max<1, 64>(mq);
        float Sq = 0.f;
        for (int t = lane; t < T; t += 64) Sq += ex2(a.ua[r * T + t] + a.ub[r * T + t] - finite_or_zero(mq));
        Sq = xor_sum<1, 64>(Sq);
        lzq = ((double)(mq + lg2(Sq)) + a.Oa[r] + a.Ob[r]) * kLn2;
    } else {
        lzq = logZq[b];
    }
    if (lane == 0) {
        const double E = (double)acc + a.hoff[2 * b] + a.hoff[2 * b + 1];
        const double lzp = (a.Oa[vb + h] + a.Ob[vb + h] + (double)m + (double)lg2(S)) * kLn2;
        out[b] = (float)(kl ? E - lzp + lzq : lzq - E);
    }
}

bool cross_runs_both(int N, int T) { return N >= 2 && !stream_supported(T); }

hipError_t launch_cross(bool kl, int dtype, const void* phi_p, const void* phi_q, const int32_t* lengths, int B, int N,
                        int T, float* ua, float* ub, double* Oa, double* Ob, float* ha, float* hb, double* hoff,
                        const double* logZq, float* out, hipStream_t st) {
    ChainArgs a{phi_p, lengths, B, N, T, ua, ub, Oa, Ob, nullptr, nullptr, 0, nullptr, 0, 1, nullptr, nullptr, nullptr, nullptr};
    a.ha = ha;
    a.hb = hb;
    a.hoff = hoff;
    a.psi = phi_q;
    a.psi_chains = logZq ? 0 : 1;
    const hipError_t e = kl ? launch_entropy_mode<2>(dtype, a, st) : launch_entropy_mode<1>(dtype, a, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(cross_combine_kernel, dim3(B), dim3(64), 0, st, a, logZq, out, kl ? 1 : 0);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Backward sweep of forward-filtering backward-sampling (paper, section "Sampling a Structure"):
// y_{L-1} ~ exp(alpha_{L-1}(t)), then y_i ~ exp(alpha_i(s) + phi_{i+1}(s, y_{i+1})) going down.
// The randomness is an input: uniforms[b][i] decides position i by inversion of the cumulative
// weights over ascending tags (the smallest tag whose cumulative weight exceeds u * total; the
// last tag of positive weight if rounding leaves none).
//
// With the uniforms fixed, position i is a MAP from the tag above it to its own tag, and that map
// does not depend on any other position: F_i[t] = the tag drawn for y_i if y_{i+1} = t.  So the
// sweep splits into a pass that is parallel over all positions and reads phi once
// (sample_map_kernel: all T columns of every matrix, T^2 work a position like a forward step) and
// a walk through the table of maps that touches one byte a position (sample_walk_kernel), instead
// of N dependent column gathers from HBM.  The total weight of column t is alpha_{i+1}(t), which
// the forward pass has stored, so one sweep over the rows of a column finds where the running sum
// crosses u (weights relative to that total; it equals the sum up to the rounding of the forward
// step, which matters only for a draw closer than that to the edge of a tag's interval).

// Where the uniforms come from: the caller's array, or (given == null) the counter-based generator
// Philox4x32-10 (Salmon, Moraes, Dror and Shaw, "Parallel random numbers: as easy as 1, 2, 3", 2011) keyed
// by the caller's 64-bit seed: the uniform of position i of sequence b is the first output word of the
// counter (b N + i, 0) under that key, its upper 24 bits times 2^-24.  A draw is a function of (seed, b, i)
// alone, so a call is reproducible whatever the launch shape, and any draw can be regenerated on its own.
struct Uniforms {
    const float* given;
    unsigned long long seed;
    __device__ __forceinline__ float at(size_t idx) const {
        if (given) return given[idx];
        unsigned c0 = (unsigned)(idx & 0xffffffffull), c1 = (unsigned)(idx >> 32), c2 = 0u, c3 = 0u;
        unsigned k0 = (unsigned)(seed & 0xffffffffull), k1 = (unsigned)(seed >> 32);
#pragma unroll
        for (int round = 0; round < 10; ++round) {
            const unsigned hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
            const unsigned hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
            c0 = hi1 ^ c1 ^ k0;
            c1 = lo1;
            c2 = hi0 ^ c3 ^ k1;
            c3 = lo0;
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        return (float)(c0 >> 8) * 0x1p-24f;
    }
};

// LPP lanes serve one position (16, 32 or 64: the tag count rounded up, one column a lane); a wave serves 64 / LPP positions, a
// workgroup four waves.
template <typename TIN, int LPP>
__global__ __launch_bounds__(256) void sample_map_kernel(const TIN* __restrict__ phi, const int32_t* __restrict__ lengths,
                                                         const float* __restrict__ ua, const double* __restrict__ Oa,
                                                         const Uniforms uniforms, int B, int N, int T,
                                                         uint8_t* __restrict__ F) {
    constexpr int PPW = 64 / LPP;
    __shared__ float alds[4][PPW][LPP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int pl = lane / LPP, tl = lane % LPP;
    const long long unit = ((long long)blockIdx.x * 4 + wave) * PPW + pl;  // (b, i), i = 0 .. N-2
    if (unit >= (long long)B * (N - 1)) return;
    const int b = (int)(unit / (N - 1)), i = (int)(unit % (N - 1));
    const int L = clamp_length(lengths, b, N);
    if (i >= L - 1) return;
    const size_t TT = (size_t)T * T, vb = (size_t)b * N;
    const int col = tl < T ? tl : T - 1;
    const TIN* mat = phi + (vb + i + 1) * TT + col;  // phi_{i+1}
    const float dO = (float)(Oa[vb + i] - Oa[vb + i + 1]);
    const float u = uniforms.at(vb + i);
    float base = tl < T ? dO - ua[(vb + i + 1) * T + tl] : LCCRF_NEG_INF;  // an unreachable tag above: +inf, no weight
    if (!(base < __builtin_huge_valf())) base = LCCRF_NEG_INF;
    alds[wave][pl][tl] = tl < T ? ua[(vb + i) * T + tl] : LCCRF_NEG_INF;
    float cum = 0.f;
    int first = -1, last = -1;
    const float* arow = alds[wave][pl];
#pragma unroll 4
    for (int s = 0; s < T; ++s) {
        const float w = ex2(__builtin_fmaf(Elem<TIN>::get(mat + (size_t)s * T), kLog2e, base) + arow[s]);
        cum += w;
        last = w > 0.f ? s : last;
        first = (first < 0 && cum > u) ? s : first;
    }
    const int pick = first >= 0 ? first : (last >= 0 ? last : 0);
    if (tl < T) F[(vb + i) * T + tl] = (uint8_t)pick;
}

// The same maps at 65 .. 256 tags, a workgroup a position.  One wave a position read the rows of its matrix one after the other, two or
// four bytes a lane: what a row takes from memory T / 4 times over, and at most 2.1 TB/s (B=40 N=256 T=200 785 us, a lone sequence of 19 positions
// at 144 tags 60).  Here the whole matrix is requested at once: the rows are cut into G = W / ceil(T / 4) groups of consecutive ones, a thread
// holds four columns of at most R rows and their weights stay in its registers.  The groups' sums of a column meet in LDS, a thread a column finds the
// group in which the running sum passes u, and the thread that holds it finds the row.  (A row's last piece is moved back to end with
// it, T >= 4; what is then held twice has the same sums and the same row.)
template <typename TIN, bool ALIGNED, int W, int R>
__global__ __launch_bounds__(W, 4) void sample_map_wide_kernel(const TIN* __restrict__ phi, const int32_t* __restrict__ lengths,
                                                               const float* __restrict__ ua, const double* __restrict__ Oa,
                                                               const Uniforms uniforms, unsigned from, int N, int T, uint8_t* __restrict__ F) {
    using Raw = RawPiece<TIN>;
    __shared__ __attribute__((aligned(16))) float part[4 * W];  // [group][T]: G T <= 4 W
    __shared__ float av[256], bv[256], before[256];
    __shared__ int where[256];  // the group that holds the row; negative: of none that passes u the last of positive weight (-1 - group)
    __shared__ unsigned char pick[256];
    __shared__ float us;
    const int tid = threadIdx.x;
    const unsigned at = from + blockIdx.x;
    const int b = at / (unsigned)(N - 1), i = at % (unsigned)(N - 1);
    const int L = clamp_length(lengths, b, N);
    if (i >= L - 1) return;
    const size_t TT = (size_t)T * T, vb = (size_t)b * N;
    const int Q4 = (T + 3) >> 2, G = W / Q4, rows = (T + G - 1) / G;  // (rows <= R)
    const int g = tid / Q4, cl = tid - g * Q4, c4 = min(4 * cl, T - 4), row0 = g * rows;
    const GlobalBytes* mat = (const GlobalBytes*)(phi + (vb + i + 1) * TT);  // phi_{i+1}
    typename Raw::type raw[R];
#pragma unroll
    for (int k = 0; k < R; ++k) raw[k] = Raw::template load<ALIGNED>(mat + ((size_t)min(row0 + min(k, rows - 1), T - 1) * T + c4) * sizeof(TIN));
    for (int t = tid; t < T; t += W) {
        const float base = (float)(Oa[vb + i] - Oa[vb + i + 1]) - ua[(vb + i + 1) * T + t];
        bv[t] = base < __builtin_huge_valf() ? base : LCCRF_NEG_INF;  // an unreachable tag above: +inf, no weight
        av[t] = ua[(vb + i) * T + t];
        pick[t] = 0;
    }
    if (tid == 0) us = uniforms.at(vb + i);
    __syncthreads();
    const float u = us;
    float w[R][4], base[4], sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) base[j] = bv[c4 + j];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const bool mine = k < rows && row0 + k < T;
        const float as = mine ? av[min(row0 + k, T - 1)] : LCCRF_NEG_INF;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w[k][j] = ex2(__builtin_fmaf(Raw::get(raw[k], j), kLog2e, base[j]) + as);
            w[k][j] = mine ? w[k][j] : 0.f;
            sum[j] += w[k][j];
        }
    }
    if (g < G) {
#pragma unroll
        for (int j = 0; j < 4; ++j) part[g * T + c4 + j] = sum[j];
    }
    __syncthreads();
    for (int t = tid; t < T; t += W) {
        float cum = 0.f, at = 0.f;
        int found = -1, last = -1;
        for (int q = 0; q < G; ++q) {
            const float p = part[q * T + t], next = cum + p;
            const bool over = found < 0 && next > u;
            if (over || (found < 0 && p > 0.f)) at = cum;
            last = p > 0.f ? q : last;
            found = over ? q : found;
            cum = next;
        }
        before[t] = at;
        where[t] = found >= 0 ? found : -1 - last;  // (no weight at all: 0, nobody's, and tag 0)
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int at = where[c4 + j], group = at >= 0 ? at : -1 - at;
        if (group == g && g < G) {
            float cum = before[c4 + j];
            int first = -1, last = 0;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                cum += w[k][j];
                last = w[k][j] > 0.f ? k : last;
                first = first < 0 && cum > u ? k : first;
            }
            // (a group whose sum passes u may stop short of it row by row, by rounding: its last row of positive weight)
            pick[c4 + j] = (unsigned char)(row0 + (at >= 0 && first >= 0 ? first : last));
        }
    }
    __syncthreads();
    for (int t = tid; t < T; t += W) F[(vb + i) * T + t] = pick[t];
}

constexpr int kWalkWindow = 16384;  // bytes of the table of maps held in LDS at a time

// The tag of the last position: inversion over exp(alpha_{L-1}) by one wave, K tags a lane (lane l owns
// tags l K .. l K + K - 1, so that lane-wise prefix sums keep the tag order).  -1: no finite path.
template <int K>
__device__ __forceinline__ int draw_last_tag(const float* __restrict__ alpha_last, float u, int T, int lane) {
    float w[K], m = LCCRF_NEG_INF;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int s = lane * K + k;
        w[k] = s < T ? alpha_last[s] : LCCRF_NEG_INF;
        m = fmaxf(m, w[k]);
    }
    m = xor_max<1, 64>(m);
    if (m == LCCRF_NEG_INF) return -1;
    float part = 0.f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        w[k] = ex2(w[k] - m);
        part += w[k];
    }
    float incl = part;  // inclusive prefix sum over lanes (ascending lane = ascending tag)
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float v = __shfl_up(incl, off, 64);
        if (lane >= off) incl += v;
    }
    const float target = u * __shfl(incl, 63, 64);
    float cum = incl - part;
    int first_over = 0x7fffffff, last_pos = -1;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int s = lane * K + k;
        cum += w[k];
        if (w[k] > 0.f) last_pos = s;
        if (first_over == 0x7fffffff && cum > target && s < T) first_over = s;
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        first_over = min(first_over, __shfl_xor(first_over, off, 64));
        last_pos = max(last_pos, __shfl_xor(last_pos, off, 64));
    }
    return first_over != 0x7fffffff ? first_over : last_pos;
}

constexpr int kWalkShort = 128;

// The walk through a window of the table, by a workgroup.  Walked tag by tag it is one look-up in LDS behind the other, 60 ns each; so
// the window is cut into stretches, a thread takes a tag that a stretch may be entered on and follows it to the end of the stretch, and
// what is left one behind the other is a look-up a stretch.
template <int THREADS>
struct WalkShared {
    __attribute__((aligned(16))) uint8_t win[kWalkWindow];  // the maps, [position][tag]
    static constexpr int ITEMS = THREADS == 64 ? 4 : 1;  // stretches and tags a thread follows side by side
    static constexpr int ALL = ITEMS * THREADS;          // (T <= 256: at least one stretch)
    __attribute__((aligned(16))) uint8_t passed[kWalkWindow + ALL];  // [step][stretch][tag entered on]: the tag reached by that step
    uint8_t left_on[ALL];      // [stretch][tag entered on]
    uint8_t entered[ALL + 1];  // the tag every stretch is entered on
    int last;
};

// The maps of positions lo .. lo + np - 1 of a sequence (Fb: its rows of the table) into LDS.
template <int THREADS>
__device__ __forceinline__ void load_window(uint8_t* win, const uint8_t* __restrict__ Fb, int lo, int np, int T) {
    const uint8_t* src = Fb + (size_t)lo * T;
    const int nbytes = np * T, tid = threadIdx.x;
    if (((reinterpret_cast<uintptr_t>(src) | (uintptr_t)nbytes) & 15) == 0) {
        for (int k = tid; k < nbytes / 16; k += THREADS)
            reinterpret_cast<uint4*>(win)[k] = reinterpret_cast<const uint4*>(src)[k];
    } else if (((reinterpret_cast<uintptr_t>(src) | (uintptr_t)nbytes) & 3) == 0) {
        for (int k = tid; k < nbytes / 4; k += THREADS)
            reinterpret_cast<unsigned*>(win)[k] = reinterpret_cast<const unsigned*>(src)[k];
    } else {
        for (int k = tid; k < nbytes; k += THREADS) win[k] = src[k];
    }
}

// Stretches of a window of np positions: as many steps in a stretch as there are stretches, if there are the threads for it.
struct Stretches {
    int steps, count;
};
template <int THREADS>
__device__ __forceinline__ Stretches stretches_of(int np, int T) {
    const int most = WalkShared<THREADS>::ALL / T;
    const int steps = max((np + most - 1) / most, (int)sqrtf((float)np) + 1);
    return {steps, (np + steps - 1) / steps};
}

// Every stretch from every tag (downwards from position np - 1).  Called by the whole workgroup, behind a barrier; one has to follow.
template <int THREADS>
__device__ __forceinline__ void walk_stretches(WalkShared<THREADS>& sm, const Stretches& st, int np, int T) {
    constexpr int ITEMS = WalkShared<THREADS>::ITEMS;
    int g[ITEMS], t[ITEMS], cur[ITEMS], top[ITEMS], n[ITEMS];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const int k = threadIdx.x + q * THREADS;
        g[q] = k / T;
        t[q] = cur[q] = k - g[q] * T;
        top[q] = np - 1 - g[q] * st.steps;
        n[q] = g[q] < st.count ? min(st.steps, top[q] + 1) : 0;
    }
    for (int j = 0; j < st.steps; ++j) {
        int next[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) next[q] = sm.win[max(top[q] - j, 0) * T + cur[q]];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            cur[q] = next[q];  // (past the end of the stretch: never used)
            if (THREADS > 64 && j < n[q]) sm.passed[(j * st.count + g[q]) * T + t[q]] = (uint8_t)next[q];
            if (j == n[q] - 1) sm.left_on[g[q] * T + t[q]] = (uint8_t)next[q];
        }
    }
}

// Positions lo .. lo + np - 1 (their maps in sm.win, behind a barrier) from the tag `cur` above them, tags written to y; returns the tag of
// position lo.
template <int THREADS>
__device__ __forceinline__ int walk_window(WalkShared<THREADS>& sm, int lo, int np, int T, int cur, int32_t* __restrict__ y) {
    const Stretches st = stretches_of<THREADS>(np, T);
    walk_stretches(sm, st, np, T);
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 0; q < st.count; ++q) {
            sm.entered[q] = (uint8_t)cur;
            cur = sm.left_on[q * T + cur];
        }
        sm.entered[st.count] = (uint8_t)cur;
    }
    __syncthreads();
    if constexpr (THREADS > 64) {
        for (int k = threadIdx.x; k < np; k += THREADS) {
            const int q = k / st.steps, j = k - q * st.steps;
            y[lo + np - 1 - k] = sm.passed[(j * st.count + q) * T + sm.entered[q]];
        }
    } else {  // (one wave: writing down every tag passed costs more than a second walk, a lane a stretch: B=512 N=512 T=16 20.0 / 16.2 us, with eight stretches and tags a thread)
        for (int q = threadIdx.x; q < st.count; q += THREADS) {
            const int top = np - 1 - q * st.steps, n = min(st.steps, top + 1);
            int t = sm.entered[q];
            for (int j = 0; j < n; ++j) {
                t = sm.win[(top - j) * T + t];
                y[lo + top - j] = t;
            }
        }
    }
    return sm.entered[st.count];
}

// The tag of the last position, in every thread (-1: no finite path).
template <int K, int THREADS>
__device__ __forceinline__ void share_last_tag(WalkShared<THREADS>& sm, const float* __restrict__ alpha_last, float u, int T) {
    if (threadIdx.x < 64) {
        const int last = draw_last_tag<K>(alpha_last, u, T, threadIdx.x);
        if (threadIdx.x == 0) sm.last = last;
    }
}

// One workgroup a sequence (a grid of bounded size): draws y_{L-1} from alpha_{L-1}, then follows the maps down through LDS
// windows of the table, one after the other.
// us a draw, by a wave, one lane of it where a window has up to 128 positions / so: B=64 N=128 T=20 48 / 42, B=128 N=256 T=32 90.9 / 87.6, B=32 N=100
// T=100 135 / 122, B=4 N=4096 T=16 (several windows) 87 / 77, the walk alone at B=1000 N=120 T=8 11.3 / 5.7.
template <int K, int THREADS>
__global__ __launch_bounds__(THREADS) void sample_walk_kernel(const int32_t* __restrict__ lengths, const float* __restrict__ ua,
                                                                   const Uniforms uniforms, const uint8_t* __restrict__ F,
                                                                   int B, int N, int T, int32_t* __restrict__ tags) {
    __shared__ WalkShared<THREADS> sm;
    const int tid = threadIdx.x;
    const int wp = kWalkWindow / T;  // positions a window (T <= 256: at least 64)
    for (int b = blockIdx.x; b < B; b += gridDim.x) {
        const int L = clamp_length(lengths, b, N);
        int32_t* y = tags + (size_t)b * N;
        for (int i = L + tid; i < N; i += THREADS) y[i] = -1;
        if (L == 0) continue;
        const size_t vb = (size_t)b * N;
        int hi = L - 1;  // positions [0, hi) still to walk
        int lo = hi - wp > 0 ? hi - wp : 0;
        load_window<THREADS>(sm.win, F + vb * T, lo, hi - lo, T);
        share_last_tag<K>(sm, ua + (vb + L - 1) * T, uniforms.at(vb + L - 1), T);
        __syncthreads();
        int cur = sm.last;
        if (cur < 0) {  // no finite path: all tags 0
            for (int i = tid; i < L; i += THREADS) y[i] = 0;
            hi = 0;
        } else if (tid == 0) {
            y[L - 1] = cur;
        }
        while (hi > 0) {
            cur = walk_window(sm, lo, hi - lo, T, cur, y);
            hi = lo;
            lo = hi - wp > 0 ? hi - wp : 0;
            __syncthreads();
            if (hi > 0) load_window<THREADS>(sm.win, F + vb * T, lo, hi - lo, T);
            __syncthreads();
        }
        __syncthreads();
    }
}

// Short sequences, one window each: a wave a sequence, one of its lanes walks.
template <int K>
__global__ __launch_bounds__(64) void sample_short_walk_kernel(const int32_t* __restrict__ lengths, const float* __restrict__ ua,
                                                               const Uniforms uniforms, const uint8_t* __restrict__ F,
                                                               int N, int T, int32_t* __restrict__ tags) {
    __shared__ __attribute__((aligned(16))) uint8_t win[kWalkWindow];
    __shared__ uint8_t path[kWalkShort];
    const int b = blockIdx.x, lane = threadIdx.x;
    const int L = clamp_length(lengths, b, N);
    int32_t* y = tags + (size_t)b * N;
    for (int i = L + lane; i < N; i += 64) y[i] = -1;
    if (L == 0) return;
    const size_t vb = (size_t)b * N;
    load_window<64>(win, F + vb * T, 0, L - 1, T);
    const int last = draw_last_tag<K>(ua + (vb + L - 1) * T, uniforms.at(vb + L - 1), T, lane);
    __syncthreads();
    if (last >= 0 && lane == 0) {
        int cur = last;
        for (int r = L - 2; r >= 0; --r) {
            cur = win[r * T + cur];
            path[r] = (uint8_t)cur;
        }
    }
    __syncthreads();
    for (int i = lane; i < L; i += 64) y[i] = last < 0 ? 0 : i == L - 1 ? last : path[i];  // (no finite path: all tags 0)
}

// Long sequences, all windows at once (W windows a sequence, counted from the top: window w holds the
// positions below L - 1 - w wp).  First every window's maps are composed into one map of the tag above
// the window to the tag of its lowest position (winmap [B][W][T] bytes) ...
template <int THREADS>
__global__ __launch_bounds__(THREADS) void sample_window_map_kernel(const int32_t* __restrict__ lengths,
                                                                         const uint8_t* __restrict__ F, int N, int T, int W,
                                                                         uint8_t* __restrict__ winmap) {
    __shared__ WalkShared<THREADS> sm;
    const int b = blockIdx.x / W, w = blockIdx.x % W;
    const int L = clamp_length(lengths, b, N);
    const int wp = kWalkWindow / T;
    const int hi = L - 1 - w * wp;
    if (hi <= 0) return;
    const int lo = hi - wp > 0 ? hi - wp : 0, np = hi - lo;
    load_window<THREADS>(sm.win, F + (size_t)b * N * T, lo, np, T);
    __syncthreads();
    const Stretches st = stretches_of<THREADS>(np, T);
    walk_stretches(sm, st, np, T);
    __syncthreads();
    for (int t = threadIdx.x; t < T; t += THREADS) {
        int cur = t;
        for (int q = 0; q < st.count; ++q) cur = sm.left_on[q * T + cur];
        winmap[((size_t)b * W + w) * T + t] = (uint8_t)cur;
    }
}

// ... then every window finds the tag above it by passing the tag of the last position through the
// maps of the windows above (at most W look-ups in LDS) and walks its own positions.
template <int K, int THREADS>
__global__ __launch_bounds__(THREADS) void sample_window_walk_kernel(const int32_t* __restrict__ lengths, const float* __restrict__ ua,
                                                                          const Uniforms uniforms, const uint8_t* __restrict__ F,
                                                                          int N, int T, int W, const uint8_t* __restrict__ winmap,
                                                                          int32_t* __restrict__ tags) {
    __shared__ WalkShared<THREADS> sm;
    const int b = blockIdx.x / W, w = blockIdx.x % W, tid = threadIdx.x;
    const int L = clamp_length(lengths, b, N);
    int32_t* y = tags + (size_t)b * N;
    if (w == 0)
        for (int i = L + tid; i < N; i += THREADS) y[i] = -1;
    if (L == 0) return;
    const size_t vb = (size_t)b * N;
    const int wp = kWalkWindow / T;
    const int hi = L - 1 - w * wp;
    const int lo = hi - wp > 0 ? hi - wp : 0;
    if (hi <= 0 && w > 0) return;
    if (hi > 0) load_window<THREADS>(sm.win, F + vb * T, lo, hi - lo, T);
    const uint8_t* above = winmap + (size_t)b * W * T;  // (W T <= kWalkWindow bytes)
    for (int k = tid; k < w * T; k += THREADS) sm.passed[k] = above[k];
    share_last_tag<K>(sm, ua + (vb + L - 1) * T, uniforms.at(vb + L - 1), T);
    __syncthreads();
    int cur = sm.last;
    if (cur < 0) {  // no finite path: all tags 0
        if (w == 0 && tid == 0) y[L - 1] = 0;
        for (int i = lo + tid; i < hi; i += THREADS) y[i] = 0;
        return;
    }
    if (w == 0 && tid == 0) y[L - 1] = cur;
    if (hi <= 0) return;
    for (int v = 0; v < w; ++v) cur = sm.passed[v * T + cur];
    __syncthreads();
    walk_window(sm, lo, hi - lo, T, cur, y);
}

// Four waves a position up to 128 tags (sixteen rows a thread at most), eight up to 176, sixteen above.
// (A launch holds fewer than 2^32 threads: 2^22 positions of sixteen waves.  Launches of 2^18 positions take half a millisecond and more each.)
constexpr unsigned kWidePart = 1u << 18;
template <typename TIN, bool ALIGNED>
static void launch_sample_map_wide(const TIN* phi, const int32_t* lengths, const float* ua, const double* Oa, const Uniforms uniforms, int B,
                                   int N, int T, uint8_t* F, hipStream_t st) {
    const unsigned positions = (unsigned)B * (unsigned)(N - 1);  // (below 2^31: the potentials of as many would be 18 TB)
    const int W = T <= 128 ? 256 : T <= 176 ? 512 : 1024, G = W / ((T + 3) / 4), rows = (T + G - 1) / G;
#define LCCRF_SAMPLE_MAP(W_, R_) hipLaunchKernelGGL((sample_map_wide_kernel<TIN, ALIGNED, W_, R_>), grid, dim3(W_), 0, st, phi, lengths, ua, Oa, uniforms, from, N, T, F)
    for (unsigned from = 0; from < positions; from += kWidePart) {
        const dim3 grid(positions - from < kWidePart ? positions - from : kWidePart);
        if (W == 256) {
            if (rows <= 5) LCCRF_SAMPLE_MAP(256, 5);
            else if (rows <= 6) LCCRF_SAMPLE_MAP(256, 6);
            else if (rows <= 8) LCCRF_SAMPLE_MAP(256, 8);
            else if (rows <= 10) LCCRF_SAMPLE_MAP(256, 10);
            else if (rows <= 13) LCCRF_SAMPLE_MAP(256, 13);
            else LCCRF_SAMPLE_MAP(256, 16);
        } else if (W == 512) {
            if (rows <= 10) LCCRF_SAMPLE_MAP(512, 10);
            else if (rows <= 12) LCCRF_SAMPLE_MAP(512, 12);
            else if (rows <= 14) LCCRF_SAMPLE_MAP(512, 14);
            else LCCRF_SAMPLE_MAP(512, 16);
        } else {
            if (rows <= 9) LCCRF_SAMPLE_MAP(1024, 9);
            else if (rows <= 10) LCCRF_SAMPLE_MAP(1024, 10);
            else if (rows <= 11) LCCRF_SAMPLE_MAP(1024, 11);
            else if (rows <= 12) LCCRF_SAMPLE_MAP(1024, 12);
            else if (rows <= 14) LCCRF_SAMPLE_MAP(1024, 14);
            else LCCRF_SAMPLE_MAP(1024, 16);
        }
    }
#undef LCCRF_SAMPLE_MAP
}

// A lane walks short sequences (us a draw, so / in stretches: B=4 N=16 T=12 13.3 / 12.9, B=2048 N=16 T=16 32.8 / 39.5, B=1000 N=120 T=8 105 / 102).
// Eight waves a workgroup while each has a compute unit to itself; beyond, one.  (Two or eight waves there walk as fast, but the next call's
// forward chains, workgroups of one wave, then come to lie two to a SIMD: B=512 N=512 T=16 312 us, behind them 348.)
// The windows of long sequences: eight waves where the forward chains are workgroups of many waves (up to 256 sequences), four elsewhere; one wave takes
// twice as long over a window of twenty tags as four.  us a draw, one wave / four / eight: B=118 N=2213 T=20 638 / 601 / 593, B=44 N=3177 T=31 589 / 557 / 550,
// B=300 N=1370 T=12 448 / 415 / 410, but B=441 N=767 T=24 748 / 761 / 798.
#define LCCRF_WALK_BY_TAGS(LAUNCH_, threads_) \
    do {                                      \
        if (T <= 64) LAUNCH_(1, threads_);    \
        else if (T <= 128) LAUNCH_(2, threads_); \
        else LAUNCH_(4, threads_);            \
    } while (0)

template <typename TIN>
static hipError_t launch_sample_T(const TIN* phi, const int32_t* lengths, const float* ua, const double* Oa,
                                  const Uniforms uniforms, int B, int N, int T, uint8_t* F, uint8_t* winmap, int32_t* tags,
                                  hipStream_t st) {
    if (N > 1) {
        const long long units = (long long)B * (N - 1);
        auto blocks = [&](int ppw) { return dim3((unsigned)((units + 4 * ppw - 1) / (4 * ppw))); };
        if (T <= 16)
            hipLaunchKernelGGL((sample_map_kernel<TIN, 16>), blocks(4), dim3(256), 0, st, phi, lengths, ua, Oa, uniforms, B, N, T, F);
        else if (T <= 32)
            hipLaunchKernelGGL((sample_map_kernel<TIN, 32>), blocks(2), dim3(256), 0, st, phi, lengths, ua, Oa, uniforms, B, N, T, F);
        else if (T <= 64)
            hipLaunchKernelGGL((sample_map_kernel<TIN, 64>), blocks(1), dim3(256), 0, st, phi, lengths, ua, Oa, uniforms, B, N, T, F);
        else if ((T & 3) == 0) launch_sample_map_wide<TIN, true>(phi, lengths, ua, Oa, uniforms, B, N, T, F, st);
        else launch_sample_map_wide<TIN, false>(phi, lengths, ua, Oa, uniforms, B, N, T, F, st);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // Several windows a sequence: all of them at once, two launches, if their maps fit the LDS staging.
    const int wp = kWalkWindow / T, W = N > 1 ? (N - 1 + wp - 1) / wp : 1;
    if (W >= 2 && (size_t)W * T <= kWalkWindow && winmap) {
        const dim3 grid(B * W);
#define LCCRF_WINDOWS(K_, THREADS_)                                                                                                          \
    do {                                                                                                                                     \
        hipLaunchKernelGGL(sample_window_map_kernel<THREADS_>, grid, dim3(THREADS_), 0, st, lengths, F, N, T, W, winmap);                    \
        const hipError_t e = hipGetLastError();                                                                                              \
        if (e != hipSuccess) return e;                                                                                                       \
        hipLaunchKernelGGL((sample_window_walk_kernel<K_, THREADS_>), grid, dim3(THREADS_), 0, st, lengths, ua, uniforms, F, N, T, W, winmap, tags); \
    } while (0)
        if (B <= 256) LCCRF_WALK_BY_TAGS(LCCRF_WINDOWS, 512);
        else LCCRF_WALK_BY_TAGS(LCCRF_WINDOWS, 256);
#undef LCCRF_WINDOWS
        return hipGetLastError();
    }
    if (N - 1 <= wp && N <= (B > 2048 ? kWalkShort : B > 256 ? 64 : 12)) {  // (of many sequences the look-ups of the ones hide behind those of the others)
        if (T <= 64) hipLaunchKernelGGL(sample_short_walk_kernel<1>, dim3(B), dim3(64), 0, st, lengths, ua, uniforms, F, N, T, tags);
        else if (T <= 128) hipLaunchKernelGGL(sample_short_walk_kernel<2>, dim3(B), dim3(64), 0, st, lengths, ua, uniforms, F, N, T, tags);
        else hipLaunchKernelGGL(sample_short_walk_kernel<4>, dim3(B), dim3(64), 0, st, lengths, ua, uniforms, F, N, T, tags);
        return hipGetLastError();
    }
    const dim3 grid(B < (1 << 20) ? B : 1 << 20);
#define LCCRF_WALK(K_, THREADS_) hipLaunchKernelGGL((sample_walk_kernel<K_, THREADS_>), grid, dim3(THREADS_), 0, st, lengths, ua, uniforms, F, B, N, T, tags)
    if (B <= 256) LCCRF_WALK_BY_TAGS(LCCRF_WALK, 512);
    else LCCRF_WALK_BY_TAGS(LCCRF_WALK, 64);
#undef LCCRF_WALK
    return hipGetLastError();
}

// ua, Oa: alpha of every position from the forward pass ([B][N][T] normalised vectors, [B][N] offsets);
// F: [B][N][T] bytes of scratch for the maps; winmap: sample_winmap_bytes(B, N, T) bytes of scratch for
// the composed maps of the windows of long sequences (null: windows are walked one after the other).
size_t sample_winmap_bytes(int B, int N, int T) {
    const int wp = kWalkWindow / T;
    return (size_t)B * ((N + wp - 1) / wp + 1) * T;
}

hipError_t launch_backward_sample(int dtype, const void* phi, const int32_t* lengths, const float* ua, const double* Oa,
                                  const float* uniforms, unsigned long long seed, int B, int N, int T, uint8_t* F,
                                  uint8_t* winmap, int32_t* tags, hipStream_t st) {
    const Uniforms us{uniforms, seed};
    if (dtype == 0)
        return launch_sample_T(static_cast<const float*>(phi), lengths, ua, Oa, us, B, N, T, F, winmap, tags, st);
    return launch_sample_T(static_cast<const uint16_t*>(phi), lengths, ua, Oa, us, B, N, T, F, winmap, tags, st);
}

}  // namespace lccrf
