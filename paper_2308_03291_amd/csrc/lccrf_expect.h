// The half chains behind the entropy, the cross-entropy and the divergence in scaled probabilities, 33 .. 64 tags, by a
// workgroup of four or eight waves (the queries, and which: lccrf_extras.hip; scaled steps: lccrf_linear.h).
//
// Beside V(u), the scaled sum over the paths behind tag u, a chain carries X(u) = V(u) h(u), h the expectation of what those
// paths add up to.  That is linear too,
//     S(t) = sum_s V(s) E(s,t),   U(t) = sum_s X(s) E(s,t) + V(s) F(s,t),   E = 2^(phi log2 e - c),   F = E f,
// f(s,t) what the edge adds: the exponent of E for the entropy, which is log alpha(t) less the expected score (base 2, the shifts in
// the offsets: what the heavy edges add is small, and so are the roundings); psi for the cross-entropy; phi - psi for the
// divergence.  E and F of the next position are made while the sums of this one are
// exchanged, so a step has no exponential, logarithm or division on its dependent path, and one barrier: a forward wave sums its
// rows over its lanes, the waves' sums meet in LDS and every wave adds them up for itself (lane = tag); a backward wave
// completes its rows and every wave reads them all.  Each wave therefore knows the new vector and decides for itself, all alike,
// whether the step is accepted.
//
// V is S rescaled by the power of two that gives tag 0 the exponent kExpectHead, its offset an integer.  Only differences of h
// between the tags matter, so every step takes h of the heaviest tag of the vector it starts from out of all of them, into a
// double-precision offset (found while the sums of the step are exchanged): X of the tags that carry the weight, and with it
// the rounding of U, stays as small as what one step adds, also where a single path carries nearly all of it.  (Centred at tag 0,
// which such a path leaves tens of bits behind, the entropy of a chain of 256 positions was off by 1.3e-4.)
// The shift of a matrix is what tag 0 grew by at the step before (the first: its largest entry plus the vector's), so that
// the exponents of the heavy edges are near zero, where they are rounded least.  Accepted: every S at least 2^-40 before and within
// [2^-28, 2^52] after rescaling (2^40 either side of tag 0), every |X| at most 2^72.  What underflowed in S (an E below 2^-126: its
// products are held down to 2^-149) is then at most 64 2^52 2^-126 of 2^-40, 2^-28; the same of U, times the size of f.  The
// first step that is not accepted ends the run.
//
// A step costs 0.6 us (48 tags, entropy; the log-domain steps 1.0): two LDS round trips and a barrier on the dependent path, and
// the issue of some 250 instructions by the one wave of a SIMD.  The trip of the new vector through LDS is covered by the
// exponentials of the next matrix, and the matrices are counted as they arrive (see `step`): entropy B=128 N=128 T=48 48.5 -> 45.8 us
// (log-domain steps 69), divergence B=64 N=256 T=64 130 -> 121, with eight waves 110 (172), there at 4.8 TB/s of p once and q twice.
// At B=512 the entropy is bound by memory either way (N=64, 64 tags 99 / 98).
#pragma once

#include "lccrf_device.h"
#include "lccrf_linear.h"

#include <type_traits>

namespace lccrf {

constexpr int kExpectHead = 12;
constexpr int kExpectLanes = 16;  // sixteen lanes a row
constexpr int kExpectPlain = 3;                     // MODE: V alone, no expectation (0, 1, 2: as in lccrf_extras.hip)

template <int WAVES>
struct ExpectSmem {
    // Forward: [2][wave][64] partial sums (S, U) of the steps in turn, and the vector (V, X), 64 entries and a zero.
    // Backward: the sums themselves, S and U apart, 64 entries and from 64 on those of a row's last piece (zero where its neighbour
    // holds them already), then four zeros.
    alignas(16) float part[2][WAVES][64][2];
    alignas(16) float vec[68][2];
    alignas(16) float row[2][2][72];
};

// The state of a chain, in every wave: lane = tag.  v: base-2 logarithms (-inf past T), h: expectation, natural units (MODE 0: base 2).
struct ExpectState {
    float v, h;
    double O, Hoff;  // offsets of v and h
};

// Takes steps of the chain while they are accepted (step s: the matrix of position first + s, backward first - s) and returns their
// number.  Called by the whole workgroup.
template <int WAVES, int ITEMS, typename TIN, bool ALIGNED, bool BACKWARD, int MODE>
__device__ __forceinline__ int expect_run(ExpectSmem<WAVES>& sm, const TIN* phib, const TIN* psib, int T, int first, int n, ExpectState& st) {
    using Raw = RawPiece<TIN>;
    constexpr int LPR = kExpectLanes, W = 64 * WAVES, G = W / LPR, PH = 3;
    constexpr bool CARRY = MODE != kExpectPlain, PSI = MODE == 1 || MODE == 2;
    constexpr int QN = PSI ? ITEMS : 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (n <= 0) return 0;
    phib = uniform(phib);
    psib = uniform(psib);
    first = uniform(first);
    n = uniform(n);
    // the vector the run starts from: what it holds without loss, and finite expectations
    const float top = finite_or_zero(xor_max<1, 64>(st.v));
    const float d = ceilf(top);
    const float v0 = ex2(st.v - d + (float)kExpectHead), x0 = v0 > 0.f ? v0 * (MODE == 0 ? st.h - d : st.h) : 0.f;
    if (!__all((st.v == LCCRF_NEG_INF || st.v - d >= -100.f) && fabsf(x0) <= 0x1p72f && fabsf(d) <= 0x1p20f)) return 0;

    const size_t TT = (size_t)T * T;
    const int Q4 = (T + 3) >> 2;
    const int g = tid / LPR, cl = tid % LPR, c4 = min(4 * cl, T - 4);
    unsigned voff[ITEMS];
#pragma unroll
    for (int m = 0; m < ITEMS; ++m) voff[m] = (unsigned)(min(g + G * m, T - 1) * T + c4) * (unsigned)sizeof(TIN);
    typename Raw::type raw[PH][ITEMS], qraw[PH][QN];
    float e[ITEMS][4], f[CARRY ? ITEMS : 1][4];
    const auto matrix = [&](const TIN* p, int s) {
        const int q = uniform(s < n ? s : n - 1);
        auto base = (const GlobalBytes*)(p + (size_t)(BACKWARD ? first - q : first + q) * TT);
        asm("" : "+s"(base));
        return base;
    };
    const auto fetch = [&](int s, int p) __attribute__((always_inline)) {
        const auto base = matrix(phib, s);
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) raw[p][m] = Raw::template load<ALIGNED>(base + voff[m]);
        if constexpr (PSI) {
            const auto qbase = matrix(psib, s);
#pragma unroll
            for (int m = 0; m < ITEMS; ++m) qraw[p][m] = Raw::template load<ALIGNED>(qbase + voff[m]);
        }
    };
#pragma unroll
    for (int p = 0; p < PH; ++p) fetch(p, p);
    const auto prepare = [&](int p, int s, int shift, auto more) __attribute__((always_inline)) {  // the matrix in slot p, then that of step s into it
        const float c = (float)shift;
#pragma unroll
        for (int m = 0; m < ITEMS; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x = Raw::get(raw[p][m], j);
                const float arg = __builtin_fmaf(x, kLog2e, -c);
                e[m][j] = ex2(arg);
                if constexpr (CARRY) {
                    // an edge without weight adds nothing, whatever its score
                    if constexpr (MODE == 0) {
                        f[m][j] = e[m][j] * fmaxf(arg, -0x1p100f);
                    } else {
                        const float q = Raw::get(qraw[p][m], j);
                        f[m][j] = e[m][j] > 0.f ? e[m][j] * (MODE == 1 ? q : x - q) : 0.f;
                    }
                }
            }
        if constexpr (decltype(more)::value) fetch(s, p);
    };

    // which row or column a lane is left with by the exchanges below, and where the entries lie
    const int last = 4 * (Q4 - 1), me = min(lane, T - 1);
    const int zero_from = BACKWARD ? 68 : 64;
    for (int k = tid; k < (int)(sizeof(ExpectSmem<WAVES>) / sizeof(float)); k += W) reinterpret_cast<float*>(&sm)[k] = 0.f;
    __syncthreads();
    if (!BACKWARD && lane < T) {
        sm.vec[lane][0] = v0;
        sm.vec[lane][1] = x0;
    }
    if (BACKWARD && lane < T) {
        sm.row[1][0][lane] = v0;
        sm.row[1][1][lane] = x0;
        if (lane >= last) {
            sm.row[1][0][64 + lane - (T - 4)] = v0;
            sm.row[1][1][64 + lane - (T - 4)] = x0;
        }
    }
    __syncthreads();
    const int vfrom = !BACKWARD ? 0 : cl < Q4 - 1 ? 4 * cl : cl == Q4 - 1 ? 64 : zero_from;  // backward: this lane's four columns
    int vrow[ITEMS];                                                                         // forward: its rows
#pragma unroll
    for (int m = 0; m < ITEMS; ++m) vrow[m] = g + G * m < T ? g + G * m : zero_from;
    // forward: the swaps leave accumulator 2 (lane >> 5) + ((lane >> 4) & 1) of the sixteen lanes' four columns in a lane
    const int wslot = 4 * cl + 2 * (lane >> 5) + ((lane >> 4) & 1), rslot = me < last ? me : last + me - (T - 4);
    // backward: reduce4_over_lanes leaves row number 2 (lane & 1) + ((lane >> 1) & 1) in a lane
    const int item = 2 * (lane & 1) + ((lane >> 1) & 1), srow = g + G * item;
    const bool publishes = cl < 4 && item < ITEMS && srow < T;

    // the first step grows by the largest entry that meets a path
    float big = LCCRF_NEG_INF;
#pragma unroll
    for (int m = 0; m < ITEMS; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            big = fmaxf(big, __builtin_fmaf(Raw::get(raw[0][m], j), kLog2e, lg2(BACKWARD ? sm.row[1][0][vfrom + j] : sm.vec[vrow[m]][0])));
    big = xor_max<1, 64>(big);
    if (lane == 0) sm.part[1][wave][0][0] = big;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) big = fmaxf(big, sm.part[1][w][0][0]);
    int grew = uniform((int)fminf(fmaxf(ceilf(finite_or_zero(big)), -0x1p20f), 0x1p20f)) - kExpectHead, c_cur = grew;
    __syncthreads();
    prepare(0, PH, c_cur, std::true_type{});

    int done = 0;
    long long Oi = 0, Hi = 0;
    float V = lane < T ? v0 : 0.f, X = x0;  // of the last accepted step, lane = tag
    double shift = 0.0;         // what has moved out of h so far
    float hc = 0.f;             // backward: the shift of h and the scale that the sums at hand have yet to be given
    int k = 0;
    const auto heaviest = [&]() __attribute__((always_inline)) {  // h of the heaviest tag of the vector at hand (any number near it will do)
        const float m = xor_max<1, 64>(V);
        const int at = __builtin_ctzll(__ballot(V == m) | 1ull << 63);
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(X), at)) * __builtin_amdgcn_rcpf(fmaxf(uniform_f(m), 0x1p-126f));
    };
    const auto pair32 = [](float x, float y) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(y), false, false);
        return __int_as_float(r[0]) + __int_as_float(r[1]);
    };
    const auto pair16 = [](float x, float y) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(y), false, false);
        return __int_as_float(r[0]) + __int_as_float(r[1]);
    };
    // The entries of the vector that this thread multiplies by (forward: of its rows; backward: of its columns, as the last
    // step's sums came out), requested as soon as they are written: the exponentials of the next matrix cover the trip.
    float2 vq[BACKWARD ? 1 : ITEMS];
    float4 vr, xr;
    const auto request = [&](int par) __attribute__((always_inline)) {
        if constexpr (!BACKWARD) {
#pragma unroll
            for (int m = 0; m < ITEMS; ++m) vq[m] = *reinterpret_cast<const float2*>(sm.vec[vrow[m]]);
        } else {
            vr = *reinterpret_cast<const float4*>(&sm.row[par][0][vfrom]);
            xr = CARRY ? *reinterpret_cast<const float4*>(&sm.row[par][1][vfrom]) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    request(1);
    // (No branch around a load in here, and none out of the loop over the ring's slots: where paths with and without a step's
    // loads meet, the compiler takes none of them for granted and waits for the newest before it uses the oldest.  A step that
    // is not accepted, and those behind it, change nothing that is returned.  The steps past the last whole round of three stand behind the
    // loop, where nothing is fetched any more: as a round with steps that do nothing, short chains lost to it what the loop gains,
    // entropy B=10 N=27 T=63 15.9 -> 16.7 us, so 15.6; in all by 3 .. 8 %, bfloat16 B=512 N=64 T=63 66.7 -> 63.)
    bool going = true;
    int at = 0;  // steps begun
    const auto step = [&](int next, auto more) __attribute__((always_inline)) {
        const int c_next = max(min(grew, 1 << 20), -(1 << 20)), par = at & 1;
        float S = 0.f, U = 0.f, centre = 0.f;
        if constexpr (!BACKWARD) {
            float as[4] = {0.f, 0.f, 0.f, 0.f}, au[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int m = 0; m < ITEMS; ++m) {
                const float2 q = vq[m];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    as[j] = __builtin_fmaf(e[m][j], q.x, as[j]);
                    if constexpr (CARRY) au[j] = __builtin_fmaf(f[m][j], q.x, __builtin_fmaf(e[m][j], q.y, au[j]));
                }
            }
            float2 mine;
            mine.x = pair16(pair32(as[0], as[2]), pair32(as[1], as[3]));
            mine.y = CARRY ? pair16(pair32(au[0], au[2]), pair32(au[1], au[3])) : 0.f;
            *reinterpret_cast<float2*>(sm.part[par][wave][wslot]) = mine;
            __syncthreads();
            float2 q[WAVES];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) q[w] = *reinterpret_cast<const float2*>(sm.part[par][w][rslot]);
            if (CARRY) centre = heaviest();
#pragma unroll
            for (int w = 0; w < WAVES; w += 4) {
                S += (q[w].x + q[w + 1].x) + (q[w + 2].x + q[w + 3].x);
                if (CARRY) U += (q[w].y + q[w + 1].y) + (q[w + 2].y + q[w + 3].y);
            }
        } else {
            // (the rows at hand are the last step's sums as they came out: scaled and shifted here)
            float v[4] = {vr.x, vr.y, vr.z, vr.w}, x[4] = {xr.x, xr.y, xr.z, xr.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = __builtin_amdgcn_ldexpf(v[j], -k);
                if (CARRY) x[j] = __builtin_fmaf(-hc, v[j], __builtin_amdgcn_ldexpf(x[j], -k));
            }
            float ps[4] = {0.f, 0.f, 0.f, 0.f}, pu[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int m = 0; m < ITEMS; ++m) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    ps[m] = __builtin_fmaf(e[m][j], v[j], ps[m]);
                    if constexpr (CARRY) pu[m] = __builtin_fmaf(f[m][j], v[j], __builtin_fmaf(e[m][j], x[j], pu[m]));
                }
            }
            const float s = reduce4_over_lanes<LPR>(ps[0], ps[1], ps[2], ps[3], lane);
            const float t = CARRY ? reduce4_over_lanes<LPR>(pu[0], pu[1], pu[2], pu[3], lane) : 0.f;
            if (publishes) {
                sm.row[par][0][srow] = s;
                if (CARRY) sm.row[par][1][srow] = t;
                if (srow >= last) {
                    sm.row[par][0][64 + srow - (T - 4)] = s;
                    if (CARRY) sm.row[par][1][64 + srow - (T - 4)] = t;
                }
            }
            __syncthreads();
            S = sm.row[par][0][me];
            if (CARRY) U = sm.row[par][1][me];
            request(par);
            if (CARRY) centre = heaviest();
        }
        const int k_new = uniform(__builtin_amdgcn_frexp_expf(S)) - kExpectHead;  // tag 0's
        const float vn = __builtin_amdgcn_ldexpf(S, -k_new);
        const float xn = CARRY ? __builtin_fmaf(-centre, vn, __builtin_amdgcn_ldexpf(U, -k_new)) : 0.f;
        going = going && __all(S >= 0x1p-40f && vn >= 0x1p-28f && vn <= 0x1p52f && fabsf(xn) <= 0x1p72f);
        V = going ? vn : V;
        X = going ? xn : X;
        k = k_new;
        hc = centre;
        if constexpr (!BACKWARD) {
            *reinterpret_cast<float2*>(sm.vec[me]) = make_float2(vn, xn);  // (every wave, the same values)
            request(0);
        }
        if (CARRY) shift += going ? (double)centre : 0.0;
        grew = c_cur + k_new;
        Oi += going ? grew : 0;
        Hi += going ? c_cur : 0;
        done += going ? 1 : 0;
        going = going && done < n;
        c_cur = c_next;
        ++at;
        prepare(next, at + PH, c_next, more);
    };
    const int rest = n % 3;
    while (going && at + 3 <= n) {
        step(1, std::true_type{});
        step(2, std::true_type{});
        step(0, std::true_type{});
    }
    if (rest > 0) step(1, std::false_type{});
    if (rest > 1) step(2, std::false_type{});
    __syncthreads();  // (the shared state may be used for something else now)
    // (the largest entry brought below 1: the closer the logarithms are to zero, the less their rounding takes)
    const int kv = uniform(__builtin_amdgcn_frexp_expf(xor_max<1, 64>(V)));
    st.v = lane < T ? lg2(__builtin_amdgcn_ldexpf(V, -kv)) : LCCRF_NEG_INF;
    st.h = CARRY && V > 0.f ? X / V : 0.f;
    st.O += (double)d + (double)(Oi + kv - kExpectHead);
    st.Hoff += MODE == 0 ? shift + (double)d + (double)Hi : shift;
    return done;
}

}  // namespace lccrf
