// Semi-Markov CRF, log-partition (paper, section "Segmentation with Semi-Markov CRF": the linear
// chain's transition-matrix parametrisation, except that a transition may jump over several
// positions; forward algorithm in O(K T^2 L) for segments of at most K positions).
//
// phi[b][i][k][s][t]: log-potential of a segment tagged t that ends at position i and covers
// k + 1 positions, after a segment tagged s (row 0 for the first segment).  The forward step
//     alpha_i(t) = logsumexp over k = 0 .. min(K-1, i) and s of  alpha_{i-k-1}(s) + phi[i][k][s][t]
// is a vector-matrix product in the log semiring whose matrix is the (K T) x T block phi[b][i]
// (contiguous in memory) and whose vector is the last K alphas laid end to end.  One workgroup per
// sequence keeps those K vectors in LDS (a ring, each with a double-precision offset of its own)
// and streams the block through registers in batches of rows (every batch within one or a few of
// the K matrices, so which earlier vector it meets is the same for all threads), prefetched across
// step boundaries: the loads of a step do not depend on the step before it.  Per column a thread keeps a running
// maximum and a sum rescaled to it (exact log-sum-exp in one read), the partial results meet in
// LDS, and the new vector replaces the oldest one.
#include "lccrf_device.h"
#include "lccrf_launch.h"
#include "lccrf_linear.h"
#include "lccrf_rotate.h"

#include <type_traits>

namespace lccrf {

struct SemiArgs {
    const void* phi;
    const int32_t* lengths;
    int B, N, K, T;
    float* logZ;
};

constexpr int kSemiItems = 4;  // rows of a batch held by one thread
constexpr int kSemiPF = 3;     // batches in flight

// LDS: base[K] doubles (padded to an even count), ring[K][T] floats (padded to a multiple of 4), pmax and
// psum [WAVES][4 LPR]: every part starts on a 16-byte boundary.
static size_t semi_lds_bytes(int K, int T, int lpr, int waves) {
    const size_t ring = ((size_t)K * T + 3) / 4 * 4;
    return (size_t)((K + 1) / 2 * 2) * sizeof(double) + ring * sizeof(float) + (size_t)2 * waves * 4 * lpr * sizeof(float) + 16;
}

// Positions `from` .. L - 1 of sequence b in the log domain, from the shared state described above (ring, base: the K last
// vectors and their offsets, `cur` the slot of position from - 1, the newest vector's maximum in *dlast; a barrier lies
// behind it), then logZ.
template <int LPR, int WAVES, typename TIN, bool ALIGNED>
__device__ __forceinline__ void semi_log_steps(const SemiArgs& a, int b, int L, int from, int cur, double R, unsigned char* semi_smem) {
    constexpr int W = 64 * WAVES, RPP = W / LPR, CAP = 4 * LPR, ITEMS = kSemiItems, PF = kSemiPF;
    // One pass of the workgroup covers RPP rows (thread: row r0, columns c4 .. c4+3): a part of one
    // T x T matrix, PPT passes covering it (RPP <= CAP), or TPP whole matrices of consecutive segment
    // lengths (RPP > CAP).  A batch is ITEMS passes.  Which row of its matrix a thread holds in
    // pass p, and which segment length that matrix belongs to, follow from p alone.
    constexpr int PPT = CAP / RPP > 0 ? CAP / RPP : 1, TPP = RPP / CAP > 0 ? RPP / CAP : 1;
    static_assert((PPT * RPP == CAP || TPP * CAP == RPP) && (PPT <= 2 || PPT == 4 || PPT == 16) && ITEMS == 4, "geometry");
    const int K = a.K, T = a.T, N = a.N;
    const int KT = K * T;
    double* base = reinterpret_cast<double*>(semi_smem);
    float* ring = reinterpret_cast<float*>(base + (K + 1) / 2 * 2);
    float* pmax = ring + (KT + 3) / 4 * 4;
    float* psum = pmax + WAVES * CAP;
    float* dlast = psum + WAVES * CAP;  // maximum of the newest vector (T <= 64)

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c4 = 4 * (tid % LPR), r0 = (tid / LPR) % CAP, k0 = (tid / LPR) / CAP;  // k0 = 0 unless TPP > 1
    const size_t TT = (size_t)T * T;
    const TIN* phib = static_cast<const TIN*>(a.phi) + (size_t)b * N * K * TT;
    const int nb = ((K + TPP - 1) / TPP * PPT + ITEMS - 1) / ITEMS;  // batches per position
    const int total = (L - from) * nb;

    float tile[PF][ITEMS][4];
    int li = from, lbt = 0;  // position and batch of the next load
    auto load = [&](int q, int slot) {
        const TIN* mat = phib + (size_t)li * K * TT;
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) {
            const int p = ITEMS * lbt + m;
            const int k = (p / PPT) * TPP + k0, s = r0 + (p % PPT) * RPP;
            const TIN* matk = mat + (size_t)(k < K ? k : K - 1) * TT;
            if (ALIGNED) {
                const TIN* row = matk + (size_t)(s < T ? s : T - 1) * T;
                Elem<TIN>::get4(row + (c4 < T ? c4 : T - 4), tile[slot][m]);
            } else if ((b != a.B - 1 || li != N - 1) && T > 1) {  // (matrices of a later position lie behind these)
                load_row4_anywhere<TIN, true>(matk, T, s, c4, tile[slot][m]);
            } else {
                load_row4_anywhere<TIN, false>(matk, T, s, c4, tile[slot][m]);
            }
        }
        if (q < total - 1 && ++lbt == nb) {
            lbt = 0;
            ++li;
        }
    };

    int i = from, bt = 0;  // position and batch being consumed (R: the offset the new vector is relative to)
    float mx[4], sm[4];
    walk<PF>(0, total - 1, +1, load, [&](int, int slot) {
        if (bt == 0) {
            // The newest vector is stored as it came out of its step; its maximum (found by the threads
            // that formed it, or here by every thread when they span several waves) moves into the
            // offset of the vector being formed.
            float d;
            if constexpr (CAP <= 64) {
                d = *dlast;
            } else {
                d = LCCRF_NEG_INF;
                for (int t = lane; t < T; t += 64) d = fmaxf(d, ring[cur * T + t]);
                d = finite_or_zero(xor_max<1, 64>(d));
            }
            R += (double)d;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mx[j] = LCCRF_NEG_INF;
                sm[j] = 0.f;
            }
        }
        float x[ITEMS][4];
        float bm[4] = {LCCRF_NEG_INF, LCCRF_NEG_INF, LCCRF_NEG_INF, LCCRF_NEG_INF};
        // The entries of the vectors that the rows meet, and the offsets of those: read whatever the row is (the address is inside the ring
        // either way), all of them before any is waited for.  (One after the other they are eight trips to LDS where the compiler
        // does not think of overlapping them: 24 tags, K = 5, N=64, a forbidden tag, 145 us instead of 122.)
        float rv[ITEMS];
        double ro[ITEMS];
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) {
            const int p = ITEMS * bt + m;
            const int k = (p / PPT) * TPP + k0, s = r0 + (p % PPT) * RPP;
            int sl = cur - (k < K ? k : K - 1);  // ring slot of position i - 1 - k
            if (sl < 0) sl += K;
            rv[m] = ring[sl * T + (s < T ? s : T - 1)];
            ro[m] = base[sl];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) {
            const int p = ITEMS * bt + m;
            const int k = (p / PPT) * TPP + k0, s = r0 + (p % PPT) * RPP;
            // a segment of k + 1 positions ending at i starts at i - k >= 0; the first segment reads row 0 only
            const bool row_ok = k < K && s < T && (k < i || (k == i && s == 0));
            const float v = rv[m] + (float)(ro[m] - R);
            if constexpr (!ALIGNED) settle_row4(tile[slot][m], T, c4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[m][j] = row_ok ? __builtin_fmaf(tile[slot][m][j], kLog2e, v) : LCCRF_NEG_INF;
                bm[j] = fmaxf(bm[j], x[m][j]);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float mn = fmaxf(mx[j], bm[j]);
            const float mf = finite_or_zero(mn);
            float acc = sm[j] * ex2(mx[j] - mf);
#pragma unroll
            for (int m = 0; m < ITEMS; ++m) acc += ex2(x[m][j] - mf);
            sm[j] = acc;
            mx[j] = mn;
        }
        if (++bt == nb) {
            float M[4], S[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                M[j] = xor_max<LPR, 64>(mx[j]);
                S[j] = xor_sum<LPR, 64>(sm[j] * ex2(mx[j] - finite_or_zero(M[j])));
            }
            if (lane < LPR) {
                *reinterpret_cast<float4*>(&pmax[wave * CAP + c4]) = make_float4(M[0], M[1], M[2], M[3]);
                *reinterpret_cast<float4*>(&psum[wave * CAP + c4]) = make_float4(S[0], S[1], S[2], S[3]);
            }
            __syncthreads();  // every thread has read the ring for this position
            const int nxt = cur + 1 == K ? 0 : cur + 1;
            float rnew = LCCRF_NEG_INF;
            if (tid < T) {
                float Mt = LCCRF_NEG_INF;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) Mt = fmaxf(Mt, pmax[w * CAP + tid]);
                const float mf = finite_or_zero(Mt);
                float St = 0.f;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) St += psum[w * CAP + tid] * ex2(pmax[w * CAP + tid] - mf);
                rnew = Mt + lg2(St);  // no term at all: -inf
                ring[nxt * T + tid] = rnew;
            }
            if (CAP <= 64 && wave == 0) {  // T <= 64: all of the new vector is in wave 0
                const float d = xor_max<1, 64>(rnew);
                if (lane == 0) *dlast = finite_or_zero(d);
            }
            if (tid == 0) base[nxt] = R;
            __syncthreads();
            cur = nxt;
            bt = 0;
            ++i;
        }
    });

    // logZ = logsumexp of the vector of the last position
    if (wave == 0) {
        float d = LCCRF_NEG_INF;
        for (int t = lane; t < T; t += 64) d = fmaxf(d, ring[cur * T + t]);
        d = xor_max<1, 64>(d);
        float S = 0.f;
        for (int t = lane; t < T; t += 64) S += ex2(ring[cur * T + t] - finite_or_zero(d));
        S = xor_sum<1, 64>(S);
        if (lane == 0) a.logZ[b] = (d == LCCRF_NEG_INF) ? LCCRF_NEG_INF : (float)((base[cur] + (double)d + (double)lg2(S)) * kLn2);
    }
}

template <int LPR, int WAVES, typename TIN, bool ALIGNED>
__global__ __launch_bounds__(64 * WAVES) void semi_forward_kernel(SemiArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char semi_smem[];
    const int K = a.K, T = a.T, KT = K * T, W = 64 * WAVES;
    double* base = reinterpret_cast<double*>(semi_smem);
    float* ring = reinterpret_cast<float*>(base + (K + 1) / 2 * 2);
    float* dlast = ring + (KT + 3) / 4 * 4 + 2 * WAVES * 4 * LPR;
    const int tid = threadIdx.x, b = blockIdx.x;
    const int L = clamp_length(a.lengths, b, a.N);
    if (L == 0) {
        if (tid == 0) a.logZ[b] = 0.f;
        return;
    }
    // The empty prefix sits in the slot "position -1": potential 1 for row 0, nothing else.
    for (int k = tid; k < KT; k += W) ring[k] = LCCRF_NEG_INF;
    for (int k = tid; k < K; k += W) base[k] = 0.0;
    __syncthreads();
    if (tid == 0) {
        ring[(K - 1) * T] = 0.f;
        *dlast = 0.f;
    }
    __syncthreads();
    semi_log_steps<LPR, WAVES, TIN, ALIGNED>(a, b, L, 0, K - 1, 0.0, semi_smem);
}

// ---------------------------------------------------------------------------------------
// The same recursion in scaled probabilities (see lccrf_linear.h for the linear chain's), 8 .. 64 tags: a step is a product of
// the K last vectors, laid end to end, with the (K T) x T block exponentiated one step AHEAD, so that no exponential and no
// logarithm is on the dependent path.  A wave sums its rows' products over its lanes (halving the values a lane carries with
// every permlane swap), the waves' sums meet in LDS behind the step's one barrier, and every wave adds them up for
// itself: lane = tag, so the new vector, its scale and the decision whether the step is accepted need no second exchange.
//
// Vectors are V_i 2^O_i with an integer O_i; entry (k, s, t) of the block of position i is held as
//     E = 2^(phi log2 e - c_i - (O_{i-1} - O_{i-1-k})),
// the vectors' different offsets in the exponents, so that the sums take the vectors as they lie.  V_i is the sum rescaled by the
// power of two that brings tag 0 into [1/2, 1).  c_i has to be chosen before V_{i-1} is known: it is what tag 0 grew by at the
// step before the last one (the first two blocks: the largest first potential), less kSemiHead.  A step is accepted if every
// sum is at least 2^-40 before and within [2^-40, 2^40] after rescaling: what underflowed in it is then at most
// K T 2^40 2^-126 of a sum of 2^-40, below 2^-30 for K T <= 2^16.  At a step that is not accepted the rest of the sequence goes to
// the log-domain steps, from the vectors at hand.
//
// Layout: row r = k T + s of the block, LPR lanes a row, G = W / LPR row groups; thread (g, cl) holds rows g, g + G, ...; the
// last piece of a row is moved back to end with it, rows past the block are its last one again, as in lccrf_linear.h.
// A step of 32 tags, K = 8 costs 0.81 us (log-domain steps 2.0): two LDS round trips and the barrier on the dependent path, then
// the next block's exponentials, which wait for the newest offset.
constexpr int kSemiHead = 24;
constexpr int kSemiLookFirst = 256;  // batches above the number of compute units
constexpr float kSemiLo = 0x1p-40f, kSemiHi = 0x1p40f;
template <int WAVES, int LPR>
static size_t semi_linear_bytes(int K) {  // vec[K + 2][4 LPR], partial sums [2][WAVES][4 LPR], offsets [K + 1]
    return ((size_t)(K + 2) * 4 * LPR + (size_t)2 * WAVES * 4 * LPR + (size_t)K + 1) * sizeof(float);
}

template <int WAVES, int LPR, int ITEMS, typename TIN, bool ALIGNED>
__global__ __launch_bounds__(64 * WAVES) void semi_linear_kernel(SemiArgs a) {
    using Raw = RawPiece<TIN>;
    constexpr int W = 64 * WAVES, G = W / LPR, VS = 4 * LPR, PH = ITEMS <= 2 ? 3 : WAVES == 16 && sizeof(TIN) == 4 ? 1 : 2;  // (PH positions in flight; sixteen waves have 128 registers)
    static_assert(LPR == 4 || LPR == 8 || LPR == 16, "16, 32 or 64 tags");
    extern __shared__ __attribute__((aligned(16))) unsigned char semi_smem[];
    const int K = a.K, T = a.T, N = a.N, KT = K * T;
    const int KR = K + 1;  // slots: the K vectors a step takes and the one it makes; slot KR holds zeros
    float* vec = reinterpret_cast<float*>(semi_smem);
    float* part = vec + (KR + 1) * VS;
    int* Oslot = reinterpret_cast<int*>(part + 2 * WAVES * VS);  // (modulo 2^32: only differences of near ones count)
    const int tid = threadIdx.x, lane = tid & 63, b = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = clamp_length(a.lengths, b, N);
    if (L == 0) {
        if (tid == 0) a.logZ[b] = 0.f;
        return;
    }
    const size_t block = (size_t)K * T * T;
    const TIN* phib = static_cast<const TIN*>(a.phi) + (size_t)b * N * block;
    const int g = tid / LPR, cl = tid % LPR;
    const int c4 = min(4 * cl, T - 4);

    unsigned voff[ITEMS];
    int kk[ITEMS], slot[ITEMS], srow[ITEMS];  // segment length less one; ring slot of the vector it meets, and the entry there
#pragma unroll
    for (int m = 0; m < ITEMS; ++m) {
        const int rc = min(g + G * m, KT - 1);
        kk[m] = rc / T;
        srow[m] = rc - kk[m] * T;
        voff[m] = (unsigned)(rc * T + c4) * (unsigned)sizeof(TIN);
        slot[m] = K - kk[m];  // at position 0 the newest vector (position -1) sits in slot K
        if (g + G * m >= KT) srow[m] = -1;
    }
    typename Raw::type raw[PH][ITEMS];
    float e[ITEMS][4];
    auto fetch = [&](int i, int m) {
        auto base = (const GlobalBytes*)(phib + (size_t)(i < L ? i : L - 1) * block);
        asm("" : "+s"(base));
        return Raw::template load<ALIGNED>(base + voff[m]);
    };
    // A tag that the sequence cannot start with is an exact zero in the first vector, which is not accepted.  With many sequences
    // it is looked for before the first blocks are fetched: others hide the wait, and nothing is read twice.
    float big = lane < T ? Elem<TIN>::get(phib + lane) * kLog2e : LCCRF_NEG_INF;
    bool rejected = a.B > kSemiLookFirst && __any(lane < T && big == LCCRF_NEG_INF);
    if (!rejected) {
#pragma unroll
        for (int p = 0; p < PH; ++p)
#pragma unroll
            for (int m = 0; m < ITEMS; ++m) raw[p][m] = fetch(p, m);
    }

    for (int k = tid; k < (KR + 1) * VS; k += W) vec[k] = 0.f;
    for (int k = tid; k < 2 * WAVES * VS; k += W) part[k] = 0.f;
    for (int k = tid; k < KR; k += W) Oslot[k] = 0;
    // position 0 grows by the largest entry of its first row (looked at by every wave for itself)
    big = xor_max<1, 64>(big);
    int c_cur = uniform((int)fminf(fmaxf(ceilf(finite_or_zero(big)), -0x1p20f), 0x1p20f)) - kSemiHead, grew = c_cur + kSemiHead;
    __syncthreads();
    // the empty prefix, "position -1": potential 1 for row 0, nothing else
    if (tid == 0) vec[K * VS] = 1.f;
    __syncthreads();

    // the block of position i, shift c; O: offset of the vector of position i - 1
    auto prepare = [&](int i, int p, int shift, int O) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) {
            const float c = (float)(shift + (O - Oslot[slot[m]]));
#pragma unroll
            for (int j = 0; j < 4; ++j) e[m][j] = ex2(__builtin_fmaf(Raw::get(raw[p][m], j), kLog2e, -c));
            if (i < K) {  // segments that would start before position 0, rows s > 0 of first segments: never used
                const bool ok = srow[m] >= 0 && (kk[m] < i || (kk[m] == i && srow[m] == 0));
#pragma unroll
                for (int j = 0; j < 4; ++j) e[m][j] = ok ? e[m][j] : 0.f;
            }
            raw[p][m] = fetch(i + PH, m);
        }
    };
    if (!rejected) prepare(0, 0, c_cur, 0);

    // Which column of the wave's sums a lane ends up with: the swaps leave accumulator 2 (lane >> 5) + ((lane >> 4) & 1) there.
    const int jcol = 2 * (lane >> 5) + ((lane >> 4) & 1);
    const int wslot = wave * VS + 4 * cl + jcol;
    const int last = 4 * ((T + 3) / 4 - 1);  // first column slot of the piece that was moved back
    const int me = min(lane, T - 1), rslot = me < last ? me : last + me - (T - 4);
    int i = 0, cur = K;   // position, slot of the vector in front of it
    long long Oi = 0;     // its offset
    float V = 0.f;        // lane = tag
    const auto step = [&](int next) __attribute__((always_inline)) -> bool {  // false: the run is over
        const int c_next = max(min(grew, 1 << 20), -(1 << 20)) - kSemiHead;
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) {
            const float v = vec[srow[m] >= 0 ? slot[m] * VS + srow[m] : KR * VS];
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = __builtin_fmaf(e[m][j], v, acc[j]);
        }
        // over the wave's row groups: after the swap of a pair the lower half holds the one accumulator, the upper the other
        const auto pair32 = [](float x, float y) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(y), false, false);
            return __int_as_float(r[0]) + __int_as_float(r[1]);
        };
        const auto pair16 = [](float x, float y) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(y), false, false);
            return __int_as_float(r[0]) + __int_as_float(r[1]);
        };
        float x = pair16(pair32(acc[0], acc[2]), pair32(acc[1], acc[3]));
        if (LPR <= 8) x += dpp<kDppRowRor8>(x);
        if (LPR <= 4) x += dpp<kDppRowRor4>(x);
        float* mine = part + (i & 1) * WAVES * VS;
        mine[wslot] = x;
        __syncthreads();
        float s = mine[rslot];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) s += mine[w * VS + rslot];
        const int k = uniform(__builtin_amdgcn_frexp_expf(s));  // tag 0's
        const float v = __builtin_amdgcn_ldexpf(s, -k);
        if (!__all(s >= kSemiLo && v >= kSemiLo && v <= kSemiHi)) {
            rejected = true;
            return false;
        }
        const int nxt = cur == K ? 0 : cur + 1;
        vec[nxt * VS + me] = v;  // (every wave, the same values)
        V = v;
        grew = c_cur + k;
        Oi += grew;
        Oslot[nxt] = (int)Oi;
        cur = nxt;
        ++i;
        if (i == L) return false;
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) slot[m] = slot[m] == K ? 0 : slot[m] + 1;
        c_cur = c_next;
        prepare(i, next, c_next, (int)Oi);
        return true;
    };
    if (rejected) {
    } else if constexpr (PH == 1) {
        while (step(0)) {}
    } else if constexpr (PH == 2) {
        while (step(1) && step(0)) {}
    } else {
        while (step(1) && step(2) && step(0)) {}
    }
    if (!rejected) {  // logZ = logsumexp of the vector of the last position
        if (wave == 0) {
            const float S = xor_sum<1, 64>(lane < T ? V : 0.f);
            if (lane == 0) a.logZ[b] = (float)(((double)Oi + (double)lg2(S)) * kLn2);
        }
        return;
    }
    // The sums of position i were not accepted: from there on in the log domain, from the K vectors in front of it (those
    // of positions i - 1, i - 2, ... into slots K - 1, K - 2, ... of the other state; both begin where the other does: through registers).
    double* base = reinterpret_cast<double*>(semi_smem);
    float* ring = reinterpret_cast<float*>(base + (K + 1) / 2 * 2);
    float* dlast = ring + (KT + 3) / 4 * 4 + 2 * WAVES * VS;
    const auto slot_here = [&](int q) {  // where the vector that goes to slot q lies
        const int x = cur - (K - 1 - q);
        return x < 0 ? x + KR : x;
    };
    float keep[ITEMS];  // (K T <= ITEMS W / LPR)
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const int x = tid + q * W;
        keep[q] = x < KT ? lg2(vec[slot_here(x / T) * VS + x % T]) : 0.f;
    }
    const int keepO = tid < K ? (int)Oi - Oslot[slot_here(tid)] : 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ITEMS; ++q)
        if (tid + q * W < KT) ring[tid + q * W] = keep[q];
    if (tid < K) base[tid] = (double)(Oi - keepO);
    __syncthreads();
    if (wave == 0) {
        const float d = xor_max<1, 64>(lane < T ? ring[(K - 1) * T + lane] : LCCRF_NEG_INF);
        if (lane == 0) *dlast = finite_or_zero(d);
    }
    __syncthreads();
    semi_log_steps<LPR, WAVES, TIN, ALIGNED>(a, b, L, i, K - 1, (double)Oi, semi_smem);
}

// ---------------------------------------------------------------------------------------
// The same in scaled probabilities with the recursion taken off the streaming work, as in lccrf_lane.hip.  Of the K T rows that the step
// of position p sums over, only the T of segments of one position meet the vector that the step before has just made; the others
// meet older ones.  So one wave takes the dependent part alone: a T x T product by lane rotations (lccrf_rotate.h), the sums of
// the other rows added to it.  The other waves ("helpers") work ahead of it: while it makes V_p they exponentiate the first matrix
// of position p + 2 into LDS and sum up the rows of longer segments of position p + 1.  The waves meet at one barrier a position.
//
// Offsets and tests are those of the kernel above.  With g_p the running average of what tag 0 grows by, up to position p, the first
// matrix of p is held with the shift c_p = g_{p-3} less kSemiHead and the helpers' sums of p are in units of
// 2^(O_{p-2} + 2 g_{p-2} - kSemiSumHead): their exponents reach kSemiSumHead - kSemiHead further below the sum they go into, which
// is what the chain may stray from that forecast.  If it strays further the sums are scaled up, by up to kSemiSumUp bits (what underflowed
// in them is then at most K T 2^40 2^-126 2^7 of a sum of 2^-40, below 2^-30 for the K T <= 256 here); past that the step is not
// accepted (independent normal potentials: none of 100 chains of 64 positions up to a deviation of 5, at 8 none that is not refused
// for the spread of its vector as well).  With K = 1 there are no such sums.
//
// A position of 32 tags costs 0.42 us with K = 1, which is the chain, and 0.04 .. 0.08 more for every row of longer segments a helper thread
// holds: 0.50 with K = 4, 0.67 with K = 8 where every wave doing the whole step costs 0.81 (from N=64 to N=256 at B=1; whole calls of
// N=64 56.7 -> 48.7 us); 0.33 for 11 tags, K = 3 (0.62).
constexpr int kSemiSumHead = kSemiHead + 40, kSemiSumUp = 7;
template <int WAVES, int NBLK>
struct SemiChainShape {
    static constexpr int U = 16 * NBLK, RS = U + 4, VS = U, H = WAVES - 1;
    static constexpr int E0 = (U + 1) * RS;             // floats of an exponentiated matrix, in the chain wave's order (row U: zeros)
    static constexpr int FIXED = 2 * E0 + 2 * H * 64;   // two of them, and the helpers' sums
    static size_t bytes(int K) { return (size_t)(FIXED + (K + 1) * VS + (K + 1 + 3) / 4 * 4 + 12) * sizeof(float); }
};

// MR: rows of longer segments a helper thread holds; M0: rows of the first matrix.
template <int WAVES, int NBLK, int MR, int M0, typename TIN, bool ALIGNED>
__global__ __launch_bounds__(64 * WAVES) void semi_chain_kernel(SemiArgs a) {
    using Raw = RawPiece<TIN>;
    using S = SemiChainShape<WAVES, NBLK>;
    constexpr int W = 64 * WAVES, LPR = 4 * NBLK, H = S::H, G = 64 * H / LPR, ITEMS = MR + M0;
    constexpr int PH = Raw::WORDS * ITEMS * 3 <= 96 ? 3 : 2;  // positions in flight
    static_assert(WAVES <= 8, "the registers of two waves a SIMD");
    static_assert(G * M0 >= S::U, "the helpers cover a matrix");
    constexpr bool kSplit = NBLK == 2;
    constexpr int NB = kSplit ? 1 : NBLK;
    extern __shared__ __attribute__((aligned(16))) unsigned char semi_smem[];
    const int K = a.K, T = a.T, N = a.N, KT = K * T, KR = K + 1;
    float* E0 = reinterpret_cast<float*>(semi_smem);
    float* part = E0 + 2 * S::E0;      // [2][H][64]
    float* vec = part + 2 * H * 64;    // [K + 1][VS]: V_q in slot (q + 1) % (K + 1)
    int* Oslot = reinterpret_cast<int*>(vec + KR * S::VS);
    int* info = Oslot + (KR + 3) / 4 * 4;  // [2][4]: for the interval of position p, at p & 1: forecast of O_{p+1}, shift of the first matrix of p + 2, whether to go on
    double* Odouble = reinterpret_cast<double*>(info + 8);  // the offset the log-domain steps go on from, and its low word behind it
    const int tid = threadIdx.x, lane = tid & 63, b = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = clamp_length(a.lengths, b, N);
    if (L == 0) {
        if (tid == 0) a.logZ[b] = 0.f;
        return;
    }
    const size_t block = (size_t)K * T * T;
    const TIN* phib = static_cast<const TIN*>(a.phi) + (size_t)b * N * block;
    for (int k = tid; k < S::FIXED + KR * S::VS; k += W) E0[k] = 0.f;
    for (int k = tid; k < KR; k += W) Oslot[k] = 0;
    int stop = 0;         // position that is not accepted (L: none)
    if (wave == 0) {
        // ---------------- the chain ----------------
        __builtin_amdgcn_s_setprio(2);
        const int u = kSplit ? lane & 31 : lane, copy = kSplit ? lane >> 5 : 0;
        const bool on = u < T;
        const int urow = on ? u : S::U;
        const float x0 = on ? Elem<TIN>::get(phib + u) * kLog2e : LCCRF_NEG_INF;
        const int m0 = uniform((int)fminf(fmaxf(ceilf(finite_or_zero(xor_max<1, 64>(x0))), -0x1p20f), 0x1p20f));
        const auto accepted = [&](float s, float v) { return __all(!on || (s >= kSemiLo && v >= kSemiLo && v <= kSemiHi)); };
        float s = on ? ex2(x0 - (float)(m0 - kSemiHead)) : 0.f;
        int k = uniform(__builtin_amdgcn_frexp_expf(s));
        float V = __builtin_amdgcn_ldexpf(s, -k);
        long long O = m0 - kSemiHead + k;
        // What tag 0 grows by, on average: the last growth alone strays with the potentials (deviation 3: by ten bits and more)
        int grew4 = 4 * (m0 + 5);
        const auto average = [&]() { return max(min(grew4 >> 2, 1 << 20), -(1 << 20)); };
        // (offsets and forecasts outside this wave are taken modulo 2^32: only differences of near ones count)
        const auto low = [&](int more) { return (int)((unsigned)O + (unsigned)more); };
        int grew = average();
        const bool good0 = accepted(s, V);
        __syncthreads();  // (everything is cleared)
        // (the empty prefix, V_{-1}: potential 1 for row 0, nothing else)
        if (lane == 0) vec[0] = 1.f;
        if (on && copy == 0) vec[1 % KR * S::VS + u] = V;
        int bA = low(grew), bB = low(2 * grew);   // forecasts of O_p and O_{p+1}
        int cA = grew - kSemiHead, cB = cA, cC = cA;      // shifts of the first matrices of p, p + 1, p + 2
        if (lane == 0) {
            Oslot[1 % KR] = low(0);
            info[0] = bA; info[1] = cA; info[2] = good0 ? 1 : 0;
            info[4] = bB; info[5] = cA; info[6] = 1;
            *Odouble = 0.0;
            info[10] = 0;
        }
        __syncthreads();
        stop = good0 ? L : 0;
        if (good0 && L > 1) {
            __syncthreads();  // the helpers' interval 0
            struct Tile {
                float e[NB][16];
            } tA, tB;
            const auto read_tile = [&](int p, Tile& t) __attribute__((always_inline)) {
                const float* row = E0 + (p & 1) * S::E0 + urow * S::RS + (kSplit ? 16 * copy : 0);
#pragma unroll
                for (int bk = 0; bk < NB; ++bk)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const float4 v = *reinterpret_cast<const float4*>(row + 16 * bk + 4 * g);
                        t.e[bk][4 * g] = v.x; t.e[bk][4 * g + 1] = v.y; t.e[bk][4 * g + 2] = v.z; t.e[bk][4 * g + 3] = v.w;
                    }
            };
            read_tile(1, tA);
            __syncthreads();
            int slot = 2 % KR;  // of V_p
            const auto step = [&](int p, const Tile& cur, Tile& nxt) __attribute__((always_inline)) -> bool {  // false: the chain ends here
                float r[H];
                const float* mine = part + (p & 1) * H * 64 + u;
#pragma unroll
                for (int w = 0; w < H; ++w) r[w] = mine[64 * w];
                read_tile(p + 1, nxt);  // (made an interval ago; past the end whatever is there, never used)
                __builtin_amdgcn_sched_barrier(0);
                float Ab[4], acc[4];
                rotation_blocks<NBLK>(V, copy, Ab);
                mul_rotations(acc, Ab[0], cur.e[0]);
#pragma unroll
                for (int bk = 1; bk < NB; ++bk) fmac_rotations(acc, Ab[bk], cur.e[bk]);
                float x = (acc[0] + acc[1]) + (acc[2] + acc[3]);
                if constexpr (kSplit) {
                    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
                    x = __int_as_float(h[0]) + __int_as_float(h[1]);
                }
#pragma unroll
                for (int step = 1; step < H; step *= 2)
#pragma unroll
                    for (int w = 0; w + step < H; w += 2 * step) r[w] += r[w + step];
                const float sum = r[0];
                const int D = (int)((unsigned)bA - (unsigned)low(cA)) - kSemiSumHead;
                x += on ? __builtin_amdgcn_ldexpf(sum, D) : 0.f;
                const int kx = uniform(__builtin_amdgcn_frexp_expf(x));
                const float v = __builtin_amdgcn_ldexpf(x, -kx);
                const bool good = accepted(x, v) && (D <= kSemiSumUp || K == 1);
                if (good) {
                    V = v;
                    O += cA + kx;
                    grew4 += cA + kx - (grew4 >> 2);
                    grew = average();
                    bA = bB;
                    bB = low(2 * grew);
                    cA = cB;
                    cB = cC;
                    cC = grew - kSemiHead;
                }
                if (on) vec[slot * S::VS + u] = V;
                Oslot[slot] = low(0);
                slot = slot + 1 == KR ? 0 : slot + 1;
                *reinterpret_cast<int4*>(info + 4 * ((p + 1) & 1)) = make_int4(bB, cC, good ? 1 : 0, 0);
                if (!good) {
                    stop = p;
                    *Odouble = (double)O;
                    info[10] = low(0);
                }
                __syncthreads();
                return good && p + 1 < L;
            };
            for (int p = 1;; p += 2) {
                if (!step(p, tA, tB)) break;
                if (!step(p + 1, tB, tA)) break;
            }
        }
        if (stop == L) {  // logZ = logsumexp of the vector of the last position
            const float z = xor_sum<1, 64>(on && copy == 0 ? V : 0.f);
            if (lane == 0) a.logZ[b] = (float)(((double)O + (double)lg2(z)) * kLn2);
            return;
        }
        __builtin_amdgcn_s_setprio(0);
    } else {
        // ---------------- the helpers ----------------
        const int h = tid - 64, g = h / LPR, cl = h % LPR, c4 = min(4 * cl, T - 4);
        unsigned voff[ITEMS];
        int kk[MR], srow[MR], slot[MR];  // segment length less one, row (-1: none), where the vector it meets stands
        const int RT = KT - T;
#pragma unroll
        for (int m = 0; m < MR; ++m) {
            const int rc = max(min(g + G * m, RT - 1), 0);
            kk[m] = K > 1 ? 1 + rc / T : 0;
            srow[m] = g + G * m < RT ? rc % T : -1;
            voff[m] = (unsigned)((kk[m] * T + rc % T) * T + c4) * (unsigned)sizeof(TIN);
            slot[m] = kk[m] <= 1 ? 0 : 1 - kk[m] + KR;  // of V_{-kk}, for the rows of position 1
        }
#pragma unroll
        for (int m = 0; m < M0; ++m) voff[MR + m] = (unsigned)(min(g + G * m, T - 1) * T + c4) * (unsigned)sizeof(TIN);
        typename Raw::type raw[PH][ITEMS], first[M0];
        const auto position = [&](int p) {
            auto base = (const GlobalBytes*)(phib + (size_t)(p < L ? p : L - 1) * block);
            asm("" : "+s"(base));
            return base;
        };
        const auto fetch = [&](int p, int at) __attribute__((always_inline)) {  // what the interval of position p takes
            const auto next = position(p + 1), after = position(p + 2);
#pragma unroll
            for (int m = 0; m < MR; ++m) raw[at][m] = Raw::template load<false>(next + voff[m]);
#pragma unroll
            for (int m = MR; m < ITEMS; ++m) raw[at][m] = Raw::template load<false>(after + voff[m]);
        };
        // (a tag that the sequence cannot start with: with many sequences looked for before anything is fetched, as above)
        const bool vain = a.B > kSemiLookFirst && __any(lane < T && Elem<TIN>::get(phib + min(lane, T - 1)) == LCCRF_NEG_INF);
        if (!vain) {
            const auto next = position(1);
#pragma unroll
            for (int m = 0; m < M0; ++m) first[m] = Raw::template load<false>(next + voff[MR + m]);
#pragma unroll
            for (int p = 0; p < PH; ++p) {
                fetch(p, p);
                asm volatile("" ::: "memory");  // (in this order: the loop's waits count on it)
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // where the entries of a row of the first matrix go
        int eaddr[M0][4];
#pragma unroll
        for (int m = 0; m < M0; ++m) {
            const int v = min(g + G * m, T - 1);
#pragma unroll
            for (int j = 0; j < 4; ++j) eaddr[m][j] = (c4 + j) * S::RS + 16 * (v >> 4) + ((c4 + j - v) & 15);
        }
        // over the wave's row groups: the swaps leave accumulator 2 (lane >> 5) + ((lane >> 4) & 1) in a lane
        const auto pair32 = [](float x, float y) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(y), false, false);
            return __int_as_float(r[0]) + __int_as_float(r[1]);
        };
        const auto pair16 = [](float x, float y) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(y), false, false);
            return __int_as_float(r[0]) + __int_as_float(r[1]);
        };
        const int jcol = 2 * (lane >> 5) + ((lane >> 4) & 1);
        const int target = c4 + jcol;  // the tag whose sum this lane ends up with (several lanes the same, with the same sum)
        __syncthreads();
        __syncthreads();
        bool going = L > 1 && !vain;
        if (going) {   // the first matrix of position 1
            const float c = (float)uniform(info[1]);
#pragma unroll
            for (int m = 0; m < M0; ++m)
                if (g + G * m < T) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) E0[S::E0 + eaddr[m][j]] = ex2(__builtin_fmaf(Raw::get(first[m], j), kLog2e, -c));
                }
        }
        int p = 0;
        const auto interval = [&](int at) __attribute__((always_inline)) {
            // (everything from LDS is requested before any of it is waited for)
            const int4 in = *reinterpret_cast<const int4*>(info + 4 * (p & 1));
            float xv[MR];
            int Ov[MR];
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                xv[m] = vec[slot[m] * S::VS + max(srow[m], 0)];
                Ov[m] = Oslot[slot[m]];
            }
            __builtin_amdgcn_sched_barrier(0);
            going = going && uniform(in.z) != 0 && p < L;
            const int base = (int)((unsigned)uniform(in.x) - (unsigned)kSemiSumHead), shift = uniform(in.y);
            float e[MR][4];
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                // (no row: weight zero by the exponent.  Against the offset of a vector it does not meet a potential may be infinite: K = 1,
                // potentials of -100, sent every chain to the log-domain steps, 30 -> 99 us)
                const float c = srow[m] >= 0 ? (float)((int)((unsigned)base - (unsigned)Ov[m])) : __builtin_huge_valf();
#pragma unroll
                for (int j = 0; j < 4; ++j) e[m][j] = ex2(__builtin_fmaf(Raw::get(raw[at][m], j), kLog2e, -c));
            }
            if (p + 1 < K) {  // segments that would start before position 0, rows s > 0 of first segments: never used
#pragma unroll
                for (int m = 0; m < MR; ++m) {
                    const bool ok = kk[m] <= p || (kk[m] == p + 1 && srow[m] == 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j) e[m][j] = ok ? e[m][j] : 0.f;
                }
            }
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int m = 0; m < MR; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[j] = __builtin_fmaf(e[m][j], xv[m], acc[j]);
            float x = pair16(pair32(acc[0], acc[2]), pair32(acc[1], acc[3]));
            if (LPR <= 8) x += dpp<kDppRowRor8>(x);
            if (LPR <= 4) x += dpp<kDppRowRor4>(x);
            float e0[M0][4];
#pragma unroll
            for (int m = 0; m < M0; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) e0[m][j] = ex2(__builtin_fmaf(Raw::get(raw[at][MR + m], j), kLog2e, -(float)shift));
            // All of it made here, in front of the loads that go where the potentials were: left to itself the compiler moves some of it
            // behind them and then waits for the new ones.
            asm volatile("" : "+v"(x));
#pragma unroll
            for (int m = 0; m < M0; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(e0[m][j]));
            __builtin_amdgcn_sched_barrier(0);
            if (going) {
                part[((p + 1) & 1) * H * 64 + (wave - 1) * 64 + target] = x;
                float* to = E0 + (p & 1) * S::E0;
#pragma unroll
                for (int m = 0; m < M0; ++m)
                    if (g + G * m < T) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) to[eaddr[m][j]] = e0[m][j];
                    }
            }
#pragma unroll
            for (int m = 0; m < MR; ++m) slot[m] = slot[m] + 1 == KR ? 0 : slot[m] + 1;
            fetch(p + PH, at);
            ++p;
            if (going) {
                __syncthreads();
                if (p == 1) __syncthreads();  // (the chain has read the matrix of position 1 before that of position 3 takes its place)
            }
        };
        while (going) {
            interval(0);
            interval(1);
            if constexpr (PH > 2) interval(2);
        }
        if (L > 1) {
            // the chain's last word: the interval it ended in
            const int4 in0 = *reinterpret_cast<const int4*>(info), in1 = *reinterpret_cast<const int4*>(info + 4);
            if (uniform(in0.z) != 0 && uniform(in1.z) != 0) return;
        } else if (uniform(info[2]) != 0) {
            return;
        }
    }
    // Not accepted at some position: from there on in the log domain, from the K vectors in front of it, through registers (both
    // states begin where the other does).  By one wave, four or eight, as their rows take (more meet at more barriers: K=4 T=16 B=200 N=64,
    // deviation 12, by all four 110 us, by one 86; fewer take more rounds: 27 tags, K = 5, a forbidden tag, N=64, by eight 127, by four
    // 160); the others leave.
    if (wave == 0 && lane == 0) info[3] = stop;
    __syncthreads();
    stop = uniform(info[3]);
    const double O = uniform(*Odouble);
    const unsigned Olow = (unsigned)uniform(info[10]);  // (of the double a conversion to 32 bits would be the nearest value, not the low word)
    constexpr bool kEither = NBLK == 2 && MR == 2 && WAVES > 4;  // (K T on both sides of 128)
    constexpr int MOST = NBLK == 1 || (MR <= 2 && !kEither) ? 4 : WAVES;
    const bool one = NBLK == 1 && K <= 4, four = kEither && KT <= 128;
    const int waves = one ? 1 : four ? 4 : MOST;
    double* base = reinterpret_cast<double*>(semi_smem);
    float* ring = reinterpret_cast<float*>(base + (K + 1) / 2 * 2);
    float* dlast = ring + (KT + 3) / 4 * 4 + 2 * waves * 4 * LPR;
    const auto slot_here = [&](int q) {  // where the vector that goes to slot q lies: V_{stop - 1} to K - 1, the older ones below
        const int x = (stop % KR) - (K - 1 - q);
        return x < 0 ? x + KR : x;
    };
    float keep[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int x = tid + q * W;
        keep[q] = x < KT ? lg2(vec[slot_here(x / T) * S::VS + x % T]) : 0.f;
    }
    const int keepO = tid < K ? (int)(Olow - (unsigned)Oslot[slot_here(tid)]) : 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (tid + q * W < KT) ring[tid + q * W] = keep[q];
    if (tid < K) base[tid] = O - (double)keepO;
    __syncthreads();
    if (wave == 0) {
        const float d = xor_max<1, 64>(lane < T ? ring[(K - 1) * T + lane] : LCCRF_NEG_INF);
        if (lane == 0) *dlast = finite_or_zero(d);
    }
    __syncthreads();
    if (wave >= waves) return;
    const auto go_on = [&](auto n) __attribute__((always_inline)) {
        semi_log_steps<LPR, decltype(n)::value, TIN, ALIGNED>(a, b, L, stop, K - 1, O, semi_smem);
    };
    if constexpr (NBLK == 1) {
        if (one) return go_on(std::integral_constant<int, 1>{});
    }
    if constexpr (kEither) {
        if (four) return go_on(std::integral_constant<int, 4>{});
    }
    go_on(std::integral_constant<int, MOST>{});
}

template <int LPR, int WAVES>
static hipError_t launch_semi_geo(int dtype, const SemiArgs& a, hipStream_t st) {
    const size_t lds = semi_lds_bytes(a.K, a.T, LPR, WAVES);
    const bool aligned = (a.T % 4) == 0;
    const dim3 grid(a.B), block(64 * WAVES);
    if (dtype == 0) {
        if (aligned) hipLaunchKernelGGL((semi_forward_kernel<LPR, WAVES, float, true>), grid, block, lds, st, a);
        else hipLaunchKernelGGL((semi_forward_kernel<LPR, WAVES, float, false>), grid, block, lds, st, a);
    } else {
        if (aligned) hipLaunchKernelGGL((semi_forward_kernel<LPR, WAVES, uint16_t, true>), grid, block, lds, st, a);
        else hipLaunchKernelGGL((semi_forward_kernel<LPR, WAVES, uint16_t, false>), grid, block, lds, st, a);
    }
    return hipGetLastError();
}

template <int WAVES, int LPR, int ITEMS>
static bool launch_semi_items(int dtype, const SemiArgs& a, hipStream_t st, hipError_t& e) {
    size_t bytes = semi_linear_bytes<WAVES, LPR>(a.K);
    const size_t log = semi_lds_bytes(a.K, a.T, LPR, WAVES);
    if (log > bytes) bytes = log;
    if (bytes > 64 * 1024 || a.K > 64 * WAVES) return false;
    const bool aligned = (a.T % 4) == 0;
    const dim3 grid(a.B), block(64 * WAVES);
    if (dtype == 0) {
        if (aligned) hipLaunchKernelGGL((semi_linear_kernel<WAVES, LPR, ITEMS, float, true>), grid, block, bytes, st, a);
        else hipLaunchKernelGGL((semi_linear_kernel<WAVES, LPR, ITEMS, float, false>), grid, block, bytes, st, a);
    } else {
        if (aligned) hipLaunchKernelGGL((semi_linear_kernel<WAVES, LPR, ITEMS, uint16_t, true>), grid, block, bytes, st, a);
        else hipLaunchKernelGGL((semi_linear_kernel<WAVES, LPR, ITEMS, uint16_t, false>), grid, block, bytes, st, a);
    }
    e = hipGetLastError();
    return true;
}
// The scaled-probability kernel where it serves the shape: up to eight rows of the (K T) x T block a thread.  false: it does not.
// Few rows a wave are worth more than few waves (us, N=256 B=1, so / log-domain steps, the smaller of these before the chain wave took
// them: 32 tags K=8 214 (four waves of eight rows: 289) / 513, K=2 132 / 333; 16 tags K=8 134 / 392; 64 tags K=8 553 / 2044; N=64
// B=1024: 32 tags K=8 355 / 383, 20 tags K=3 55 / 151).  A tag that is forbidden everywhere sends a sequence to the log-domain steps at its first position; in
// large batches before anything is fetched (32 tags K=8 N=64, so / log-domain steps alone: B=1024 384 / 391 (blocks fetched first:
// 393), B=300 167 / 176, B=1 108 / 127; 20 tags K=3 B=1024 152 / 151).
template <int LPR>
static bool launch_semi_linear(int dtype, const SemiArgs& a, hipStream_t st, hipError_t& e) {
    const long long rows = (long long)a.K * a.T;
    constexpr int G = 64 / LPR;  // rows a wave holds at a time
    if (rows <= 2 * 4 * G) return launch_semi_items<4, LPR, 2>(dtype, a, st, e);
    if (rows <= 4 * 4 * G) return launch_semi_items<4, LPR, 4>(dtype, a, st, e);
    if (rows <= 4 * 8 * G) return launch_semi_items<8, LPR, 4>(dtype, a, st, e);
    if (rows <= 8 * 8 * G) return launch_semi_items<8, LPR, 8>(dtype, a, st, e);
    if (rows <= 8 * 16 * G) return launch_semi_items<16, LPR, 8>(dtype, a, st, e);
    return false;
}

template <int WAVES, int NBLK, int MR, int M0>
static bool launch_semi_chain_items(int dtype, const SemiArgs& a, hipStream_t st, hipError_t& e) {
    constexpr int LPR = 4 * NBLK;
    size_t bytes = SemiChainShape<WAVES, NBLK>::bytes(a.K);
    const size_t log = semi_lds_bytes(a.K, a.T, LPR, WAVES);
    if (log > bytes) bytes = log;
    if (bytes > 64 * 1024 || (long long)a.K * a.T > 2 * 64 * WAVES || a.K > 64 * WAVES) return false;
    const bool aligned = (a.T % 4) == 0;
    const dim3 grid(a.B), block(64 * WAVES);
    if (dtype == 0) {
        if (aligned) hipLaunchKernelGGL((semi_chain_kernel<WAVES, NBLK, MR, M0, float, true>), grid, block, bytes, st, a);
        else hipLaunchKernelGGL((semi_chain_kernel<WAVES, NBLK, MR, M0, float, false>), grid, block, bytes, st, a);
    } else {
        if (aligned) hipLaunchKernelGGL((semi_chain_kernel<WAVES, NBLK, MR, M0, uint16_t, true>), grid, block, bytes, st, a);
        else hipLaunchKernelGGL((semi_chain_kernel<WAVES, NBLK, MR, M0, uint16_t, false>), grid, block, bytes, st, a);
    }
    e = hipGetLastError();
    return true;
}
// Where it is taken.  Up to 16 tags always with few rows, with more while every workgroup has a compute unit to itself (us, so / every
// wave the whole step, single precision: K=4 T=16, N=64, B=256 25.7 / 42.2, B=1024 42.6 / 45.7; K=8 T=16 B=1 N=256 107 / 137, K=8 T=12
// bfloat16 B=300 N=64 44.4 / 41.8; K=3 T=11 B=4 N=90 bfloat16 35.9 / 61.0); with three helpers where their threads hold a row of
// longer segments each (K=4 T=16 B=64 N=100 37.5, with seven 44), with seven above (K=6 T=16 B=4 N=100 43.7, with three 49.4).  At 17 .. 32
// tags while every workgroup has a compute unit to itself (N=64: K=4 T=32 B=256 39.8 / 51.7; K=2 T=32 B=512 42.9 / 40.7, K=3 T=20 B=512
// 41.8 / 39.5), with most rows half of them (K=8 T=32 B=256 90.4 / 88.0).  Above 32 tags the helpers cannot keep ahead of the chain (K=2
// T=64 B=1 N=256 233 / 213, K=7 T=45 B=6 N=31 73.9 / 74.2).
static bool launch_semi_chain(int dtype, const SemiArgs& a, hipStream_t st, hipError_t& e) {
    const long long rows = (long long)(a.K - 1) * a.T;
    if (a.T <= 16) {
        if (rows <= 48) return launch_semi_chain_items<4, 1, 1, 1>(dtype, a, st, e);
        if (rows <= 112 && a.B <= 256) return launch_semi_chain_items<8, 1, 1, 1>(dtype, a, st, e);
        if (rows <= 224 && a.B <= 256) return launch_semi_chain_items<8, 1, 2, 1>(dtype, a, st, e);
    } else if (a.T <= 32 && a.B <= (rows <= 168 ? 256 : 128)) {
        if (rows <= 56) return launch_semi_chain_items<8, 2, 1, 1>(dtype, a, st, e);
        if (rows <= 112) return launch_semi_chain_items<8, 2, 2, 1>(dtype, a, st, e);
        if (rows <= 168) return launch_semi_chain_items<8, 2, 3, 1>(dtype, a, st, e);
        if (rows <= 224) return launch_semi_chain_items<8, 2, 4, 1>(dtype, a, st, e);
    }
    return false;
}

// Geometry by tag count: 4 LPR >= T columns; four waves up to T = 64 (one when T <= 16 and the K
// matrices have no more rows than one wave covers in a batch), sixteen above.
static void semi_geometry(int K, int T, int& lpr, int& waves) {
    lpr = T <= 16 ? 4 : T <= 32 ? 8 : T <= 64 ? 16 : T <= 128 ? 32 : 64;
    waves = T <= 16 ? (K <= 4 ? 1 : 4) : T <= 64 ? 4 : 16;
}

// The K vectors must fit the 64 KB of LDS a workgroup may take without opting in to more.
bool semi_markov_supported(int K, int T) {
    if (K < 1 || T < 1 || T > 256) return false;
    int lpr, waves;
    semi_geometry(K, T, lpr, waves);
    return semi_lds_bytes(K, T, lpr, waves) <= 64 * 1024 && K <= (1 << 24);
}

hipError_t launch_semi_markov_forward(int dtype, const void* phi, const int32_t* lengths, int B, int N, int K, int T,
                                      float* logZ, hipStream_t st) {
    const SemiArgs a{phi, lengths, B, N, K, T, logZ};
    if (T >= 8 && T <= 64) {
        hipError_t e = hipSuccess;
        if (launch_semi_chain(dtype, a, st, e)) return e;
        if (T <= 16 ? launch_semi_linear<4>(dtype, a, st, e) : T <= 32 ? launch_semi_linear<8>(dtype, a, st, e) : launch_semi_linear<16>(dtype, a, st, e))
            return e;
    }
    if (T <= 16) return K <= 4 ? launch_semi_geo<4, 1>(dtype, a, st) : launch_semi_geo<4, 4>(dtype, a, st);
    if (T <= 32) return launch_semi_geo<8, 4>(dtype, a, st);
    if (T <= 64) return launch_semi_geo<16, 4>(dtype, a, st);
    if (T <= 128) return launch_semi_geo<32, 16>(dtype, a, st);
    return launch_semi_geo<64, 16>(dtype, a, st);
}

}  // namespace lccrf
