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
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) {
            const int p = ITEMS * bt + m;
            const int k = (p / PPT) * TPP + k0, s = r0 + (p % PPT) * RPP;
            // a segment of k + 1 positions ending at i starts at i - k >= 0; the first segment reads row 0 only
            const bool row_ok = k < K && s < T && (k < i || (k == i && s == 0));
            int sl = cur - (k < K ? k : K - 1);  // ring slot of position i - 1 - k
            if (sl < 0) sl += K;
            // read whatever the row is (the address is inside the ring either way) and decide
            // afterwards: the reads of all rows of the batch are then in flight together
            float rv = ring[sl * T + (s < T ? s : T - 1)];
            asm volatile("" : "+v"(rv));
            const float v = rv + (float)(base[sl] - R);
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
// A step of 32 tags, K = 8 costs 0.84 us (log-domain steps 2.0): two LDS round trips and the barrier on the dependent path, then
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
// Few rows a wave are worth more than few waves (us, N=256 B=1, so / log-domain steps: 32 tags K=8 214 (four waves of eight rows:
// 289) / 513, K=2 132 / 333; 16 tags K=8 134 / 392; 64 tags K=8 553 / 2044; 8 tags K=2 166 / 321; N=64 B=1024: 32 tags K=8 355 / 383,
// 20 tags K=3 55 / 151).  A tag that is forbidden everywhere sends a sequence to the log-domain steps at its first position; in
// large batches before anything is fetched (32 tags K=8 N=64, so / log-domain steps alone: B=1024 384 / 391 (blocks fetched first:
// 393), B=300 167 / 176, B=1 108 / 127; 20 tags K=3 B=1024 152 / 151).
template <int LPR>
static bool launch_semi_linear(int dtype, const SemiArgs& a, hipStream_t st, hipError_t& e) {
    const long long rows = (long long)a.K * a.T;
    constexpr int G = 64 / LPR;  // rows a wave holds at a time
    if constexpr (LPR == 4) {
        if (a.K <= 4) return launch_semi_items<1, LPR, 4>(dtype, a, st, e);
    }
    if (rows <= 2 * 4 * G) return launch_semi_items<4, LPR, 2>(dtype, a, st, e);
    if (rows <= 4 * 4 * G) return launch_semi_items<4, LPR, 4>(dtype, a, st, e);
    if (rows <= 4 * 8 * G) return launch_semi_items<8, LPR, 4>(dtype, a, st, e);
    if (rows <= 8 * 8 * G) return launch_semi_items<8, LPR, 8>(dtype, a, st, e);
    if (rows <= 8 * 16 * G) return launch_semi_items<16, LPR, 8>(dtype, a, st, e);
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
