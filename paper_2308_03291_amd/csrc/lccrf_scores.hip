// Max-plus chains at 65 .. 256 tags in two steps: the scores alone along the chains, then every pointer at once.
//
// A chain of lccrf_viterbi.hip carries with every score the tag it came from: a comparison and three selections a candidate where
// a maximum is one instruction, all on the dependent path.  The recursion needs the scores only, and the pointers of a
// position need nothing but the scores in front of it and the potentials.  So
//   viterbi_scores_kernel    runs the two half chains of a sequence with additions and maxima (double precision, the very additions
//                            of the other kernels: every score is the same number) and stores the vector in front of every position;
//   viterbi_pointers_kernel  finds the pointers of all positions from them, the whole chip at once;
// the trace follows as behind the other kernels.  A chain is bound by its double-precision additions, conversions and maxima
// (T^2 a step on one compute unit), the pointers of large calls by the second reading of the potentials (6.1 TB/s at B=4 N=512 T=128, 6.2
// at B=8 N=512 T=256, 3.6 for bfloat16 rows off the 8-byte grid, B=32 N=256 T=201), structured ones by their comparisons.
// Measured, whole argmax, us, chains with tags / these: B=8 N=64 T=78 65 / 39 (the chains 29, the pointers 5), bf16 B=32 N=100
// T=96 125 / 72, B=4 N=50 T=145 134 / 60, bf16 B=2 N=60 T=201 234 / 94, B=8 N=30 T=256 107 / 71; structured B=5 N=41 T=70 66 / 28,
// B=64 N=100 T=96 150 / 75, B=600 N=30 T=100 223 / 147.  Where it is not taken: B=64 N=40 T=128 46 / 57, B=128 N=40 T=145 130 / 167.
//
// Layout of a chain: sixteen waves, LPR lanes a row with four columns each, ITEMS rows a thread.  Loads never leave a matrix: rows
// past it are its last row again, and the last piece of a row is moved back to end with it; what is then held twice is the
// same candidate twice, which a maximum does not mind.  A row of the next position is requested where the one at hand has been used.
#include "lccrf_chain_args.h"
#include "lccrf_device.h"
#include "lccrf_launch.h"
#include "lccrf_linear.h"
#include "lccrf_viterbi_args.h"

namespace lccrf {

namespace {

template <int LPR_, int ITEMS_>
struct ScoreGeo {
    static constexpr int LPR = LPR_, ITEMS = ITEMS_, RPP = 1024 / LPR_, TC = 4 * LPR_;
    static constexpr int RP = LPR_ / 4 + 1;  // doubles between the partial maxima of two rows (backward)
    static constexpr int PART = 16 * TC > RPP * ITEMS_ * RP ? 16 * TC : RPP * ITEMS_ * RP;
};

// n steps of a chain from the vector in vec[0] (a barrier behind it); DIR 0: position first + s and so on, 1: first - s.  delta: where
// the vector in front of every step goes (row of the position it belongs to).  Returns the buffer of the last vector.
template <typename G, int DIR, typename TIN, bool STRUCT>
__device__ __forceinline__ int score_steps(const VitArgs& a, int b, int first, int n, double* vec, double* part, double* delta) {
    using Raw = RawPiece<TIN>;
    constexpr int ITEMS = G::ITEMS, LPR = G::LPR, TC = G::TC;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = a.T;
    const size_t TT = (size_t)T * T, vb = (size_t)b * a.N;
    if (n <= 0) return 0;
    const int cl = tid % LPR, g = tid / LPR, c4 = min(4 * cl, T - 4), Q4 = (T + 3) >> 2;
    const TIN* phib = STRUCT ? nullptr : static_cast<const TIN*>(a.phi) + vb * TT;
    unsigned voff[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) voff[k] = (unsigned)(min(g + G::RPP * k, T - 1) * T + c4) * (unsigned)sizeof(TIN);
    typename Raw::type raw[ITEMS];  // dense: the matrix at hand; structured: the transitions
    vec4f em = {0.f, 0.f, 0.f, 0.f};
    const auto position = [&](int s) { return DIR == 0 ? first + (s < n ? s : n - 1) : first - (s < n ? s : n - 1); };
    const auto fetch = [&](int s, int k) __attribute__((always_inline)) {
        auto base = (const GlobalBytes*)(phib + (size_t)position(s) * TT);
        asm("" : "+s"(base));
        raw[k] = Raw::template load<false>(base + voff[k]);
    };
    const auto scores = [&](int s) __attribute__((always_inline)) {  // structured: the emission scores of this thread's columns
        em = *reinterpret_cast<const vec4f_anywhere*>(a.emit + (vb + position(s)) * T + c4);
    };
    if constexpr (STRUCT) {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) raw[k] = Raw::template load<false>((const GlobalBytes*)a.trans + voff[k]);
        scores(0);
    } else {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) fetch(0, k);
    }
    // forward: column u of a wave's partial maxima stands at column slot u, or where its piece was moved back from
    const int last = 4 * (Q4 - 1), me = min(tid, T - 1), cslot = me < last ? me : last + me - (T - 4);
    int buf = 0;
    for (int s = 0; s < n; ++s) {
        const double* v = vec + buf * TC;
        double* next = vec + (buf ^ 1) * TC;
        if (tid < T) delta[(vb + (DIR == 0 ? first + s - 1 : first - s)) * T + tid] = v[tid];
        const vec4f emit = em;
        if constexpr (STRUCT) scores(s + 1);
        if constexpr (DIR == 0) {
            double acc[4] = {-__builtin_huge_val(), -__builtin_huge_val(), -__builtin_huge_val(), -__builtin_huge_val()};
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const double d = v[min(g + G::RPP * k, T - 1)];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float x = STRUCT ? Raw::get(raw[k], j) + emit[j] : Raw::get(raw[k], j);
                    acc[j] = max_plain(acc[j], d + (double)x);
                }
                if constexpr (!STRUCT) {
                    __builtin_amdgcn_sched_barrier(0);  // (the new row goes where the old one was)
                    fetch(s + 1, k);
                }
            }
            if constexpr (LPR == 32) {  // the wave's two rows of a pass
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const long long x = __double_as_longlong(acc[j]);
                    const auto lo = __builtin_amdgcn_permlane32_swap((int)x, (int)x, false, false);
                    const auto hi = __builtin_amdgcn_permlane32_swap((int)(x >> 32), (int)(x >> 32), false, false);
                    acc[j] = max_plain(__longlong_as_double(((long long)(int)hi[0] << 32) | (unsigned)lo[0]),
                                       __longlong_as_double(((long long)(int)hi[1] << 32) | (unsigned)lo[1]));
                }
            }
            if (lane < LPR) {
#pragma unroll
                for (int j = 0; j < 4; ++j) part[wave * TC + 4 * cl + j] = acc[j];
            }
            __syncthreads();
            if (tid < TC) {  // (whole waves)
                double m = part[cslot];
#pragma unroll
                for (int w = 1; w < 16; ++w) m = max_plain(m, part[w * TC + cslot]);
                if (tid < T) next[tid] = m;
            }
        } else {
            double v4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v4[j] = v[c4 + j];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                double m = -__builtin_huge_val();
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float x = STRUCT ? Raw::get(raw[k], j) + emit[j] : Raw::get(raw[k], j);
                    m = max_plain(m, (double)x + v4[j]);
                }
                if constexpr (!STRUCT) {
                    __builtin_amdgcn_sched_barrier(0);
                    fetch(s + 1, k);
                }
                m = max_quad(m);
                if ((lane & 3) == 0) part[(g + G::RPP * k) * G::RP + cl / 4] = m;
            }
            __syncthreads();
            {   // four threads a row (their quarter of its partial maxima), 256 rows a pass
                constexpr int PER = LPR / 16;  // partial maxima a thread takes
                const int q = tid & 3, row = tid >> 2;
                if (row < TC) {
                    const double* p = part + (row < G::RPP * ITEMS ? row : 0) * G::RP + q * PER;
                    double m = p[0];
#pragma unroll
                    for (int k = 1; k < PER; ++k) m = max_plain(m, p[k]);
                    m = max_quad(m);
                    if (q == 0 && row < T) next[row] = m;
                }
            }
        }
        __syncthreads();
        buf ^= 1;
    }
    return buf;
}

}  // namespace

template <typename G, typename TIN, bool STRUCT>
__global__ __launch_bounds__(1024) void viterbi_scores_kernel(VitArgs a, double* delta) {
    __shared__ __attribute__((aligned(16))) double vec[2 * G::TC], part[G::PART];
    const int tid = threadIdx.x, T = a.T;
    const int dir = blockIdx.x & 1, b = blockIdx.x >> 1;
    const int L = clamp_length(a.lengths, b, a.N);
    if (L == 0) return;
    const int e = L - 1, h = meeting_point(0, e);
    if (tid < G::TC) {
        double v = -__builtin_huge_val();
        if (tid < T) {
            v = 0.0;
            if (dir == 0) {
                if constexpr (STRUCT) v = (double)(a.trans[tid] + a.emit[(size_t)b * a.N * T + tid]);
                else v = (double)Elem<TIN>::get(static_cast<const TIN*>(a.phi) + (size_t)b * a.N * T * T + tid);
            }
        }
        vec[tid] = v;
    }
    __syncthreads();
    const int buf = dir == 0 ? score_steps<G, 0, TIN, STRUCT>(a, b, 1, h, vec, part, delta)
                             : score_steps<G, 1, TIN, STRUCT>(a, b, e, e - h, vec, part, delta);
    if (tid < T) a.mid[((size_t)b * 2 + dir) * T + tid] = vec[buf * G::TC + tid];
}

constexpr unsigned kNoTag = 256;
constexpr int kPointerThreads = 512;
constexpr unsigned kPointerGroups = 4096, kPointerStep = 2531;  // (a power of two, and an odd number near five eighths of it)
constexpr unsigned kPointersOneEach = 12288;                    // workgroups, one a position, up to which no positions are searched

// The pointers of every position: up to the meeting position h the best tag in front of each tag, behind it the best tag behind each;
// the first of equals, tag 0 where nothing is finite (as the other kernels).  The best scores are there already, so a candidate
// takes its addition and one comparison for equality.  A workgroup takes a position, from 129 tags on one half of its tags (PARTS
// 2: half the columns forward, half the rows backward), so that two of them share a compute unit and one computes while the other
// waits for its matrix, which is requested whole before anything is waited for.  Forward a thread keeps the first of its rows for each
// of its columns and they meet in LDS; backward the first lane of a row that holds its best score names the tag.
template <int PARTS, int ITEMS, typename TIN, bool STRUCT>
__device__ __forceinline__ void point_position(const VitArgs& a, const double* delta, int part, int b, int i, int L, double* v, double* m, unsigned* arg) {
    using Raw = RawPiece<TIN>;
    constexpr int TC = 128 * PARTS;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // (addresses formed again for every position: kept over a loop around this they are half the registers)
    const int lane = tid & 63, N = a.N, T = a.T;
    const int h = meeting_point(0, L - 1);
    const bool forward = i <= h;
    const size_t vb = (size_t)b * N;
    const auto base = (const GlobalBytes*)(STRUCT ? (const void*)a.trans : (const void*)(static_cast<const TIN*>(a.phi) + (vb + i) * T * T));
    const auto vectors = [&]() __attribute__((always_inline)) {  // in front of the position, and the best scores
        const double* from = delta + (vb + (forward ? i - 1 : i)) * T;
        const double* best = i == h ? a.mid + (size_t)b * 2 * T : i == h + 1 ? a.mid + ((size_t)b * 2 + 1) * T : delta + (vb + (forward ? i : i - 1)) * T;
        if (tid < TC) {
            v[tid] = tid < T ? from[tid] : 0.0;
            arg[tid] = kNoTag;
        }
        const int t = kPointerThreads - 1 - tid;
        if (t < TC) m[t] = t < T ? best[t] : 0.0;
        __syncthreads();
    };
    typename Raw::type raw[ITEMS];
    vec4f emit = {0.f, 0.f, 0.f, 0.f};
    int first_tag, last_tag;  // of this workgroup's part
    if (forward) {
        constexpr int LPR = 32, RPP = kPointerThreads / LPR;
        const int cl = tid % LPR, g = tid / LPR, c4 = min(TC / PARTS * part + 4 * cl, T - 4);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            raw[k] = Raw::template load<false>(base + (unsigned)(min(g + RPP * k, T - 1) * T + c4) * (unsigned)sizeof(TIN));
        if constexpr (STRUCT) emit = *reinterpret_cast<const vec4f_anywhere*>(a.emit + (vb + i) * T + c4);
        vectors();
        double best[4];
        unsigned first[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { best[j] = m[c4 + j]; first[j] = kNoTag; }
#pragma unroll
        for (int k = ITEMS - 1; k >= 0; --k) {
            const int s = min(g + RPP * k, T - 1);
            const double d = v[s];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x = STRUCT ? Raw::get(raw[k], j) + emit[j] : Raw::get(raw[k], j);
                first[j] = d + (double)x == best[j] ? (unsigned)s : first[j];
            }
            if (k % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // (reads of the vector hoisted further would spill)
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (first[j] != kNoTag) atomicMin(&arg[c4 + j], first[j]);
        first_tag = TC / PARTS * part;
        last_tag = min(first_tag + TC / PARTS, T);
    } else {
        constexpr int LPR = 32 * PARTS, RPP = kPointerThreads / LPR;
        const int cl = tid % LPR, g = tid / LPR + RPP * ITEMS * part, c4 = min(4 * cl, T - 4);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            raw[k] = Raw::template load<false>(base + (unsigned)(min(g + RPP * k, T - 1) * T + c4) * (unsigned)sizeof(TIN));
        if constexpr (STRUCT) emit = *reinterpret_cast<const vec4f_anywhere*>(a.emit + (vb + i) * T + c4);
        vectors();
        double vt[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) vt[j] = v[c4 + j];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int s = min(g + RPP * k, T - 1);
            const double best = m[s];
            unsigned first = kNoTag;
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                const float x = STRUCT ? Raw::get(raw[k], j) + emit[j] : Raw::get(raw[k], j);
                first = (double)x + vt[j] == best ? (unsigned)(c4 + j) : first;
            }
            unsigned long long hit = __ballot(first != kNoTag);
            if constexpr (LPR == 32) hit &= 0xffffffffull << (lane & 32);
            if (lane == __ffsll(hit) - 1) arg[s] = first;
            if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        first_tag = RPP * ITEMS * part;
        last_tag = min(first_tag + RPP * ITEMS, T);
    }
    __syncthreads();
    const int t = first_tag + tid;
    if (t < last_tag) a.bp[(vb + i) * T + t] = (uint8_t)(m[t] == -__builtin_huge_val() ? 0u : arg[t]);
}

// SEARCH: padding is to cost next to nothing.  A workgroup looks at 64 positions at once, a lane each, and takes those that are
// inside their sequences.  Of every kPointerGroups positions in a row it looks at one, not always at the same place (a long sequence
// among short ones, and the first positions of all sequences, are spread over all workgroups).  Otherwise a workgroup a position.
// An empty workgroup costs 0.6 ns, so sequences of 8 in rows of 512 were bound by them (structured, whole argmax, us, a workgroup a
// position / searching / chains with tags: B=256 T=96 99 / 27 / 33, B=512 T=100 219 / 48 / 58; of 30 in 900, B=900 T=70 553 / 185 / 360).  Sequences
// of full length lose up to 3 % of the call by the search, most with few positions a workgroup (structured, N=100, B=256 T=70 154 /
// 159, bfloat16 B=32 N=256 T=201 649 / 660), or gain (B=1000 N=600 T=80 3380 / 3310); hence the line: up to it
// padding costs 5 us at most.  With twice as many workgroups padding costs more (B=256 T=96 32), with half as many full lengths do (B=300
// N=300 T=128 794 -> 806).
template <int PARTS, int ITEMS, typename TIN, bool STRUCT, bool SEARCH>
__global__ __launch_bounds__(kPointerThreads, 4) void viterbi_pointers_kernel(VitArgs a, const double* delta) {
    constexpr int TC = 128 * PARTS;
    __shared__ double v[TC], m[TC];
    __shared__ unsigned arg[TC];
    const unsigned N = (unsigned)a.N;
    const auto take = [&](unsigned item) __attribute__((always_inline)) {
        const int part = (int)(item % PARTS), b = (int)(item / PARTS / N), i = (int)(item / PARTS % N), L = clamp_length(a.lengths, b, a.N);
        if (i > 0 && i < L) point_position<PARTS, ITEMS, TIN, STRUCT>(a, delta, part, b, i, L, v, m, arg);
    };
    if constexpr (!SEARCH) {
        take(blockIdx.x);
    } else {
        const unsigned all = (unsigned)a.B * N * PARTS;
        const auto item_of = [&](unsigned k) { return k * kPointerGroups + ((blockIdx.x + k * kPointerStep) & (kPointerGroups - 1)); };
        for (unsigned k0 = 0; k0 * kPointerGroups < all; k0 += 64) {
            const unsigned mine = item_of(k0 + (threadIdx.x & 63)), q = min(mine, all - 1) / PARTS;
            const int i = (int)(q % N);
            unsigned long long inside = __ballot(mine < all && i > 0 && i < clamp_length(a.lengths, (int)(q / N), a.N));
            for (; inside; inside &= inside - 1) {
                take(item_of(k0 + (unsigned)__builtin_ctzll(inside)));
                __syncthreads();  // (its results have been read)
            }
        }
    }
}

template <typename G, typename TIN, bool STRUCT>
static hipError_t launch_scores_geo(const VitArgs& a, double* delta, hipStream_t st) {
    hipLaunchKernelGGL((viterbi_scores_kernel<G, TIN, STRUCT>), dim3(2 * a.B), dim3(1024), 0, st, a, delta);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int PARTS = G::LPR / 32, ITEMS = (G::ITEMS * G::RPP + 15) / 16;
    static_assert(kPointerThreads / (32 * PARTS) * ITEMS * PARTS >= G::ITEMS * G::RPP, "every row");
    const unsigned all = (unsigned)a.B * a.N * PARTS;
    if (all <= kPointersOneEach) hipLaunchKernelGGL((viterbi_pointers_kernel<PARTS, ITEMS, TIN, STRUCT, false>), dim3(all), dim3(kPointerThreads), 0, st, a, delta);
    else hipLaunchKernelGGL((viterbi_pointers_kernel<PARTS, ITEMS, TIN, STRUCT, true>), dim3(kPointerGroups), dim3(kPointerThreads), 0, st, a, delta);
    return hipGetLastError();
}
template <typename TIN, bool STRUCT>
static hipError_t launch_scores_T(const VitArgs& a, double* delta, hipStream_t st) {
    hipError_t e = hipErrorInvalidValue;
    if (a.T <= 96) e = launch_scores_geo<ScoreGeo<32, 3>, TIN, STRUCT>(a, delta, st);
    else if (a.T <= 128) e = launch_scores_geo<ScoreGeo<32, 4>, TIN, STRUCT>(a, delta, st);
    else if constexpr (!STRUCT) {
        if (a.T <= 160) e = launch_scores_geo<ScoreGeo<64, 10>, TIN, STRUCT>(a, delta, st);
        else if (a.T <= 208) e = launch_scores_geo<ScoreGeo<64, 13>, TIN, STRUCT>(a, delta, st);
        else e = launch_scores_geo<ScoreGeo<64, 16>, TIN, STRUCT>(a, delta, st);
    }
    return e;
}

// Whether the scores and pointers go separately.  Structured potentials are read again from a cache, so from six positions on it
// always pays (N=8: B=1 T=65 18 / 14 us, B=1024 T=128 97 / 74; fewer do not pay the third launch).  Dense ones cost a second
// reading, at 5 TB/s while the memory-side cache holds them and 3.5 beyond, against the time that the chains save a position (a step
// of both chains is two): the difference of the two schedules with that reading taken out, B 32 .. 128, N=40: f32 0.35 .. 0.45 us at
// 96 .. 128 tags, 0.47 .. 0.6 where rows are off the 16-byte grid (78, 97), bf16 0.53 .. 0.7 and 1.2 .. 1.35, twice that where two
// chains share a compute unit; above 128 tags 1.7 .. 2.4 and 1.9 .. 2.8.  The larger margin of 4 us is the launch and the spread.
// (The scores' rows are held to half a gigabyte.)
bool max_scores_pay(int dtype, int B, int N, int T, bool structured) {
    if (T <= 64 || T > (structured ? 128 : 256) || N < 6 || (double)B * N * T > 6.4e7) return false;
    if (structured) return true;
    const double bytes = (double)B * N * T * T * (dtype == 0 ? 4.0 : 2.0);
    const double saved = T > 128 ? (dtype == 0 ? 1.7 : 1.9) : dtype == 0 ? ((T % 4) == 0 ? 0.37 : 0.47) : ((T % 4) == 0 ? 0.53 : 1.2) * (B > 128 ? 2.0 : 1.0);
    return N * saved - bytes / (bytes <= 256e6 ? 5e6 : 3.5e6) > 4.0;
}

hipError_t launch_max_scores(int dtype, const VitArgs& a, double* delta, hipStream_t st) {
    if (a.T <= 64 || a.T > 256 || a.chunk > 0 || !delta || (a.emit && (a.T > 128 || dtype != 0 || !a.trans))) return hipErrorInvalidValue;
    if (a.emit) return launch_scores_T<float, true>(a, delta, st);
    return dtype == 0 ? launch_scores_T<float, false>(a, delta, st) : launch_scores_T<uint16_t, false>(a, delta, st);
}

}  // namespace lccrf
