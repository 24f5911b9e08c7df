// A stretch of a sum-product chain in scaled probabilities, by a whole workgroup: the quick way through the first
// pass at 33 .. 256 tags (lccrf_chain.hip, lccrf_stream.hip).
//
// A step of the log-domain kernels exponentiates the matrix once its own input vector is known, so the exponentials
// sit on the chain of dependent work, and while the partial sums are merged nothing else runs.  Here a step is a
// plain vector-matrix product,
//     S_n(u) = 2^(kLinearHead - k_{n-1}) sum_v S_{n-1}(v) E_n(v, u),      E_n = 2^(phi_n log2 e - c_n),
// (k_{n-1} the exponent of the largest entry of S_{n-1}, c_n an integer) whose matrix is exponentiated one step AHEAD,
// between the two barriers of the step before: the dependent part of a step is one fused multiply-add a potential,
// one exchange through LDS and no exponential or logarithm.  All scales are powers of two, so they round nothing.
//
// c_n has to be chosen before S_{n-1} is known: it is the growth of the step before the last one (the exponent the
// largest entry gained there), the first two matrices taking what the first step will grow by.  The exponents of the heavy
// edges are then near zero, where they are rounded least; the head stands in the vectors, whose largest entry is near
// 2^kLinearHead: their entries reach further below it than the growth strays from one step to the next.  A step is accepted if every
// sum lies in [2^-60, 2^60] and the largest entry of the vector it started from was at least 2^-30: an E below 2^-126 is
// flushed, which takes at most 256 2^k 2^-126 of a sum of 2^(-60 - kLinearHead + k) before scaling, 2^-34, and a product below
// 2^-126 is still held to 2^-149 (denormals are kept): 256 2^-150 of 2^(-84 - 30), 2^-28, for every entry
// separately.  At a step that is not accepted the stretch ends, with the vector in front of that step; the caller's log-domain steps take over from there.
//
// Layout.  Q4 = ceil(T / 4) threads cover a row, four columns each (whatever lanes and waves they fall into: nothing here
// reduces across lanes of a row), so the G = W / Q4 row groups of a workgroup fit the tag count, not the next power of two.
// Thread (g, cl) holds rows g, g + G, ... : the threads of a wave read one contiguous stretch of the matrix.  The last piece of a
// row is moved back to end with it (T >= 4) and rows past the matrix are its last row again (linear_row): every load lies inside
// the matrix whatever the tag count.  What is then held twice meets an exact zero in the sums over it, or is never looked at.
// Forward, the groups' partial sums of a column meet in LDS; backward, the Q4 threads' partial sums of a row: Q threads
// share a column or row there.
#pragma once

#include "lccrf_device.h"


namespace lccrf {

constexpr int kLinearHead = 24;

template <int WAVES_, int TCAP_, int ITEMS_>
struct LinGeo {
    static constexpr int WAVES = WAVES_, TCAP = TCAP_, ITEMS = ITEMS_, W = 64 * WAVES_;
    static constexpr int Q = W / TCAP;     // threads that merge a column or a row
    static constexpr int most_groups() {   // of the tag counts that take this ITEMS (or fewer rows than that)
        int most = 0;
        for (int t = TCAP / 2 + 1; t <= TCAP; ++t) {
            const int groups = W / ((t + 3) / 4);
            const int need = (t + groups - 1) / groups;
            if (need <= ITEMS && need > ITEMS - (ITEMS > 12 ? 2 : 1) && groups > most) most = groups;
        }
        return most;
    }
    static constexpr int PARTS = (most_groups() + Q - 1) / Q;  // partial sums of a column a merging thread adds up
    static constexpr int GMAX = PARTS * Q + 1;     // groups there is room for (the last: threads that are left over)
    static constexpr int STRIDE = TCAP + 64 / Q;   // floats between the groups' partial sums: no bank conflicts either way
    static constexpr int ROW4 = TCAP / 4 / Q;      // floats of a row's partial sums a merging thread adds up ...
    static constexpr int RSTRIDE = TCAP / 4 + 4;   // ... and between rows
    static constexpr int IPAD = (ITEMS + 3) / 4 * 4;  // entries of the vector a group reads (forward)
    static constexpr int VEC = GMAX * IPAD > TCAP + 16 ? GMAX * IPAD : TCAP + 16;
    static constexpr int FORWARD = GMAX * STRIDE, BACKWARD = ITEMS * GMAX * RSTRIDE;
    static constexpr int SCRATCH = FORWARD > BACKWARD ? FORWARD : BACKWARD;
    static_assert((Q == 4 || Q == 8) && ROW4 % 4 == 0 && PARTS >= 1, "a column or row is merged inside eight lanes");
};
// Rows a thread has to hold for a tag count, and the number it is built for (0: none): every count up to twelve, the even ones
// above (single precision splits the tile of those in halves).
constexpr int linear_groups(int W, int T) { return W / ((T + 3) / 4); }
constexpr int linear_items(int W, int T) { return (T + linear_groups(W, T) - 1) / linear_groups(W, T); }
constexpr int linear_instance(int W, int T) {
    const int least = W == 1024 && T > 128 ? 5 : 2, need = linear_items(W, T);
    const int items = need < least ? least : need > 12 ? (need + 1) / 2 * 2 : need;
    return items <= 16 ? items : 0;
}
// The row of the matrix that item k of a thread of row group g takes.  Only the last item's may lie past the matrix, and the
// item's before it in the instances that serve one row less as well: those take the last row again.
constexpr int linear_tail(int items) { return items > 12 ? 2 : 1; }
__host__ __device__ constexpr int linear_row(int items, int T, int groups, int g, int k) {
    const int row = g + groups * k;
    return k < items - linear_tail(items) || row < T ? row : T - 1;
}
// The largest row that any thread takes (the group of the threads that are left over included), for a check on the host.
constexpr int linear_largest_row(int W, int T) {
    const int items = linear_instance(W, T), groups = linear_groups(W, T), pieces = (T + 3) / 4;
    int most = 0;
    for (int g = 0; g <= (W - 1) / pieces; ++g)
        for (int k = 0; k < items; ++k) {
            const int row = linear_row(items, T, groups, g, k);
            if (row > most) most = row;
        }
    return most;
}

template <typename LG>
struct LinSmem {
    alignas(16) float part[LG::SCRATCH];  // partial sums: [group][STRIDE] forward, [row = (item, group)][RSTRIDE] backward
    // S_n.  Forward: entry v = g + G k at g IPAD + k, as the groups read it; zeros in between.  Backward: in order, zeros
    // from TCAP on, and from TCAP + 8 on the entries of a row's last piece, zero where its neighbour holds them already.
    alignas(16) float vec[2][LG::VEC];
    alignas(16) float wmax[2][16];        // per-wave largest entries of S_n; +inf: the step was not accepted
    alignas(16) float over[2][16], under[2][16];  // comparing runs: per-wave largest D - tol and -(D + tol) of a row (LinMatch)
};

// Four consecutive potentials as they lie in memory (bfloat16 is widened where the piece is used: widening at the load
// would wait for it there).  ALIGNED: the tag count is a multiple of four; otherwise a row starts wherever an element may.
// (Odd counts of bfloat16 tags: 8-byte loads from odd half words take the memory pipeline longer, 3.5 us a step at 201 tags
// where 202 tags take 2.8; the words around the piece with a shift, 12 bytes or 8 + 2 a piece, take 4.4 and more.  Plain loads:
// the non-temporal hint gains nothing on tensors that exceed the memory-side cache, 3.65 against 3.79 us a step at 200 tags,
// and costs a fifth on those that it holds.)
typedef __attribute__((address_space(1))) char GlobalBytes;
#define LCCRF_GLOBAL(T) const __attribute__((address_space(1))) T*
template <typename TIN> struct RawPiece;
template <> struct RawPiece<float> {
    static constexpr int WORDS = 4;
    typedef vec4f type;
    template <bool ALIGNED>
    static __device__ __forceinline__ type load(const GlobalBytes* p) {
        if constexpr (ALIGNED) return *(LCCRF_GLOBAL(vec4f))p;
        else return *(LCCRF_GLOBAL(vec4f_anywhere))p;
    }
    static __device__ __forceinline__ float get(const type& r, int j) { return r[j]; }
};
template <> struct RawPiece<uint16_t> {
    static constexpr int WORDS = 2;
    typedef vec2u type;
    template <bool ALIGNED>
    static __device__ __forceinline__ type load(const GlobalBytes* p) {
        if constexpr (ALIGNED) return *(LCCRF_GLOBAL(vec2u))p;
        else return *(LCCRF_GLOBAL(vec2u_anywhere))p;
    }
    static __device__ __forceinline__ float get(const type& r, int j) {
        return __uint_as_float((j & 1) ? r[j >> 1] & 0xffff0000u : r[j >> 1] << 16);
    }
};

__device__ __forceinline__ float max16(const float* w) {  // of sixteen floats in LDS
    const float4 q0 = *reinterpret_cast<const float4*>(w), q1 = *reinterpret_cast<const float4*>(w + 4);
    const float4 q2 = *reinterpret_cast<const float4*>(w + 8), q3 = *reinterpret_cast<const float4*>(w + 12);
    const float a = max3_raw(max3_raw(q0.x, q0.y, q0.z), q0.w, q1.x), b = max3_raw(max3_raw(q1.y, q1.z, q1.w), q2.x, q2.y);
    const float c = max3_raw(max3_raw(q2.z, q2.w, q3.x), q3.y, q3.z);
    return max3_raw(max3_raw(a, b, c), q3.w, q3.w);
}
// A value that is the same in every lane, said so: it and what follows from it stay in scalar registers.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <typename P>
__device__ __forceinline__ P* uniform(P* p) {
    const unsigned long long v = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    return (P*)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double uniform(double x) {
    const long long v = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ float uniform_f(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }

// What a stretch of log-domain steps returns, out of line: this thread's entry of the vector behind it and its offset.
struct LogStepsResult {
    float v;
    double O;
};

// How many log-domain steps follow a run that came to a step it cannot take: few if it got far (an odd position), sixteen if
// not, and the whole rest once two runs have got less than eight steps far (hard constraints at every position, potentials
// hundreds of bits apart).
struct LogBlocks {
    int poor = 0;
    bool hopeless = false;  // no run is tried
    __device__ __forceinline__ int next(int progress, int rest) {
        poor += progress < 8 ? 1 : 0;
        return hopeless || poor >= 2 ? rest : min(progress >= 16 ? 2 : 16, rest);
    }
};

// Whether a chain will not come far in scaled probabilities because a tag is forbidden everywhere, whose entry is an exact zero in every
// vector: the first of the tags that `suspect` names (each thread one: unreachable where the chain starts, or in the sequence's
// first row), looked up in the matrix the chain takes first, `mat`.  v: the thread's entry of the vector.  Called by the
// whole workgroup.  (What it saves is two runs begun in vain, and the matrices fetched for them: B=1024 N=64 T=45 bfloat16, two such tags,
// log-partition 253 -> 221 us.)
template <typename TIN>
__device__ __forceinline__ bool linear_hopeless(const TIN* mat, int T, bool backward, bool suspect, float v) {
    __shared__ int tag;
    const int tid = threadIdx.x;
    if (!__syncthreads_or(suspect)) return false;
    if (tid == 0) tag = T;
    __syncthreads();
    if (suspect) atomicMin(&tag, tid);
    __syncthreads();
    const int t = tag;
    const bool way = tid < T && v != LCCRF_NEG_INF && Elem<TIN>::get(mat + (backward ? (size_t)t * T + tid : (size_t)tid * T + t)) != LCCRF_NEG_INF;
    return !__syncthreads_or(way);
}

// What a run that compares has found.  Another workgroup has walked the same positions before, from another vector, and left its
// vectors in the rows this run is about to write.  D(t) = this run's logarithm less the one that is there, of one row: where the two
// vectors are multiples of each other D is the same for every tag, and so it is in every row behind, since the steps are
// linear.  A row is alike if one number lies within tol(t) of every D(t), and a tag is an exact zero in both or in neither (a row of
// zeros alone says nothing: what follows it may have any factor, and no path has a finite score).  tol is 2^-20,
// four roundings of a logarithm of one or two bits, and grows with the logarithm as its rounding does.  Non-negative matrices never
// widen such a gap, and all of it but a common factor shrinks from step to step as fast as it came down to tol: a run has found its match
// when rows have been alike for an eighth of the steps that the first of them took and one more, behind which less is left of the gap than storing a row takes.
// At the end of a piece half of that is enough: what is left is then no more than the rounding of the vector that the next piece begins with, and the
// rest of the chain need not be walked again (B=4 N=551 T=145 bfloat16, log-partition, emissions and transitions of deviation two, 418 / 157 us).
// (With a match at the first row that is alike, rows behind it were off by up to 9.1e-7 bits where those of a whole chain are by 5.0e-7:
// 66 tags, the diagonal raised by four.)
struct LinMatch {
    int start = 0;  // step that the run has begun with
    int alike = -1;  // step of the first of the rows that are alike (-1: the last one was not)
    bool hit = false;
    double delta = 0.0;  // what has to be added to the offsets of the rows behind
    __device__ __forceinline__ bool alike_for(int row, int shift) const { return alike >= 0 && row > alike + ((alike - start) >> shift); }
    __device__ __forceinline__ void look(int row, float over, float under, double gap) {
        alike = over > LCCRF_NEG_INF && over + under <= 0.f ? (alike < 0 ? row : alike) : -1;
        hit = alike_for(row, 3);
        delta = gap + 0.5 * (double)(over - under);
    }
};
__device__ __forceinline__ void linear_gap(float x, float old, float& over, float& under) {
    const float d = x - old, tol = 0x1p-20f * fmaxf(1.f, -0.25f * fmaxf(x, -0x1p20f));
    const bool finite = fabsf(d) < __builtin_huge_valf(), zeros = x == LCCRF_NEG_INF && old == LCCRF_NEG_INF;
    over = zeros ? LCCRF_NEG_INF : finite ? d - tol : __builtin_huge_valf();
    under = zeros ? LCCRF_NEG_INF : finite ? -(d + tol) : __builtin_huge_valf();
}

// What a run works on (uniform over the workgroup).  Step s (0 .. n - 1) of the chain takes the matrix of position
// first + s (forward) or first - s (backward).
template <typename TIN, bool BACKWARD>
struct LinJob {
    const TIN* phib;  // potentials of the sequence
    int T, first, n;
    float* uout;   // where the normalised vectors go, [N][T] of the sequence (base-2 logarithms) ...
    double* Oout;  // ... and their offsets, [N]
    __device__ __forceinline__ int matrix(int s) const { return BACKWARD ? first - s : first + s; }
    __device__ __forceinline__ int position(int s) const { return BACKWARD ? first - s : first - 1 + s; }  // of the vector behind s steps
};

// Takes steps from `from` on while they are accepted; returns the steps done in all.  v: thread tid's entry of the
// vector in front of step `from` (base-2 logarithms; -inf from tid = T on), O its offset; on return those of the
// vector behind the last step taken.  The vectors in front of every step taken are stored to uout / Oout; that of the
// last one is not (the caller stores it or goes on from it).  COMPARE: the rows are looked at before they are written, and the
// run ends behind one that matches (v0 and O are then of no use).  Called by the whole workgroup.
template <typename LG, typename TIN, bool ALIGNED, bool BACKWARD, bool COMPARE = false>
__device__ __forceinline__ int linear_run(LinSmem<LG>& ls, const LinJob<TIN, BACKWARD>& job, float& v0, int from, double& O, LinMatch& match) {
    constexpr int ITEMS = LG::ITEMS, Q = LG::Q, TCAP = LG::TCAP;
    using Raw = RawPiece<TIN>;
    // Pieces in flight: as many whole tiles as fit the registers beside E (PH of them, three at most), half or a quarter
    // of a tile of single precision where not even one does.  (bfloat16 with more than six rows: two, with ten or more one; the next one up spills registers
    // inside the loop.  Log-partition, us, one tile more / so: ten rows B=48 N=64 T=195 102.8 / 92.5, B=32 N=256 T=192 373 / 334, B=8 N=9 T=199 27.0 / 24.6;
    // seven and eight B=96 N=48 T=165 63.4 / 62.1, T=172 67.3 / 62.6.  Comparing takes registers of its own: a tile less, B=26 N=329 T=129 single
    // precision 214.7 / 181.8, B=17 N=358 T=172 bfloat16 159.5 / 152.5.)
    constexpr int kRawRegs = Raw::WORDS * ITEMS, kFree = (sizeof(TIN) == 2 ? 86 : 88) - 4 * ITEMS;
    constexpr int kTiles = sizeof(TIN) == 4 || ITEMS <= 6 ? 3 : ITEMS < 10 ? 2 : 1, kMost = COMPARE && kTiles > 1 ? kTiles - 1 : kTiles;
    constexpr bool HALF = kRawRegs > kFree;
    constexpr int PH = HALF ? 1 : kFree / kRawRegs > kMost ? kMost : kFree / kRawRegs;
    constexpr int R = HALF ? (kRawRegs / 2 + 4 * ITEMS > 92 ? ITEMS / 4 : ITEMS / 2) : PH * ITEMS;
    static_assert(!HALF || ITEMS % R == 0, "a whole fraction of a tile");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = job.T;
    const int n = job.n;
    if (from >= n) return from;
    const size_t TT = (size_t)T * T;
    const int Q4 = (T + 3) >> 2, G = linear_groups(LG::W, T);  // threads a row, row groups
    const int g = tid / Q4, cl = tid - g * Q4;    // (g = G: left over, holds zeros of the vector)
    const int c4 = min(4 * cl, T - 4);
    const unsigned voff = (unsigned)(g * T + c4) * (unsigned)sizeof(TIN);
    constexpr int TAIL = linear_tail(ITEMS), BODY = ITEMS - TAIL;  // (the rows of the first BODY items: linear_row(.., k) = g + G k)
    unsigned voff_tail[TAIL];
#pragma unroll
    for (int k = 0; k < TAIL; ++k) voff_tail[k] = (unsigned)(linear_row(ITEMS, T, G, g, BODY + k) * T + c4) * (unsigned)sizeof(TIN);
    const unsigned row_bytes = (unsigned)(uniform(G) * T) * (unsigned)sizeof(TIN);

    typename Raw::type raw[R];
    float e[ITEMS][4];
    // The matrices are requested in the order of the steps: `ahead` is the one that is taken next (past the end the last one again, never
    // used), so that an address is an addition.
    const GlobalBytes* ahead = (const GlobalBytes*)(job.phib + (size_t)job.matrix(from) * TT);
    int ahead_left = n - 1 - from;  // matrices behind it
    const ptrdiff_t stride = (BACKWARD ? -1 : 1) * (ptrdiff_t)(TT * sizeof(TIN));
    const auto advance = [&]() __attribute__((always_inline)) {
        ahead += ahead_left > 0 ? stride : 0;
        --ahead_left;
    };
    // row k of this thread's part of that matrix
    auto fetch = [&](int k) __attribute__((always_inline)) {
        auto row = ahead + (k < BODY ? row_bytes * (unsigned)k : 0u);
        unsigned offset = k < BODY ? voff : voff_tail[k < BODY ? 0 : k - BODY];
        // The base is uniform, in scalar registers (not an address of its own per row, hoisted out of the loop), and the offset is 32 bits
        // wide where it is used: the load adds the two up.
        asm("" : "+s"(row), "+v"(offset));
        return Raw::template load<ALIGNED>(row + offset);
    };
    // The largest entry, and whether every entry is an exact zero or within 2^-120 of it: held without loss, whatever its
    // products lose is below 2^-126.
    const float top = xor_max<1, 64>(v0);
    if (lane == 0) ls.wmax[0][wave] = top;
    if (tid >= LG::WAVES && tid < 16) ls.wmax[0][tid] = LCCRF_NEG_INF;
    __syncthreads();
    const float d = uniform_f(finite_or_zero(max16(ls.wmax[0])));
    const bool fine = v0 == LCCRF_NEG_INF || v0 - d >= -120.f;
    if (lane == 0) ls.wmax[1][wave] = __all(fine) ? 0.f : 1.f;
    if (tid >= LG::WAVES && tid < 16) ls.wmax[1][tid] = 0.f;
    __syncthreads();
    if (uniform_f(max16(ls.wmax[1])) != 0.f) return from;

    // E of the next step from the ring, shift c; every piece that is used up is requested again for what follows
    auto prepare = [&](int slot, int shift) __attribute__((always_inline)) {
        const float c = (float)shift;
        if constexpr (!HALF) advance();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int r = HALF ? k % R : slot * ITEMS + k;
#pragma unroll
            for (int j = 0; j < 4; ++j) e[k][j] = ex2(__builtin_fmaf(Raw::get(raw[r], j), kLog2e, -c));
            asm volatile("" : "+v"(e[k][0]), "+v"(e[k][1]), "+v"(e[k][2]), "+v"(e[k][3]));  // (here: not sunk behind the barrier to where they are used)
            if constexpr (HALF) {
                if (k + R == ITEMS) advance();
                raw[r] = fetch(k + R < ITEMS ? k + R : k + R - ITEMS);
            } else {
                raw[r] = fetch(k);
            }
            if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // (keeps the new loads from being hoisted over the old values' use)
        }
    };

#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!HALF && r > 0 && r % ITEMS == 0) advance();
        raw[r] = fetch(r % ITEMS);
    }

    // where the entries of the vector lie, for the thread that publishes (`mine`) or stores (tid) one
    const auto slot_of = [&](int v) { return BACKWARD ? v : v % G * LG::IPAD + v / G; };
    const int mine = min(tid / Q, T - 1), vmine = slot_of(mine), vstore = slot_of(min(tid, T - 1));
    const bool stores = 64 * wave < T;
    const unsigned store_offset = 4u * (unsigned)min(tid, T - 1);
    const int vcopy = BACKWARD && mine >= 4 * (Q4 - 1) ? TCAP + 8 + mine - (T - 4) : vmine;  // (or the same place again)
    for (int k = tid; k < 2 * LG::VEC; k += LG::W) (&ls.vec[0][0])[k] = 0.f;
    for (int k = tid; k < LG::SCRATCH; k += LG::W) ls.part[k] = 0.f;
    __syncthreads();
    if (tid < T) {
        const float x = ex2(v0 - d);
        ls.vec[0][slot_of(tid)] = x;
        if (BACKWARD && tid >= 4 * (Q4 - 1)) ls.vec[0][TCAP + 8 + tid - (T - 4)] = x;
    }
    if (tid < 16) ls.wmax[1][tid] = LCCRF_NEG_INF;
    __syncthreads();
    // where this thread finds the entries of its rows (forward) or columns (backward), and leaves its partial sums
    const int vfrom = !BACKWARD ? g * LG::IPAD : g == G ? TCAP : cl == Q4 - 1 ? TCAP + 8 : 4 * cl;
    const int pslot = BACKWARD ? g * LG::RSTRIDE + cl : g * LG::STRIDE + 4 * cl;
    // merging: this thread adds up part tid % Q of column or row `mine` (forward, the columns of the piece that was moved
    // back are counted from its start)
    const int mslot = BACKWARD ? (mine / G * LG::GMAX + mine % G) * LG::RSTRIDE + (tid % Q) * LG::ROW4
                               : (tid % Q) * LG::STRIDE + (mine < 4 * (Q4 - 1) ? mine : 4 * (Q4 - 1) + mine - (T - 4));
    // The first matrix's shift: the largest of its entries plus that of the vector it meets, among the pieces at hand, which
    // is what the first step grows by (up to the logarithm of the tag count).
    float big = LCCRF_NEG_INF;
#pragma unroll
    for (int k = 0; k < (R < ITEMS ? R : ITEMS); ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            big = fmaxf(big, __builtin_fmaf(Raw::get(raw[k], j), kLog2e, lg2(ls.vec[0][vfrom + (BACKWARD ? j : k)])));
    big = xor_max<1, 64>(big);
    if (lane == 0) ls.wmax[1][wave] = big;
    __syncthreads();
    // (shifts and exponents are integers in scalar registers; far inside the range of an int)
    big = max16(ls.wmax[1]);
    int c_cur = uniform((int)fminf(fmaxf(ceilf(finite_or_zero(big)), -0x1p20f), 0x1p20f)), c_last = c_cur + kLinearHead - 1;
    __syncthreads();
    if (tid < 32) ls.wmax[tid >> 4][tid & 15] = tid == 0 ? 1.f : 0.f;
    if (COMPARE && tid < 32) ls.over[tid >> 4][tid & 15] = ls.under[tid >> 4][tid & 15] = tid == 0 ? __builtin_huge_valf() : LCCRF_NEG_INF;  // (waves that store nothing leave theirs)
    // Comparing: what is in the row of the step to come, requested a step ahead of its use and ahead of that step's matrix.
    float old = 0.f;
    double oldO = 0.0, gap = 0.0;
    const auto look = [&](int s) __attribute__((always_inline)) {
        auto row = (const GlobalBytes*)(job.uout + (size_t)job.position(s < n ? s : n - 1) * T);
        unsigned offset = store_offset;
        asm("" : "+s"(row), "+v"(offset));
        old = *(LCCRF_GLOBAL(float))(row + offset);
        oldO = job.Oout[job.position(s < n ? s : n - 1)];
    };
    if constexpr (COMPARE) look(from);
    prepare(0, c_cur);
    __syncthreads();

    int done = from, buf = 0;
    const double O0 = uniform(O + (double)d);
    long long Oi = 0, Oi_last = 0;  // offset of the vector in vec[buf] and of the one before it, less O0
    float M = 1.f;  // the largest entry of the vector in vec[buf]
    // Whether there is a step to take.  (One condition and one way out of the loop below: where a path without loads joins one with them
    // the compiler waits for all of them, and a step took what memory takes.)
    const auto more = [&]() __attribute__((always_inline)) -> bool {
        if constexpr (COMPARE) {
            const float over = uniform_f(max16(ls.over[buf])), under = uniform_f(max16(ls.under[buf]));
            if (done > from) match.look(done - 1, over, under, gap);
        }
        M = uniform_f(max16(ls.wmax[buf]));
        return (M <= 0x1p60f) & (M >= 0x1p-30f) & (done != n) & !(COMPARE && match.hit);
    };
    const auto step = [&](int slot_next) __attribute__((always_inline)) {
        const int k = uniform(__builtin_amdgcn_frexp_expf(M));
        // (c_last + k - kLinearHead: what the last step grew by.  In front of the first step c_last is such that this is what the
        // first one will grow by, the exponent of its vector being 1.)
        const int c_next = max(min(c_last + k, 1 << 20), -(1 << 20)) - kLinearHead;
        const float* vin = &ls.vec[buf][vfrom];
        if constexpr (!BACKWARD) {
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r4 = 0; r4 < ITEMS; r4 += 4) {
                const float4 v4 = *reinterpret_cast<const float4*>(vin + r4);
                const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
                for (int r = r4; r < (r4 + 4 < ITEMS ? r4 + 4 : ITEMS); ++r)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[j] = __builtin_fmaf(e[r][j], v[r - r4], acc[j]);
            }
            *reinterpret_cast<float4*>(&ls.part[pslot]) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        } else {
            const float4 v = *reinterpret_cast<const float4*>(vin);
#pragma unroll
            for (int r = 0; r < ITEMS; ++r)
                ls.part[pslot + r * LG::GMAX * LG::RSTRIDE] = __builtin_fmaf(e[r][0], v.x, e[r][1] * v.y) + __builtin_fmaf(e[r][2], v.z, e[r][3] * v.w);
        }
        // the vector in front of this step is final: store it (off the dependent path), its largest entry brought below 1:
        // the closer the logarithms are to zero, the less their rounding takes.  (By the first waves, a tag a thread.)
        if (stores) {
            auto out = (__attribute__((address_space(1))) char*)(job.uout + (size_t)job.position(done) * T);
            unsigned offset = store_offset;
            asm("" : "+s"(out), "+v"(offset));  // (as above)
            const float x = lg2(__builtin_amdgcn_ldexpf(ls.vec[buf][vstore], -k));
            if constexpr (COMPARE) {
                float over, under;
                linear_gap(x, old, over, under);
                over = xor_max<1, 64>(over);
                under = xor_max<1, 64>(under);
                if (lane == 0) {
                    ls.over[buf ^ 1][wave] = over;
                    ls.under[buf ^ 1][wave] = under;
                }
                gap = O0 + (double)(Oi + k) - oldO;
                look(done + 1);
            }
            *(__attribute__((address_space(1))) float*)(out + offset) = x;
        }
        if (tid == 0) job.Oout[job.position(done)] = O0 + (double)(Oi + k);
        __syncthreads();
        const float* part = &ls.part[mslot];
        float s;
        if constexpr (!BACKWARD) {
            s = part[0];
#pragma unroll
            for (int p = 1; p < LG::PARTS; ++p) s += part[p * Q * LG::STRIDE];
        } else {
            float4 x = *reinterpret_cast<const float4*>(part);
#pragma unroll
            for (int p = 4; p < LG::ROW4; p += 4) {
                const float4 y = *reinterpret_cast<const float4*>(part + p);
                x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
            }
            s = (x.x + x.y) + (x.z + x.w);
        }
        s = __builtin_amdgcn_ldexpf(xor_sum<1, Q>(s), kLinearHead - k);
        ls.vec[buf ^ 1][vmine] = s;
        if constexpr (BACKWARD) ls.vec[buf ^ 1][vcopy] = s;
        const float m = __all(sum_in_range(s)) ? xor_max<1, 64>(s) : __builtin_huge_valf();
        if (lane == 0) ls.wmax[buf ^ 1][wave] = m;
        Oi_last = Oi;
        Oi += k - kLinearHead + c_cur;
        c_last = c_cur;
        c_cur = c_next;
        prepare(slot_next, c_next);
        buf ^= 1;
        ++done;
        __syncthreads();
    };
    for (;;) {
        if (!more()) break;
        step(PH > 1 ? 1 : 0);
        if constexpr (PH > 1) {
            if (!more()) break;
            step(PH > 2 ? 2 : 0);
        }
        if constexpr (PH > 2) {
            if (!more()) break;
            step(0);
        }
    }
    if (COMPARE && done == n && M <= 0x1p60f) match.hit = match.hit || match.alike_for(done - 1, 4);
    if (COMPARE && match.hit) return done;
    if (!(M <= 0x1p60f)) {  // the vector in front of the rejected step is still in the other buffer
        buf ^= 1;
        --done;
        Oi = Oi_last;
    }
    if (done == from) return from;
    const int k = uniform(__builtin_amdgcn_frexp_expf(uniform_f(max16(ls.wmax[buf]))));
    if (tid < T) v0 = lg2(__builtin_amdgcn_ldexpf(ls.vec[buf][slot_of(tid)], -k));
    O = O0 + (double)(Oi + k);
    __syncthreads();  // (the shared state may be used for something else now)
    return done;
}

}  // namespace lccrf
