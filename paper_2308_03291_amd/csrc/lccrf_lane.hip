// Sum-product chains for 8 .. 64 tags with the recursion taken off the streaming work: one wave of a
// workgroup runs the chain, the others stream the potentials.
//
// The sequential forward recursion (section "Sequence Tagging": O(m^2 n) work, n dependent steps) is
// what bounds batches that do not fill the chip: a step of the kernels in lccrf_wave.hip / lccrf_chain.hip
// costs 1400 to 2000 cycles, most of them the exponentials, the logarithm and the lane reductions of a
// log-sum-exp that all sit on the chain of dependent instructions.  Here a step of the chain is a plain
// vector-matrix product in the linear domain,
//     V'(u) = sum_v V(v) E(u, v),      E = 2^(phi log2 e - m),  m = ceil(max of the matrix),
// by ONE wave with lane u holding V(u): sixteen fused multiply-adds per block of sixteen source tags,
// the source values arriving by DPP row rotation (v_fmac_f32_dpp row_ror:n), the blocks by the gfx950
// permlane swaps; no exponential, no logarithm and no reduction tree on the dependent path.  The matrix
// entries a lane needs, in the order its rotations consume them, wait in LDS: the other waves of the
// workgroup ("producers") load the potentials (coalesced 16-byte loads, the next matrix of a wave in flight
// while it works on the current one), exponentiate them and scatter them into a ring of LDS slots in that
// rotated order.  A producer then waits for the chain to accept the step its matrix belongs to and does the
// step's stores: in the first pass the resulting vector (base-2 logarithms plus a double offset, the format of
// the other sum-product kernels, so either pass may be combined with theirs), in the second pass the marginals
// mu = V(s) E(s,t) G(t) of that position from the matrix it still holds in registers (coalesced 16-byte
// stores).  The waves meet only through words in LDS (ready / done / stop), never at a barrier.
//
// Vectors are kept as V 2^O with O = O0 + an integer: every matrix is shifted by an integer m, and after every
// step the vector is rescaled by the power of two that gives tag 0's entry the exponent kLaneHead (any accepted entry
// serves as the reference; lane 0's comes without a reduction).  A step is accepted only if every sum lies in
// [2^-60, 2^60] (kSumLo, kSumHi): then whatever underflowed in it (an entry below 2^-126) is below 2^-46 of the sum it belongs to,
// times what the heaviest tag has over tag 0, for every entry separately, so the loss does not compound from step to step.  First
// passes over dense potentials also accept sums that are exact zeros (a tag that is forbidden there or everywhere), once one has
// occurred: the producers say of every matrix whether its entries are all above 2^-80 or exact zeros, so that a zero can be told from
// an underflow.  A step that is not accepted (entries of one matrix hundreds of bits apart) is taken by the chain wave
// itself in the log domain, straight from memory, every log-sum-exp shifted by its own maximum, stores and
// marginals included; the fast path resumes as soon as the vector is one that scaled single precision holds
// faithfully again.  Where such steps are frequent (second passes and structured potentials: eight in a row), or if a producer does
// not deliver within the poll limit, the chain stays in the log domain for the rest of its half.  In a first pass over dense
// potentials the producers then hand on logarithms (kLaneRaw); otherwise they see `stop` and leave.
//
// What that costs (us, so / the scan or one-wave kernels that log-probability and sampling took before these; in parentheses every
// log-domain step read from memory by the chain wave): log-probability, N=256 B=128 T=32 with a tag forbidden everywhere 51 / 87 (286),
// N=128 T=48 40 / 97 (196); independent normal potentials, N=128 B=128, T=32 deviation 12 33 / 52 (46), 16 63 / 51 (141), 20 64 / 51 (147),
// T=48 12 48 / 63 (78), 20 113 / 87 (212), T=64 B=64 12 54 / 66 (81), 20 182 / 87 (286); sampling, T=32 N=256 with a forbidden tag 120 / 163
// (551), T=32 N=128 12 66 / 94 (82), 20 131 / 99 (256), T=16 N=64 12 34 / 35 (37), 20 66 / 37 (88).  A log-domain step takes
// 0.5 us (32 tags) from a producer's logarithms, 1.6 from memory; going over costs eight to sixteen of those.
#include "lccrf_chain_args.h"
#include "lccrf_device.h"
#include "lccrf_launch.h"
#include "lccrf_lds_flags.h"
#include "lccrf_linear.h"
#include "lccrf_rotate.h"

#include <cstddef>
#include <type_traits>

namespace lccrf {

// Waves of a workgroup: wave 0 runs the chain (at raised priority), the others are producers.  Up to 32 tags a
// producer needs few registers and eleven of them keep the second pass fed (B=128 N=256 T=32: second pass
// 51.8 -> 47.9 us against seven); above, seven is what the register file holds at two waves a SIMD.
constexpr int lane_waves(int nblk) { return nblk <= 2 ? 12 : 8; }
constexpr int kLaneMaxProducers = 11;
constexpr int kLaneHead = 15;           // what the entries of a vector are held above their value, in powers of two: tag 0's is
                                        // brought into [1/2, 1), sums far below the largest stay in range (see lane_up)
constexpr int kLaneVecRing = 16;        // published vectors kept (the chain leads a producer by fewer than that, see `arrived`)
static_assert(kLaneVecRing > kLaneMaxProducers + 1, "a vector is not replaced while its producer may read it");

template <int NBLK>
struct LaneShape {
    static_assert(NBLK >= 1 && NBLK <= 4, "one to four blocks of sixteen tags");
    static constexpr int U = 16 * NBLK;  // padded tag count
    static constexpr int RS = U + 4;     // floats per LDS row: 16-byte reads of consecutive rows hit distinct banks
    static constexpr int RING = 8;       // LDS slots for matrices (a power of two: slot = step & 7)
    static constexpr int NG = NBLK * NBLK;  // groups of four entries a producer lane holds of one matrix
    static constexpr int PF = 2;  // matrices per producer wave: one in hand, one in flight
};

template <int NBLK>
struct LaneShared {
    using S = LaneShape<NBLK>;
    float E[S::RING][S::U + 1][S::RS];  // E[slot][u][16 b + n] = the entry lane u multiplies with rotation n of block b
                                        // (row U stays zero: read by the lanes of the chain wave that hold no tag)
    float V[kLaneVecRing][64];      // V_q, the vector that enters step q, at [q % kLaneVecRing]
    int VOi[kLaneVecRing];          // twice its offset less O0 (the shifts and rescales so far: an integer), plus 1
                                    // if the step that produced it was taken in the log domain by the chain wave
    double O0;                      // offset of V_0
    float G[kLaneMaxProducers][64]; // per producer wave: the factors of the stored vector of the other chain
    unsigned long long ready[S::RING];  // once the matrix of step q sits in slot q % RING: q + 1 in the high word, twice
                                        // the matrix's shift (an integer) in the low word, plus 1 if no entry but exact
                                        // zeros lies below 2^-80: one read brings all
    int raw;                        // from this step on producers hand on the logarithms themselves (INT_MAX: from none)
    int done;                       // steps the chain has accepted
    int stop;                       // first step of the log-domain tail (INT_MAX: none)
};

// e[n] += a of the lane n places to the left in its row of sixteen
__device__ __forceinline__ void add_rotations(float (&e)[16], float a) {
    e[0] += a;
#define LCCRF_AR(N) e[N] += dpp<0x120 + N>(a)
    LCCRF_AR(1); LCCRF_AR(2); LCCRF_AR(3); LCCRF_AR(4); LCCRF_AR(5); LCCRF_AR(6); LCCRF_AR(7); LCCRF_AR(8);
    LCCRF_AR(9); LCCRF_AR(10); LCCRF_AR(11); LCCRF_AR(12); LCCRF_AR(13); LCCRF_AR(14); LCCRF_AR(15);
#undef LCCRF_AR
}

__device__ __forceinline__ float lane_value(float x, int src) {  // src uniform over the wave
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), src));
}

__device__ __forceinline__ float min3_raw(float a, float b, float c) {
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

constexpr int kLaneRaw = (int)0x80000000;  // in place of a matrix's shift: its entries are base-2 logarithms
// Whether the producers of this instantiation ever hand on such matrices: in first passes over dense potentials.
template <typename TIN, bool AL>
struct LaneSource;
template <typename TIN, bool AL, bool PASS2>
constexpr bool lane_takes_raw() { return !PASS2 && !LaneSource<TIN, AL>::kStruct; }
constexpr bool lane_hands_raw(int nblk) { return nblk <= 3; }  // (above 48 tags the producers have no registers for it)

// Between an entry's logarithm, near zero where it counts, and the entry as it is held.
__device__ __forceinline__ float lane_up(float l) { return __builtin_amdgcn_ldexpf(ex2(l), kLaneHead); }
__device__ __forceinline__ float lane_log(float v) { return lg2(__builtin_amdgcn_ldexpf(v, -kLaneHead)); }

// What a chain is working on (uniform over the workgroup).
struct LaneJob {
    int b, dir, L, h;
    int first, sdir, count;  // step q consumes the matrix of position first + q sdir
};

// Where the potentials of sequence b come from: a dense tensor of TIN, or (StructF) trans[s][t] + emit[b][i][t],
// the single-precision sum the materialised tensor would hold.  at(): one potential; piece(): the four of row s,
// columns t0 .. t0 + 3 (flat offset off = s T + t0), `fixed` being what fixed_part() returned for that piece.
// AL: the tag count is a multiple of four and every piece lies on a 16-byte boundary.  Otherwise the rows start at any
// multiple of the element size: the last piece of a row is moved back to end where the row ends (it overlaps the
// piece before it; the entries both hold are the same numbers, written to the same places), and a piece is loaded and
// stored through types that promise the compiler no more than the element's alignment.
struct StructF {};
template <bool AL, typename E>
__device__ __forceinline__ void lane_load4(const E* p, float (&o)[4]) {
    if constexpr (AL) Elem<E>::get4(p, o);
    else Elem<E>::get4_anywhere(p, o);
}
template <bool AL>
__device__ __forceinline__ void lane_store4(float* p, float a, float b, float c, float d) {
    if constexpr (AL) {
        *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
    } else {
        store4_anywhere(p, a, b, c, d);
    }
}
template <typename TIN, bool AL>
struct LaneSource {
    static constexpr bool kStruct = false;
    const TIN* phib;
    size_t TT;
    int T;
    __device__ __forceinline__ LaneSource(const ChainArgs& a, int b)
        : phib(static_cast<const TIN*>(a.phi) + (size_t)b * a.N * a.T * a.T), TT((size_t)a.T * a.T), T(a.T) {}
    __device__ __forceinline__ float at(int i, int s, int t) const { return Elem<TIN>::get(phib + (size_t)i * TT + (size_t)s * T + t); }
    __device__ __forceinline__ void fixed_part(int, int, float (&f)[4]) const { f[0] = f[1] = f[2] = f[3] = 0.f; }
    __device__ __forceinline__ void piece(int i, int off, int, const float (&)[4], float (&o)[4]) const {
        lane_load4<AL>(phib + (size_t)i * TT + off, o);
    }
};
template <bool AL>
struct LaneSource<StructF, AL> {
    static constexpr bool kStruct = true;
    const float* emb;
    const float* trans;
    int T;
    __device__ __forceinline__ LaneSource(const ChainArgs& a, int b) : emb(a.emit + (size_t)b * a.N * a.T), trans(a.trans), T(a.T) {}
    __device__ __forceinline__ float at(int i, int s, int t) const { return trans[(size_t)s * T + t] + emb[(size_t)i * T + t]; }
    __device__ __forceinline__ void fixed_part(int off, int, float (&f)[4]) const { lane_load4<AL>(trans + off, f); }
    __device__ __forceinline__ void piece(int i, int, int t0, const float (&f)[4], float (&o)[4]) const {
        float e[4];
        lane_load4<AL>(emb + (size_t)i * T + t0, e);
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = f[k] + e[k];
    }
};

// What ends a log-domain step of a first pass: r, the logarithms of the new vector (this lane's tag u; -inf without a tag), less an
// integer shift, which is returned, into lv, and the stores of its position (by the lanes for which `mine`).
__device__ __forceinline__ int lane_log_end(const ChainArgs& a, const LaneJob& jb, int i, float r, int u, bool mine, float& lv, double O,
                                            int meet_only) {
    const int T = a.T;
    const float d = fminf(fmaxf(ceilf(finite_or_zero(xor_max<1, 64>(r))), -0x1p30f), 0x1p30f);  // (clamped as in lane_log_step)
    lv = r - d;
    const int pos = jb.dir == 0 ? i : i - 1;
    if (!meet_only || pos == jb.h) {
        const size_t at = (size_t)jb.b * a.N + pos;
        if (mine && u < T) (jb.dir == 0 ? a.ua : a.ub)[at * T + u] = lv;
        if ((threadIdx.x & 63) == 0) (jb.dir == 0 ? a.Oa : a.Ob)[at] = O + (double)d;
    }
    return __builtin_amdgcn_readfirstlane((int)d);
}

// One position in the log domain by the chain wave alone, straight from memory: every log-sum-exp shifted by
// its own maximum.  lv: the vector that enters step q, base-2 logarithms, lane = tag (-inf from T on), O its
// offset; on return lv is the result less the integer shift that is returned (its maximum then lies in (-1, 0]).
// Writes what the step owes to memory: the marginals of its position (second pass), the stored vector (first).
template <typename TIN, bool AL, bool PASS2>
__device__ __forceinline__ int lane_log_step(const ChainArgs& a, const LaneJob& jb, int q, float& lv, double O,
                                             double lz2, int meet_only) {
    const int lane = threadIdx.x & 63, T = a.T, N = a.N, b = jb.b;
    const size_t TT = (size_t)T * T;
    const LaneSource<TIN, AL> src(a, b);
    const size_t vb = (size_t)b * N;
    const int i = jb.first + q * jb.sdir;
    const bool on = lane < T;
    const int me = on ? lane : 0;
    float other = LCCRF_NEG_INF, K = 0.f;
    float* mu_i = nullptr;
    if (PASS2) {
        // forward: beta_i(t) and its offset; backward: alpha_{i-1}(s) and its offset
        const size_t vp = jb.dir == 0 ? vb + i : vb + i - 1;
        other = on ? (jb.dir == 0 ? a.ub : a.ua)[vp * T + me] : LCCRF_NEG_INF;
        K = (float)(O + (jb.dir == 0 ? a.Ob : a.Oa)[vp] - lz2);
        mu_i = a.mu + (vb + i) * TT;
    }
    float mx = LCCRF_NEG_INF;
    for (int v = 0; v < T; ++v) {
        const float x = lane_value(lv, v) + (jb.dir == 0 ? src.at(i, v, me) : src.at(i, me, v)) * kLog2e;
        mx = fmaxf(mx, x);
    }
    const float g = finite_or_zero(mx);
    float sum = 0.f;
    for (int v = 0; v < T; ++v) {
        const float x = lane_value(lv, v) + (jb.dir == 0 ? src.at(i, v, me) : src.at(i, me, v)) * kLog2e;
        sum += ex2(x - g);
        if (PASS2 && on) {
            const float m = ex2(x + other + K);
            if (jb.dir == 0) mu_i[(size_t)v * T + lane] = m;
            else mu_i[(size_t)lane * T + v] = m;
        }
    }
    const float r = on ? mx + lg2(sum) : LCCRF_NEG_INF;
    // an integer shift, clamped far inside the range of an int: the offsets stay O0 plus an integer
    const float d = fminf(fmaxf(ceilf(finite_or_zero(xor_max<1, 64>(r))), -0x1p30f), 0x1p30f);
    lv = r - d;
    if (!PASS2) {
        const int pos = jb.dir == 0 ? i : i - 1;
        if (!meet_only || pos == jb.h) {
            if (on) (jb.dir == 0 ? a.ua : a.ub)[(vb + pos) * T + lane] = lv;
            if (lane == 0) (jb.dir == 0 ? a.Oa : a.Ob)[vb + pos] = O + (double)d;
        }
    }
    return __builtin_amdgcn_readfirstlane((int)d);  // (the same in every lane; said so, it stays in a scalar register)
}

// The log-domain tail: steps q0 .. count - 1 of the job.  Returns with lv / O the last vector.
template <typename TIN, bool AL, bool PASS2>
__device__ __forceinline__ void lane_log_tail(const ChainArgs& a, const LaneJob& jb, int q0, float& lv, double& O,
                                              double lz2, int meet_only) {
    for (int q = q0; q < jb.count; ++q) O += (double)lane_log_step<TIN, AL, PASS2>(a, jb, q, lv, O, lz2, meet_only);
}

// The same of a first pass over dense potentials.  Up to 32 tags the lanes hold the vector C times, each copy taking the C-th part of
// the sources, whose logarithms come through LDS (`buf`, which only this wave uses).  All of a lane's potentials are requested
// before the first is used, one trip to memory a step.  A lane's P sources are `start` + 4 p + k, or for C = 1 min(4 p, T - 4) + k: the last
// ones are moved back to end with the matrix, so that no load leaves it, and what is then held twice is left out.
template <int NBLK, typename TIN, bool AL>
__device__ __forceinline__ int lane_log_dense(const ChainArgs& a, const LaneJob& jb, float* buf, int q, float& lv, double O, int meet_only) {
    constexpr int C = NBLK == 1 ? 4 : NBLK == 2 ? 2 : 1, P = LaneShape<NBLK>::U / C, SPAN = 64 / C;
    const int lane = threadIdx.x & 63, N = a.N;
    int T = a.T;
    asm volatile("" : "+s"(T));  // (nothing that follows from it is kept in registers around the steps that are not taken here)
    const int u = lane % SPAN, c = lane / SPAN;
    const bool on = u < T;
    const int me = on ? u : 0;
    const int start = C == 1 ? 0 : min(c * P, T - P), skip = c * P - start;  // (C > 1: T >= P)
    const size_t vb = (size_t)jb.b * N;
    const int i = jb.first + q * jb.sdir;
    if (lane < SPAN) buf[lane] = lv;
    __builtin_amdgcn_wave_barrier();
    auto mat = (const GlobalBytes*)(static_cast<const TIN*>(a.phi) + (vb + i) * T * T);
    float y[P];
    if (jb.dir == 0) {
        const unsigned voff = (unsigned)(start * T + me) * (unsigned)sizeof(TIN);
#pragma unroll
        for (int p = 0; p < P / 4; ++p) {
            auto at = mat + (unsigned)((C == 1 ? min(4 * p, T - 4) : 4 * p) * T) * (unsigned)sizeof(TIN);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                asm volatile("" : "+s"(at));
                const TIN x = *(LCCRF_GLOBAL(TIN))(at + voff);
                y[4 * p + k] = Elem<TIN>::get(&x);
                at += (unsigned)T * (unsigned)sizeof(TIN);
            }
        }
    } else {
        const unsigned voff = (unsigned)(me * T + start) * (unsigned)sizeof(TIN);
#pragma unroll
        for (int p = 0; p < P / 4; ++p) {
            const auto x = RawPiece<TIN>::template load<AL>(mat + (unsigned)(C == 1 ? min(4 * p, T - 4) : 4 * p) * (unsigned)sizeof(TIN) + voff);
#pragma unroll
            for (int k = 0; k < 4; ++k) y[4 * p + k] = RawPiece<TIN>::get(x, k);
        }
    }
    float from[C > 1 ? P : 1];
    if constexpr (C > 1) {  // (all of them requested before one is waited for: left to the compiler it was a trip to LDS for every pair in the
                            // one build and not in the other, log-probability B=128 N=128 T=32 deviation 16 64.5 and 62.0 us; so 61.0)
#pragma unroll
        for (int p = 0; p < P; ++p) from[p] = buf[start + p];
        __builtin_amdgcn_sched_barrier(0);
    }
    float mx = LCCRF_NEG_INF;
#pragma unroll
    for (int p = 0; p < P / 4; ++p)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int s = C == 1 ? min(4 * p, T - 4) : 4 * p;
            const float x = (C > 1 ? from[C > 1 ? 4 * p + k : 0] : buf[start + s + k]) + y[4 * p + k] * kLog2e;
            y[4 * p + k] = (C == 1 ? s + k >= 4 * p : s + k >= skip) ? x : LCCRF_NEG_INF;
            mx = fmaxf(mx, y[4 * p + k]);
        }
    mx = xor_max<SPAN, 64>(mx);
    const float g = finite_or_zero(mx);
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < P; ++j) part[j & 3] += ex2(y[j] - g);
    const float sum = xor_sum<SPAN, 64>((part[0] + part[1]) + (part[2] + part[3]));
    return lane_log_end(a, jb, i, on ? mx + lg2(sum) : LCCRF_NEG_INF, u, c == 0, lv, O, meet_only);
}

// The chain wave.
template <int NBLK, typename TIN, bool AL, bool PASS2>
__device__ __forceinline__ void lane_chain_wave(const ChainArgs& a, const LaneJob& jb, LaneShared<NBLK>& sh, double lz2,
                                                bool feasible, int meet_only, int poll_limit) {
    using S = LaneShape<NBLK>;
    const int lane = threadIdx.x & 63, T = a.T, N = a.N, b = jb.b;
    const size_t TT = (size_t)T * T;
    const size_t vb = (size_t)b * N;
    // Up to 32 tags the 64 lanes hold the vector twice and each copy sums over one block of sixteen source
    // tags (half the products a step; the halves meet through one permlane swap); above, lane = tag.
    constexpr bool kSplit = NBLK == 2;
    const int u = kSplit ? (lane & 31) : lane;  // the tag of this lane
    const int copy = kSplit ? (lane >> 5) : 0;
    bool on = u < T;
    const int me = on ? u : 0;
    const int urow = u < S::U ? (u < T ? u : S::U) : S::U;  // its row of the matrices in LDS (row U: zeros)
    // the vector that enters step 0
    float lv;  // base-2 logarithm, used for the stores of the first pass and by the tail
    double O = 0.0;
    if (!PASS2) {
        if (jb.dir == 0) {
            const float x = on ? LaneSource<TIN, AL>(a, b).at(0, 0, me) * kLog2e : LCCRF_NEG_INF;  // row 0 of the first matrix
            const float d = ceilf(finite_or_zero(xor_max<1, 64>(x)));
            lv = x - d;
            O = (double)d;
        } else {
            lv = on ? 0.f : LCCRF_NEG_INF;
        }
        const int pos = jb.dir == 0 ? 0 : jb.L - 1;
        if (!meet_only || pos == jb.h) {
            if (on && copy == 0) (jb.dir == 0 ? a.ua : a.ub)[(vb + pos) * T + u] = lv;
            if (lane == 0) (jb.dir == 0 ? a.Oa : a.Ob)[vb + pos] = O;
        }
    } else {
        lv = on ? (jb.dir == 0 ? a.ua : a.ub)[(vb + jb.h) * T + me] : LCCRF_NEG_INF;
        O = (jb.dir == 0 ? a.Oa : a.Ob)[vb + jb.h];
    }
    float V = lane_up(lv);  // 0 for lanes past T
    const double O0 = O;
    int Oi = 0;  // O = O0 + Oi: the shifts of the matrices and the rescales so far
    if (copy == 0) sh.V[0][u] = V;
    if (lane == 0) {
        sh.VOi[0] = 0;
        sh.O0 = O0;
    }
    const unsigned long long onmask = __builtin_amdgcn_ballot_w64(on);
    unsigned q = 0;
    const unsigned count = (unsigned)jb.count;
    bool tail = false;
    // The vector in logarithms (carried: they are the ones that count), where scaled single precision does not hold it: a vector the
    // chain starts from with entries further apart than its exponents reach, and what the log-domain steps leave last.
    // (An entry that has vanished may be the only one that a later position leaves a path through.)
    bool carried = __builtin_amdgcn_ballot_w64(on && !(lv == LCCRF_NEG_INF || fabsf(lv) <= 110.f)) != 0;
    float lv_carry = lane < T ? lv : LCCRF_NEG_INF;
    // The matrix of a step: the entries of this lane in the order its rotations consume them, and the shift.
    constexpr int NB = kSplit ? 1 : NBLK;  // blocks of sixteen source tags a lane sums over
    struct Tile {
        float e[NB][16];
        int m;
    };
    const auto read_entries = [&](unsigned step, Tile& t) {
        const unsigned slot = step % S::RING;
#pragma unroll
        for (int bk = 0; bk < NB; ++bk)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 v = *reinterpret_cast<const float4*>(&sh.E[slot][urow][16 * (kSplit ? copy : bk) + 4 * g]);
                t.e[bk][4 * g] = v.x; t.e[bk][4 * g + 1] = v.y; t.e[bk][4 * g + 2] = v.z; t.e[bk][4 * g + 3] = v.w;
            }
    };
    const auto read_tile = [&](unsigned step, Tile& t, unsigned long long word) {
        t.m = __builtin_amdgcn_readfirstlane((int)(unsigned)word);
        read_entries(step, t);
    };
    // Waits for the matrix of `step` (bounded); false: it did not come.  No step is taken without, in the log domain neither, unless the
    // producers are given up: the producer of step q has done with q's vector and offset in their ring once it delivers its
    // next matrix, so the chain leads it by no more steps than there are producers.
    const auto arrived = [&](unsigned step, unsigned long long& word) -> bool {
        int spins = 0;
        while ((unsigned)__builtin_amdgcn_readfirstlane((int)((word = lds_load_acquire(&sh.ready[step % S::RING])) >> 32)) < step + 1)
            if (++spins > poll_limit) return false;
        return true;
    };
    // ... and reads it
    const auto fetch = [&](unsigned step, Tile& t) -> bool {
        unsigned long long word;
        if (!arrived(step, word)) return false;
        read_tile(step, t, word);
        return true;
    };
    const auto blocks_of = [&](float x, float (&Ab)[4]) __attribute__((always_inline)) { rotation_blocks<NBLK>(x, copy, Ab); };
    // Steps that the fast path does not accept (a sum out of range: entries of one matrix hundreds of bits
    // apart, or a hard zero) are taken in the log domain by this wave itself, one position at a time, until the
    // vector is again one that scaled single precision holds faithfully (every entry an exact zero or within
    // 2^-60 of the largest): then the fast path resumes with the next matrix.  The producers are told through
    // the low bit of the published offset to leave those positions alone.  After eight such steps in a row
    // (hard constraints throughout) the chain gives the producers up for good.
    // 0: go on (the matrix of step q is in `nxt`), 2: it did not come, 3: that was the last step, 4: give up.
    const auto slow_steps = [&](Tile& nxt) -> int {
        float lvs = carried ? lv_carry : lane < T ? lane_log(V) : LCCRF_NEG_INF;
        carried = false;
        for (int n = 0;; ++n) {
            unsigned long long word;
            if (!arrived(q, word)) {
                lv_carry = lvs;
                carried = true;
                return 4;
            }
            const int d = lane_log_step<TIN, AL, PASS2>(a, jb, (int)q, lvs, O0 + (double)Oi, lz2, meet_only);
            Oi += d;
            float lall = lvs;  // every copy of the vector gets its tag's value
            if constexpr (kSplit) {
                const auto h = __builtin_amdgcn_permlane32_swap(__float_as_int(lvs), __float_as_int(lvs), false, false);
                lall = __int_as_float(h[0]);
            }
            V = on ? lane_up(lall) : 0.f;
            ++q;
            sh.V[q % kLaneVecRing][u] = V;
            sh.VOi[q % kLaneVecRing] = (Oi << 1) | 1;
            lds_store_release(&sh.done, (int)q);
            if (q == count) {
                lv_carry = lvs;
                carried = true;
                return 3;
            }
            const bool faithful = !(lane < T) || lvs == LCCRF_NEG_INF || lvs >= -60.f;
            const bool inside = (unsigned)(Oi + (1 << 28)) < (1u << 29);
            if (__builtin_amdgcn_ballot_w64(!faithful) == 0 && inside) break;
            if (n >= 7 || !inside) {
                lv_carry = lvs;
                carried = true;
                return 4;
            }
        }
        return fetch(q, nxt) ? 0 : 2;
    };
    // The same for first passes over dense potentials, which do not give the producers up: where more than a third of the
    // steps are such for a while (kOften; independent normal potentials of a deviation of fifteen and more), the rest of the chain is
    // taken in the log domain, and the producers are told to hand on the logarithms of the matrices, in the same slots and the same
    // order: a step adds the rotated vector to them, takes the maximum and adds up the exponentials.  (Matrices that were
    // exponentiated already are taken from memory by this wave.)  `alone`: no producer is waited for any more.
    // 0: go on (the matrix of step q is in `nxt`), 2: it did not come, 3: that was the last step, everything is stored.
    constexpr bool kRaw = lane_takes_raw<TIN, AL, PASS2>();
    constexpr int kOften = NBLK <= 2 ? 16 : 24;
    int slow = 0, slow_at = 0;  // two for every log-domain step, less the other steps since, and where the last one led
    const auto log_steps = [&](Tile& nxt, bool alone) -> int {
        if constexpr (kRaw) {
            lv = u < T ? (carried ? lv_carry : lane_log(V)) : LCCRF_NEG_INF;
            if constexpr (kSplit) {
                const auto h = __builtin_amdgcn_permlane32_swap(__float_as_int(lv), __float_as_int(lv), false, false);
                lv = __int_as_float(h[0]);
            }
            carried = false;
            O = O0 + (double)Oi;
            bool rest = alone;
            if (alone) lds_store_release(&sh.stop, (int)q);
            for (;;) {
                unsigned long long word = 0;
                if (!alone && !arrived(q, word)) {
                    alone = rest = true;
                    word = 0;
                    lds_store_release(&sh.stop, (int)q);
                }
                int d;
                if (__builtin_amdgcn_readfirstlane((int)(unsigned)word) == kLaneRaw) {
                    Tile t;
                    read_entries(q, t);
                    float Ab[4];
                    blocks_of(lv, Ab);
                    float top[4] = {LCCRF_NEG_INF, LCCRF_NEG_INF, LCCRF_NEG_INF, LCCRF_NEG_INF};
#pragma unroll
                    for (int bk = 0; bk < NB; ++bk) add_rotations(t.e[bk], Ab[bk]);
#pragma unroll
                    for (int bk = 0; bk < NB; ++bk)
#pragma unroll
                        for (int m = 0; m < 16; m += 2) top[(m >> 1) & 3] = max3_raw(top[(m >> 1) & 3], t.e[bk][m], t.e[bk][m + 1]);
                    float mx = max3_raw(max3_raw(top[0], top[1], top[2]), top[3], top[3]);
                    if constexpr (kSplit) mx = xor_max<32, 64>(mx);
                    const float g = finite_or_zero(mx);
                    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int bk = 0; bk < NB; ++bk)
#pragma unroll
                        for (int m = 0; m < 16; ++m) part[m & 3] += ex2(t.e[bk][m] - g);
                    float sum = (part[0] + part[1]) + (part[2] + part[3]);
                    if constexpr (kSplit) sum = xor_sum<32, 64>(sum);
                    d = lane_log_end(a, jb, jb.first + (int)q * jb.sdir, on ? mx + lg2(sum) : LCCRF_NEG_INF, u, copy == 0, lv, O, meet_only);
                } else {
                    d = lane_log_dense<NBLK, TIN, AL>(a, jb, sh.G[0], (int)q, lv, O, meet_only);
                    lv = on ? lv : LCCRF_NEG_INF;
                }
                O += (double)d;
                ++q;
                if (!rest) {
                    Oi += d;
                    V = lane_up(lv);
                    sh.V[q % kLaneVecRing][u] = V;
                    sh.VOi[q % kLaneVecRing] = (Oi << 1) | 1;
                    lds_store_release(&sh.done, (int)q);
                    if (q == count) return 3;
                    const bool faithful = lv == LCCRF_NEG_INF || lv >= -110.f;
                    const bool inside = (unsigned)(Oi + (1 << 28)) < (1u << 29);
                    slow = max(slow - ((int)q - slow_at - 1), 0) + 2;
                    slow_at = (int)q;
                    if (__builtin_amdgcn_ballot_w64(!faithful) == 0 && inside && slow < kOften) return fetch(q, nxt) ? 0 : 2;
                    if (!inside || slow >= kOften) {
                        rest = true;
                        alone = !lane_hands_raw(NBLK);
                        lds_store_release(alone ? &sh.stop : &sh.raw, (int)q);
                    }
                } else {
                    if (!alone) {
                        sh.VOi[q % kLaneVecRing] = 1;  // (the stores of this step are done)
                        lds_store_release(&sh.done, (int)q);
                    }
                    if (q == count) return 3;
                }
            }
        }
        return 3;
    };
    // One step from the matrix in `cur`; meanwhile the matrix of the next step is read into `nxt`, whether it is
    // there or not, so that it comes back under the products: its flag is looked at before (LDS executes a wave's
    // instructions in order: a flag that was up when it was read means that the reads behind it found the matrix);
    // if it was not up, the matrix is waited for at the end of the step and read again.  Everything the step leaves behind for the other waves is the vector, one
    // integer and the step count in LDS: the stores to memory are theirs.
    // 0: go on, 1: the step was not accepted (q and the vector are unchanged), 2: the next matrix did not come,
    // 3: that was the last step.
    // (Flags and offsets are written by every lane, the same value to the same address: cheaper for a lone
    // wave than masking the write down to one lane.)
    // In first passes over dense potentials a sum that is zero because every one of its terms is (a tag that is forbidden there or
    // everywhere) is accepted too: the chain goes over to this form at the first step that `quick` below does not accept.
    const auto step = [&](const Tile& cur, Tile& nxt) __attribute__((always_inline)) -> int {
        unsigned long long word_next = lds_load_acquire(&sh.ready[(q + 1) % S::RING]);
        read_entries(q + 1, nxt);
        __builtin_amdgcn_sched_barrier(0);
        float Ab[4];
        blocks_of(V, Ab);
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int bk = 0; bk < NB; ++bk) fmac_rotations(acc, Ab[bk], cur.e[bk]);
        // (the flag is looked at only here, behind the products: its read has had their time to come back)
        asm volatile("" : "+v"(word_next));
        float Ssum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        if constexpr (kSplit) {  // the two halves of the sum
            const auto h = __builtin_amdgcn_permlane32_swap(__float_as_int(Ssum), __float_as_int(Ssum), false, false);
            Ssum = __int_as_float(h[0]) + __int_as_float(h[1]);
        }
        const int Onew = Oi + (cur.m >> 1);
        // accepted: every sum in range, and the integer offset far from overflow
        // (S in [kSumLo, kSumHi] as one unsigned comparison of its bits: positive floats order like their bit patterns,
        // negative ones and NaNs fall outside; the comparison leaves the lane mask in scalar registers directly)
        const unsigned long long inr = __builtin_amdgcn_uicmp(__float_as_uint(Ssum) - __float_as_uint(kSumLo),
                                                              __float_as_uint(kSumHi) - __float_as_uint(kSumLo), 37 /* unsigned <= */);
        unsigned ref = 0;  // the lane whose entry is the reference
        if ((inr & onmask) != onmask || (unsigned)(Onew + (1 << 28)) >= (1u << 29)) {
            if constexpr (!kRaw) return 1;
            // (no entry of the matrix and none of the vector but exact zeros can have taken part in an underflow)
            const unsigned long long zero = __builtin_amdgcn_ballot_w64(Ssum == 0.f), some = inr & onmask;
            if (!(cur.m & 1) || ((inr | zero) & onmask) != onmask || some == 0 || (unsigned)(Onew + (1 << 28)) >= (1u << 29) ||
                __builtin_amdgcn_ballot_w64(V > 0.f && V < 0x1p-60f) != 0)
                return 1;
            ref = (unsigned)__builtin_ctzll(some);
        }
        // Rescale by the power of two that brings tag 0 into [1/2, 1): any accepted entry serves as the
        // reference (what bounds the vector is the range test above, not where its largest entry lies), and
        // lane 0's comes without a reduction over the lanes.  Lanes without a tag hold an exact zero.
        const int kx = __builtin_amdgcn_frexp_expf(Ssum);
        const int k = kRaw ? __builtin_amdgcn_readlane(kx, ref) : __builtin_amdgcn_readfirstlane(kx);
        V = __builtin_amdgcn_ldexpf(Ssum, kLaneHead - k);
        Oi = Onew + k - kLaneHead;
        ++q;
        sh.V[q % kLaneVecRing][u] = V;
        sh.VOi[q % kLaneVecRing] = Oi << 1;
        lds_store_release(&sh.done, (int)q);
        if (q == count) return 3;
        if ((unsigned)__builtin_amdgcn_readfirstlane((int)(word_next >> 32)) >= q + 1) nxt.m = __builtin_amdgcn_readfirstlane((int)(unsigned)word_next);
        else if (!fetch(q, nxt)) return 2;
        return 0;
    };
    // The same without zeros and with no branch, two steps a round: once a step is not accepted, the last one is done or the next matrix
    // has not come, what follows in the round changes nothing and publishes again what stands there.  `mark`: what the last step
    // published beside its offset.  (A lone wave issues an instruction every five cycles and pays some twenty for a branch it takes; with a
    // way out of every step four were taken a step, of 110 instructions where 90 do: 0.25 -> 0.215 us at 32 tags.  Log-probability
    // B=128 N=256 T=32 42.5 -> 38.4 us, sampling there 99 -> 89, log-probability B=100 N=200 T=45 bfloat16 46.0 -> 42.8, marginals B=128
    // N=200 T=30 62.3 -> 59.2.  With zeros accepted, where the quick way is left often, the ways out of every step are the cheaper
    // form: independent normal potentials of deviation 16, log-probability B=128 N=128 T=32 64.9 us so, 67.4 with rounds there too; both
    // before `lane_log_dense` requested its vector at once, 61.0 since.)
    // The second pass of 33 .. 48 tags keeps the way out of every step as well: there the chain comes to wait for its producers, and a round
    // that a matrix is missing in costs more than the branches (marginals B=25 N=237 T=45 101.5 us so, 105.5 without).
    constexpr bool kQuick = !(PASS2 && NBLK == 3);
    int mark = 0;
    // (Where the shared state stands, kept in a vector register: an address in it is then one instruction.)
    typedef __attribute__((address_space(3))) char LdsBytes;
    unsigned at = (unsigned)(uintptr_t)(LdsBytes*)&sh;
    asm volatile("" : "+v"(at));
    const unsigned at_row = at + (unsigned)offsetof(LaneShared<NBLK>, E) + (unsigned)((urow * S::RS + (kSplit ? 16 * copy : 0)) * sizeof(float));
    const unsigned at_v = at + (unsigned)offsetof(LaneShared<NBLK>, V) + (unsigned)(u * sizeof(float));
#define LCCRF_LDS(T, x) (*(__attribute__((address_space(3))) T*)(uintptr_t)(x))
    const auto quick = [&](const Tile& cur, Tile& nxt, bool& going, bool& refused) __attribute__((always_inline)) {
        const unsigned slot = (q + 1) % S::RING;
        unsigned long long word_next = __hip_atomic_load(&LCCRF_LDS(unsigned long long, at + (unsigned)offsetof(LaneShared<NBLK>, ready) + 8 * slot),
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
        for (int bk = 0; bk < NB; ++bk)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const vec4f v = LCCRF_LDS(const vec4f, at_row + slot * (unsigned)sizeof(sh.E[0]) + (unsigned)((16 * bk + 4 * g) * sizeof(float)));
                nxt.e[bk][4 * g] = v[0]; nxt.e[bk][4 * g + 1] = v[1]; nxt.e[bk][4 * g + 2] = v[2]; nxt.e[bk][4 * g + 3] = v[3];
            }
        __builtin_amdgcn_sched_barrier(0);
        float Ab[4];
        blocks_of(V, Ab);
        float acc[4];
        mul_rotations(acc, Ab[0], cur.e[0]);
#pragma unroll
        for (int bk = 1; bk < NB; ++bk) fmac_rotations(acc, Ab[bk], cur.e[bk]);
        asm volatile("" : "+v"(word_next));
        float Ssum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        if constexpr (kSplit) {  // the two halves of the sum
            const auto h = __builtin_amdgcn_permlane32_swap(__float_as_int(Ssum), __float_as_int(Ssum), false, false);
            Ssum = __int_as_float(h[0]) + __int_as_float(h[1]);
        }
        const int Onew = Oi + (cur.m >> 1);
        const unsigned long long inr = __builtin_amdgcn_uicmp(__float_as_uint(Ssum) - __float_as_uint(kSumLo),
                                                              __float_as_uint(kSumHi) - __float_as_uint(kSumLo), 37 /* unsigned <= */);
        const bool in = (inr & onmask) == onmask && (unsigned)(Onew + (1 << 28)) < (1u << 29);
        const bool took = going & in;
        refused = refused | (going & !in);
        const int k = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_expf(Ssum));
        V = took ? __builtin_amdgcn_ldexpf(Ssum, kLaneHead - k) : V;
        Oi = took ? Onew + k - kLaneHead : Oi;
        mark = took ? 0 : mark;
        q += took ? 1u : 0u;
        LCCRF_LDS(float, at_v + 256 * (q % kLaneVecRing)) = V;
        LCCRF_LDS(int, at + (unsigned)offsetof(LaneShared<NBLK>, VOi) + 4 * (q % kLaneVecRing)) = (Oi << 1) | mark;
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __hip_atomic_store(&LCCRF_LDS(int, at + (unsigned)offsetof(LaneShared<NBLK>, done)), (int)q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        nxt.m = __builtin_amdgcn_readfirstlane((int)(unsigned)word_next);
        going = took & ((unsigned)__builtin_amdgcn_readfirstlane((int)(word_next >> 32)) >= q + 1) & (q != count);
    };
#undef LCCRF_LDS
    Tile tA, tB;
    if (count > 0) {
        int why = carried ? 1 : fetch(0, tA) ? 0 : 2;
        bool zeros = false;
        for (;;) {
            if constexpr (!kQuick) {
                while (why == 0) {
                    why = step(tA, tB);
                    if (why != 0) break;
                    why = step(tB, tA);
                }
            } else if (!kRaw || !zeros) {
                while (why == 0) {
                    bool refused = false, going = true;
                    do {
                        quick(tA, tB, going, refused);
                        quick(tB, tA, going, refused);
                    } while (going);
                    why = refused ? 1 : q == count ? 3 : fetch(q, tA) ? 0 : 2;
                }
            }
            if constexpr (kRaw) {
                if (why == 1 && !zeros && !carried) why = fetch(q, tA) ? 0 : 2;  // (the same matrix, which the slot still holds)
                zeros = true;
                while (why == 0) {
                    why = step(tA, tB);
                    if (why != 0) break;
                    why = step(tB, tA);
                }
            }
            if constexpr (kRaw) {
                if (why == 3) break;
                why = log_steps(tA, why == 2);
                if (why == 3) return;
            } else {
                if (why != 1) break;
                mark = 1;
                why = slow_steps(tA);  // (outside the loop of the fast path, which stays as tight as it was)
            }
        }
        tail = why != 3;
    }
    O = O0 + (double)Oi;
    on = lane < T;  // from here on lane = tag again (the first copy)
    lv = !on ? LCCRF_NEG_INF : carried ? lv_carry : lane_log(V);
    if (tail) {
        if (lane == 0) lds_store_release(&sh.stop, (int)q);
        if constexpr (!kRaw) lane_log_tail<TIN, AL, PASS2>(a, jb, (int)q, lv, O, lz2, meet_only);
    } else if (!PASS2 && meet_only && count > 0) {
        // a log-partition call keeps the vectors of the meeting position only: the last of this chain
        if (on) (jb.dir == 0 ? a.ua : a.ub)[(vb + jb.h) * T + lane] = lv;
        if (lane == 0) (jb.dir == 0 ? a.Oa : a.Ob)[vb + jb.h] = O;
    }
    if (PASS2 && jb.dir == 1) {
        // position 0: p(y_0 = t) = 2^(alpha_0(t) + beta_0(t) - log2 Z) in row 0 (the other rows were cleared at the start)
        const float z = on ? a.ua[vb * T + me] + lv + (float)(a.Oa[vb] + O - lz2) : LCCRF_NEG_INF;
        if (on) a.mu[vb * TT + lane] = feasible ? ex2(z) : 0.f;
    }
}

// A producer wave.
template <int NBLK, typename TIN, bool AL, bool PASS2>
__device__ __forceinline__ void lane_producer_wave(const ChainArgs& a, const LaneJob& jb, LaneShared<NBLK>& sh, int w,
                                                   double lz2, int meet_only, int poll_limit) {
    using S = LaneShape<NBLK>;
    constexpr int NG = S::NG, PF = S::PF, W = lane_waves(NBLK) - 1;
    constexpr bool kRaw = lane_takes_raw<TIN, AL, PASS2>(), kHandsRaw = kRaw && lane_hands_raw(NBLK);
    const int lane = threadIdx.x & 63, T = a.T, N = a.N, b = jb.b;
    const size_t TT = (size_t)T * T;
    const size_t vb = (size_t)b * N;
    const LaneSource<TIN, AL> src(a, b);
    const int nj = w < jb.count ? (jb.count - w + W - 1) / W : 0;  // matrices of this wave: steps w, w + W, ...
    if (nj == 0) return;
    // group m of this lane: piece g = lane + 64 m of the matrix, row s = g / Q, columns t0 .. t0 + 3, Q pieces a row:
    // t0 = 4 (g % Q), but the last piece of a row ends with the row (T - 4: only a tag count that is no multiple of
    // four moves it)
    int goff[NG], grow[NG], gcol[NG], laddr[NG][4];
    unsigned valid = 0;
    const int Q = (T + 3) >> 2;
#pragma unroll
    for (int m = 0; m < NG; ++m) {
        const int g = lane + 64 * m;
        const bool ok = g < T * Q;
        valid |= ok ? (1u << m) : 0u;
        const int s = ok ? g / Q : 0, t0 = ok ? min(4 * (g % Q), T - 4) : 0;
        goff[m] = s * T + t0;
        grow[m] = s;
        gcol[m] = t0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = t0 + k;
            const int u = jb.dir == 0 ? t : s, v = jb.dir == 0 ? s : t;
            laddr[m][k] = u * S::RS + 16 * (v >> 4) + ((u - v) & 15);
        }
    }
    float x[PF][NG][4], aux[PF];
    double oo[PF];
    float fixed[LaneSource<TIN, AL>::kStruct ? NG : 1][4];  // structured potentials: this lane's entries of the transition matrix
    if constexpr (LaneSource<TIN, AL>::kStruct) {
#pragma unroll
        for (int m = 0; m < NG; ++m) src.fixed_part(goff[m], gcol[m], fixed[m]);
    }
    const auto load = [&](int j, int p) {
        const int q = w + (j < nj ? j : nj - 1) * W;
        const int i = jb.first + q * jb.sdir;
#pragma unroll
        for (int m = 0; m < NG; ++m) src.piece(i, goff[m], gcol[m], fixed[LaneSource<TIN, AL>::kStruct ? m : 0], x[p][m]);
        if (PASS2) {
            const size_t vp = jb.dir == 0 ? vb + i : vb + i - 1;
            aux[p] = (jb.dir == 0 ? a.ub : a.ua)[vp * T + (lane < T ? lane : 0)];
            oo[p] = (jb.dir == 0 ? a.Ob : a.Oa)[vp];
        }
    };
    // Waits until the flag reaches `target` (true) or the chain has stopped at or before step `q` (false).
    // The chain wave always does one or the other: each of its own waits is bounded by the poll limit of the call.
    // The limit here, a thousand times the default, is a last resort that only keeps a wave from spinning for ever.
    const auto wait_for = [&](const int* flag, int target, int q) -> bool {
        long long spins = 0;
        while (lds_load_acquire(flag) < target) {
            if (lds_load_acquire(&sh.stop) <= q || ++spins > 1000ll * (poll_limit + 65536)) return false;
            __builtin_amdgcn_s_sleep(1);
        }
        return true;
    };
    // One matrix (number j of this wave, in buffer p): exponentiate, hand to the chain, write its marginals.
    // false: the chain has stopped before this matrix, nothing more to do.
    const auto process = [&](int j, auto pc) -> bool {
        constexpr int p = decltype(pc)::value;
        const int q = w + j * W;
        const int i = jb.first + q * jb.sdir;
        const int slot = q % S::RING;
        const auto raw_now = [&]() { return kHandsRaw && __builtin_amdgcn_readfirstlane(lds_load_acquire(&sh.raw)) <= q; };
        const auto logarithms = [&]() {
#pragma unroll
            for (int m = 0; m < NG; ++m)
#pragma unroll
                for (int k = 0; k < 4; ++k) x[p][m][k] *= kLog2e;
        };
        const bool raw = raw_now();
        float sh_m = 0.f;
        int word = kLaneRaw;
        if (raw) {
            logarithms();
        } else {
            // the shift of this matrix: the smallest integer at or above its largest entry (base 2)
            float mxr = LCCRF_NEG_INF;
#pragma unroll
            for (int m = 0; m < NG; ++m) {
                const float gm = max3_raw(fmaxf(x[p][m][0], x[p][m][1]), x[p][m][2], x[p][m][3]);
                mxr = fmaxf(mxr, (valid >> m) & 1 ? gm : LCCRF_NEG_INF);
            }
            // (clamped far inside the range of an int: beyond, the chain's offset check sends the step to the tail)
            sh_m = fminf(fmaxf(ceilf(finite_or_zero(xor_max<1, 64>(mxr)) * kLog2e), -0x1p29f), 0x1p29f);
            float least[2] = {0.f, 0.f};
#pragma unroll
            for (int m = 0; m < NG; ++m)
#pragma unroll
                for (int k = 0; k < 4; ++k) x[p][m][k] = __builtin_fmaf(x[p][m][k], kLog2e, -sh_m);
            word = (int)sh_m * 2;
            if constexpr (kRaw) {
                // whether no entry but exact zeros lies below 2^-80
#pragma unroll
                for (int m = 0; m < NG; ++m) {
                    least[0] = min3_raw(least[0], x[p][m][0], x[p][m][1]);
                    least[1] = min3_raw(least[1], x[p][m][2], x[p][m][3]);
                }
                word |= 1;
                if (__builtin_amdgcn_ballot_w64(fminf(least[0], least[1]) < -80.f) != 0) {
                    // (by the bits: read as unsigned numbers less those of -inf, the finite numbers below -80 are the largest)
                    unsigned low = 0;
#pragma unroll
                    for (int m = 0; m < NG; ++m)
#pragma unroll
                        for (int k = 0; k < 4; ++k) low = max(low, __float_as_uint(x[p][m][k]) - 0xff800000u);
                    if (__builtin_amdgcn_ballot_w64(low > 0xc2a00000u - 0xff800000u) != 0) word &= ~1;
                }
            }
#pragma unroll
            for (int m = 0; m < NG; ++m)
#pragma unroll
                for (int k = 0; k < 4; ++k) x[p][m][k] = ex2(x[p][m][k]);
        }
        // the slot is free once the chain has accepted step q - RING
        if (!wait_for(&sh.done, q - S::RING + 1, q)) return false;
        if constexpr (kHandsRaw) {
            if (!raw && raw_now()) {  // (once in a chain: the exponentials were in vain)
                word = kLaneRaw;
                const int i = jb.first + q * jb.sdir;
#pragma unroll
                for (int m = 0; m < NG; ++m) {
                    src.piece(i, goff[m], gcol[m], fixed[0], x[p][m]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                logarithms();
            }
        }
        float* Es = &sh.E[slot][0][0];
#pragma unroll
        for (int m = 0; m < NG; ++m)
            if ((valid >> m) & 1) {
#pragma unroll
                for (int k = 0; k < 4; ++k) Es[laddr[m][k]] = x[p][m][k];
            }
        if (lane == 0)
            lds_store_release(&sh.ready[slot], ((unsigned long long)(unsigned)(q + 1) << 32) | (unsigned)word);
        if (PASS2) {
            // the chain has accepted step q: V_q and this matrix make the marginals of position i
            if (!wait_for(&sh.done, q + 1, q)) return false;
            if (sh.VOi[(q + 1) % kLaneVecRing] & 1) return true;  // (the chain wave took this step itself)
            const double Oq = sh.O0 + (double)(sh.VOi[q % kLaneVecRing] >> 1);
            const float c = (float)(Oq + (double)sh_m + oo[p] - lz2);
            sh.G[w][lane] = lane < T ? __builtin_amdgcn_ldexpf(ex2(aux[p] + c), -kLaneHead) : 0.f;
            const float* rowf = jb.dir == 0 ? sh.V[q % kLaneVecRing] : sh.G[w];
            const float* colf = jb.dir == 0 ? sh.G[w] : sh.V[q % kLaneVecRing];
            float* mu_i = a.mu + (vb + i) * TT;
#pragma unroll
            for (int m = 0; m < NG; ++m)
                if ((valid >> m) & 1) {
                    const float rf = rowf[grow[m]];
                    float cf[4];
                    lane_load4<AL>(colf + gcol[m], cf);
                    lane_store4<AL>(mu_i + goff[m], x[p][m][0] * rf * cf[0], x[p][m][1] * rf * cf[1], x[p][m][2] * rf * cf[2],
                                    x[p][m][3] * rf * cf[3]);
                }
        }
        if (!PASS2 && !meet_only) {
            // the chain has accepted step q: its result is the vector of position i (forward) or i - 1 (backward)
            if (!wait_for(&sh.done, q + 1, q)) return false;
            const int pos = jb.dir == 0 ? i : i - 1;
            const int word = sh.VOi[(q + 1) % kLaneVecRing];
            if (word & 1) return true;  // (the chain wave took this step itself, stores included)
            const float v = sh.V[(q + 1) % kLaneVecRing][lane];
            if (lane < T) (jb.dir == 0 ? a.ua : a.ub)[(vb + pos) * T + lane] = lane_log(v);
            if (lane == 0) (jb.dir == 0 ? a.Oa : a.Ob)[vb + pos] = sh.O0 + (double)(word >> 1);
        }
        return true;
    };
    // Two buffers: the next matrix is requested just before the current one is worked on, so the only loads in
    // flight during a matrix are those of its successor (whatever the compiler then waits for at the top of the
    // loop, it is data the wave needs at once).
    using Buf0 = std::integral_constant<int, 0>;
    using Buf1 = std::integral_constant<int, 1>;
    load(0, 0);
    for (int j = 0; j < nj; j += 2) {
        load(j + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        if (!process(j, Buf0{})) break;
        load(j + 2, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (j + 1 < nj && !process(j + 1, Buf1{})) break;
    }
}

template <int NBLK, typename TIN, bool AL, bool PASS2>
__global__ __launch_bounds__(64 * lane_waves(NBLK)) void lane_chain_kernel(ChainArgs a, int meet_only, int poll_limit) {
    using S = LaneShape<NBLK>;
    constexpr int kLaneWaves = lane_waves(NBLK);
    extern __shared__ __attribute__((aligned(16))) unsigned char lane_smem[];
    LaneShared<NBLK>& sh = *reinterpret_cast<LaneShared<NBLK>*>(lane_smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: loops over a wave's work stay scalar
    const int T = a.T, N = a.N;
    LaneJob jb;
    // (one forward chain a sequence over the whole of it, every vector stored: the first pass of sampling)
    const bool whole = !PASS2 && a.full_forward != 0;
    jb.b = whole ? blockIdx.x : blockIdx.x >> 1;
    jb.dir = whole ? 0 : blockIdx.x & 1;
    jb.L = clamp_length(a.lengths, jb.b, N);
    const int b = jb.b, L = jb.L;
    const size_t TT = (size_t)T * T;
    const size_t vb = (size_t)b * N;
    // Marginals that carry no edge are zero: the positions past the end (forward workgroup) and rows
    // 1 .. T - 1 of position 0 (backward workgroup).  Cleared by the wave that has no other work
    // (by everyone for an empty sequence).
    const auto zero_floats = [&](float* d, size_t n, int first, int threads) {  // n floats from d on, by threads first, first + 1, ...
        for (size_t k = first; k < n / 4; k += threads) lane_store4<AL>(d + 4 * k, 0.f, 0.f, 0.f, 0.f);
        if (!AL && first < (int)(n % 4)) d[n - 1 - first] = 0.f;
    };
    const auto clear_edgeless = [&](int first_thread, int threads) {
        if (jb.dir == 0) zero_floats(a.mu + (vb + L) * TT, (size_t)(N - L) * TT, tid - first_thread, threads);
        else if (L > 0) zero_floats(a.mu + vb * TT + T, TT - T, tid - first_thread, threads);
    };
    if (L == 0) {
        if (PASS2) clear_edgeless(0, 64 * kLaneWaves);
        if (PASS2 && jb.dir == 0 && tid == 0 && a.logZ) a.logZ[b] = 0.f;
        return;
    }
    const int e = L - 1;
    jb.h = whole ? e : meeting_point(0, e);
    if (!PASS2) {
        if (jb.dir == 0) { jb.first = 1; jb.sdir = +1; jb.count = jb.h; }
        else { jb.first = e; jb.sdir = -1; jb.count = e - jb.h; }
    } else {
        if (jb.dir == 0) { jb.first = jb.h + 1; jb.sdir = +1; jb.count = e - jb.h; }
        else { jb.first = jb.h; jb.sdir = -1; jb.count = jb.h; }
    }
    // log2 Z from the two vectors stored for the meeting position
    double lz2 = 0.0;
    bool feasible = true;
    if (PASS2) {
        const float z = lane < T ? a.ua[(vb + jb.h) * T + lane] + a.ub[(vb + jb.h) * T + lane] : LCCRF_NEG_INF;
        const float M = xor_max<1, 64>(z);
        const float Ssum = xor_sum<1, 64>(ex2(z - finite_or_zero(M)));
        lz2 = (double)(M + lg2(Ssum)) + a.Oa[vb + jb.h] + a.Ob[vb + jb.h];
        feasible = lz2 > -1.0e300;
        if (jb.dir == 0 && tid == 0 && a.logZ) a.logZ[b] = (float)(lz2 * kLn2);
        if (!feasible) {  // no path has a finite score: every marginal is zero
            for (int q = 0; q < jb.count; ++q) {
                zero_floats(a.mu + (vb + jb.first + q * jb.sdir) * TT, TT, tid, 64 * kLaneWaves);
            }
            if (jb.dir == 1 && tid < T) a.mu[vb * TT + tid] = 0.f;
            clear_edgeless(0, 64 * kLaneWaves);
            return;
        }
    }
    // flags, and zeros where no producer ever writes (source tags past T)
    if (tid < S::RING) sh.ready[tid] = 0ull;
    if (tid == 0) { sh.done = 0; sh.stop = 0x7fffffff; sh.raw = 0x7fffffff; }
    if (T != S::U) {
        float* Ez = &sh.E[0][0][0];
        for (int k = tid; k < S::RING * (S::U + 1) * S::RS; k += 64 * kLaneWaves) Ez[k] = 0.f;
    } else {
        for (int k = tid; k < S::RING * S::RS; k += 64 * kLaneWaves) sh.E[k / S::RS][S::U][k % S::RS] = 0.f;
    }
    __syncthreads();
    if (wv == 0) {
        __builtin_amdgcn_s_setprio(3);
        lane_chain_wave<NBLK, TIN, AL, PASS2>(a, jb, sh, lz2, feasible, meet_only, poll_limit);
    } else {
        if (PASS2 && wv == 4) clear_edgeless(4 * 64, 64);  // (the producer that shares the chain's SIMD)
        lane_producer_wave<NBLK, TIN, AL, PASS2>(a, jb, sh, wv - 1, lz2, meet_only, poll_limit);
    }
}

// ---------------------------------------------------------------------------------------
// Dense or structured potentials, whole sequences, 8 .. 64 tags: multiples of four (16-byte pieces of a row) at every
// size, other counts (element loads) up to 48.  Five to seven tags are taken too where it pays, though no caller can ask for it.
bool lane_supported(int T) { return T >= 8 && lane_fits(T); }
bool lane_fits(int T) { return T >= 5 && T <= 64 && (T % 4 == 0 || T <= 48); }

template <int NBLK, typename TIN, bool AL, bool PASS2>
static hipError_t launch_lane_kernel(const ChainArgs& a, int meet_only, int poll_limit, hipStream_t st) {
    const size_t bytes = sizeof(LaneShared<NBLK>);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&lane_chain_kernel<NBLK, TIN, AL, PASS2>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((lane_chain_kernel<NBLK, TIN, AL, PASS2>), dim3((!PASS2 && a.full_forward ? 1 : 2) * a.B), dim3(64 * lane_waves(NBLK)), bytes, st, a, meet_only, poll_limit);
    return hipGetLastError();
}
template <int NBLK, bool AL>
static hipError_t launch_lane_al(bool second_pass, int dtype, const ChainArgs& a, int meet_only, int poll_limit, hipStream_t st) {
    if (a.emit)
        return second_pass ? launch_lane_kernel<NBLK, StructF, AL, true>(a, meet_only, poll_limit, st)
                           : launch_lane_kernel<NBLK, StructF, AL, false>(a, meet_only, poll_limit, st);
    if (dtype == 0)
        return second_pass ? launch_lane_kernel<NBLK, float, AL, true>(a, meet_only, poll_limit, st)
                           : launch_lane_kernel<NBLK, float, AL, false>(a, meet_only, poll_limit, st);
    return second_pass ? launch_lane_kernel<NBLK, uint16_t, AL, true>(a, meet_only, poll_limit, st)
                       : launch_lane_kernel<NBLK, uint16_t, AL, false>(a, meet_only, poll_limit, st);
}
template <int NBLK>
static hipError_t launch_lane_nblk(bool second_pass, int dtype, const ChainArgs& a, int meet_only, int poll_limit, hipStream_t st) {
    if (a.T % 4 == 0) return launch_lane_al<NBLK, true>(second_pass, dtype, a, meet_only, poll_limit, st);
    if constexpr (NBLK <= 3) return launch_lane_al<NBLK, false>(second_pass, dtype, a, meet_only, poll_limit, st);
    return hipErrorInvalidValue;
}

hipError_t launch_lane_pass(bool second_pass, int dtype, const ChainArgs& a, bool meet_only, int poll_limit, hipStream_t st) {
    if (!lane_fits(a.T) || a.chunk > 0 || (a.emit && (dtype != 0 || !a.trans))) return hipErrorInvalidValue;
    const int mo = meet_only ? 1 : 0;
    if (a.T <= 16) return launch_lane_nblk<1>(second_pass, dtype, a, mo, poll_limit, st);
    if (a.T <= 32) return launch_lane_nblk<2>(second_pass, dtype, a, mo, poll_limit, st);
    if (a.T <= 48) return launch_lane_nblk<3>(second_pass, dtype, a, mo, poll_limit, st);
    return launch_lane_nblk<4>(second_pass, dtype, a, mo, poll_limit, st);
}

}  // namespace lccrf
