// Chains of 65 .. 256 tags walked in pieces by several workgroups, in scaled probabilities (lccrf_linear.h); the body of the first-pass
// kernels linear_half_kernel (lccrf_chain.hip) and stream_half_kernel (lccrf_stream.hip).
//
// One workgroup a chain leaves most of the chip idle where a batch has few chains, and a step of a large tag set is bound by what one
// compute unit reads and exponentiates.  The steps of a chain are products of non-negative matrices, which forget where they started:
// whatever positive vector a chain is begun with, after a number of steps that the potentials set (about ten for scores of deviation
// one) it is a multiple of the true one.  So the chain is cut into pieces, one workgroup each, in three launches:
//   0  piece 0 is walked from the true start, all others from a vector of ones; vectors and offsets are stored, the last vector of a piece
//      beside them (ends, end_offsets);
//   1  pieces 1 .. are walked again, each from the last vector of the piece before it, until its rows agree with those that are there (LinMatch):
//      from there on launch 0's rows are right but for a constant in the offset.  Where no row does, the last vector goes to ends2;
//   2  a workgroup a chain adds up the constants and puts them into the offsets.  From the first piece on of which no row agreed, the
//      rest of the chain is walked as a whole, from that piece's last vector, which is the true one: what started behind it was not.
// Potentials that forget slowly (deviation three and up: forty steps and more) cost no more steps one after the other than without
// pieces: n/C + n/C + (C - 2) n/C.  Batches that are seen to are not cut (piece_steps): launch 0 walks their chains as a whole, or leaves them to a
// fourth launch where that is quicker at it (launch_geo in lccrf_chain.hip).
#pragma once

#include "lccrf_chain_args.h"
#include "lccrf_linear.h"

namespace lccrf {

constexpr int kPieceUnmatched = 0x7fffffff;

// The piece of a chain of n steps that workgroup c of at most C walks: steps s0 .. s1 - 1 of `count` pieces, of `least` steps or more
// where there are several.
struct Piece {
    int count, s0, s1;
};
__host__ __device__ __forceinline__ Piece piece_of(int n, int C, int least, int c) {
    const int most = n / least, cut = C < most ? C : most > 1 ? most : 1;
    const int len = n > 0 ? (n + cut - 1) / cut : 1;
    const int count = n > 0 ? (n + len - 1) / len : 1;
    const int s0 = c * len, s1 = s0 + len;
    return {count, s0, s1 < n ? s1 : n};
}

// The least steps a piece should have, guessed from four matrices of the batch: launch 1 should find its match inside.  Of a column t, whose
// sum over the predecessors s carries 1 / r = (sum_s E)^2 / sum_s E^2 terms that count, a step passes on a share of about sqrt(r) of the
// differences that its tags came with.  (Columns, whichever way the chain runs: a factor of a column's own, an emission, slows nothing
// down.)  Steps until 20 bits agree, times -log2 r (mean over 64 columns), the largest of twelve or more chains of 66 .. 256 tags: independent
// scores of deviation one 37 .. 40, two 57 .. 68, three 79 .. 102, ten 37 .. 63; emissions of deviation two with transitions of deviation
// one 62 .. 81, two 71 .. 90; a match takes an eighth of them more (LinMatch).  The guess, 85 (1 + 2 r) / -log2 r, lies a sixth and more above
// what these take.  Where the longest of these four chains gains too little by it (a.piece_overhead: what the launches take, in
// steps), one piece.  The same for all workgroups; it decides nothing but how fast a call is.  Called by the whole workgroup of 16 waves.
template <typename TIN>
__device__ __forceinline__ int piece_steps(const ChainArgs& a) {
    __shared__ __attribute__((aligned(16))) float rs[16];
    __shared__ int longest;
    if (threadIdx.x == 0) longest = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6);
    const int T = a.T, k = wave >> 2, b = (int)(((long long)k * a.B) >> 2);
    const int L = clamp_length(a.lengths, b, a.N);
    float r = 0.f;
    if (L >= 2) {
        const TIN* mat = static_cast<const TIN*>(a.phi) + ((size_t)b * a.N + 1 + (int)(((long long)k * (L - 2)) >> 2)) * T * T;
        const int row = lane >> 4, col = 16 * (wave & 3) + (lane & 15);
        float x[32], m = LCCRF_NEG_INF, s1 = 0.f, s2 = 0.f;  // (128 rows; of a larger matrix r then comes out somewhat too large)
#pragma unroll
        for (int q = 0; q < 32; ++q) x[q] = Elem<TIN>::get(mat + (size_t)min(row + 4 * q, T - 1) * T + col) * kLog2e;
#pragma unroll
        for (int q = 0; q < 32; ++q) m = fmaxf(m, x[q]);
        m = finite_or_zero(xor_max<16, 64>(m));
#pragma unroll
        for (int q = 0; q < 32; ++q) {
            const float e = row + 4 * q < T ? ex2(x[q] - m) : 0.f;
            s1 += e;
            s2 = __builtin_fmaf(e, e, s2);
        }
        s1 = xor_sum<16, 64>(s1);
        s2 = xor_sum<16, 64>(s2);
        r = xor_sum<1, 16>(s2 / (s1 * s1)) * (1.f / 64.f);
    }
    if (lane == 0) {
        rs[wave] = r;
        atomicMax(&longest, L);
    }
    __syncthreads();
    r = 0.f;
    bool fine = true;
#pragma unroll
    for (int q = 0; q < 16; q += 4) {
        const float4 w = *reinterpret_cast<const float4*>(&rs[q]);
        const float mean = (w.x + w.y) + (w.z + w.w);
        fine = fine && mean >= 0.f;  // (not NaN)
        r = fmaxf(r, mean);
    }
    const float guess = 85.f * (1.f + 2.f * r) / -lg2(r);
    if (!(fine && guess > 0.f && guess < 1e6f)) return kNoPieces;
    const int least = uniform((int)fmaxf(guess, (float)kPieceSteps));
    const int n = a.whole || a.full_forward ? uniform(longest) - 1 : uniform(longest) / 2, cut = min(a.pieces, n / least);
    return cut > 1 && (float)n / (float)cut + 0.8f * guess + (float)a.piece_overhead <= 0.85f * (float)n ? least : kNoPieces;
}

// The row that log-domain steps have come to (see LinMatch): v, O this thread's entry and the offset, against those of the row.
// Called by the whole workgroup.
__device__ __forceinline__ void look_at_row(const float* urow, double Orow, int T, int step, float v, double O, LinMatch& match) {
    __shared__ __attribute__((aligned(16))) float worst[2][16];  // (max16 reads four at a time)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float over = LCCRF_NEG_INF, under = LCCRF_NEG_INF;
    if (tid < T) linear_gap(v, urow[tid], over, under);
    over = xor_max<1, 64>(over);
    under = xor_max<1, 64>(under);
    if (tid < 16) worst[0][tid] = worst[1][tid] = LCCRF_NEG_INF;
    __syncthreads();
    if (lane == 0) {
        worst[0][wave] = over;
        worst[1][wave] = under;
    }
    __syncthreads();
    over = uniform_f(max16(worst[0]));
    under = uniform_f(max16(worst[1]));
    match.look(step, over, under, O - Orow);
    __syncthreads();
}

// What a kernel of a first pass is for: chains as a whole (without anything of the pieces: one kernel for these and launch 0 took 1.3 us a call more, B=54 N=8
// log-partition T=97 bfloat16 16.8 / 15.4, T=131 single precision 19.4 / 18.4), launches 0 and 2 of chains in pieces, or launch 1.
enum PieceMode { kChainsWhole, kChainsInPieces, kComparePieces };

// Workgroups of a launch.
__host__ __forceinline__ int piece_workgroups(const ChainArgs& a) {
    const int chains = a.full_forward ? a.B : 2 * a.B;
    return chains * (a.pieces <= 1 || a.piece_pass == 2 ? 1 : a.piece_pass == 1 ? a.pieces - 1 : a.pieces);
}

// One workgroup of a first pass.  log_steps(first position, number, v, O): that many positions in the log domain.
template <typename LG, typename TIN, bool ALIGNED, int MODE, typename LogSteps>
__device__ __forceinline__ void piece_walk(LinSmem<LG>& lin, const ChainArgs& a, LogSteps log_steps) {
    constexpr bool COMPARE = MODE == kComparePieces;
    const int tid = threadIdx.x;
    // (Neighbouring workgroups go to different XCDs: without backward chains every second one would leave half of the chip idle.)
    const int chains = a.full_forward ? a.B : 2 * a.B, unit = MODE == kChainsWhole ? blockIdx.x : blockIdx.x % chains;
    const int chain = a.full_forward ? 2 * unit : unit, c = MODE == kChainsWhole ? 0 : blockIdx.x / chains + (COMPARE ? 1 : 0);
    const int dir = chain & 1, b = chain >> 1;
    const int N = a.N, T = a.T;
    const int pass = MODE == kChainsWhole ? 0 : COMPARE ? 1 : a.piece_pass;
    const size_t slot = MODE == kChainsWhole ? 0 : (size_t)chain * a.pieces;
    // matched_from of piece 0, written by launch 0 for those behind it: twice the least steps, and one more if the chain takes no scaled steps.
    const int plan = pass > 0 ? a.matched_from[slot] : 0;
    const int L = clamp_length(a.lengths, b, N);
    if (L == 0) return;
    const int e = L - 1, mid = meeting_point(0, e);
    const size_t vb = (size_t)b * N;
    const TIN* phib = static_cast<const TIN*>(a.phi) + vb * T * T;
    float* uout = (dir == 0 ? a.ua : a.ub) + vb * T;
    double* Oout = (dir == 0 ? a.Oa : a.Ob) + vb;
    // the positions of the chain and of the piece
    const int end = dir == 0 ? (a.whole ? e : forward_end(a, 0, e)) : a.whole ? 0 : mid;
    const int first = dir == 0 ? 1 : e, n = dir == 0 ? end : e - end;
    const auto position = [&](int s) { return dir == 0 ? s : e - s; };  // of the vector behind s steps
    int least = kPieceSteps;
    bool hopeless = a.exact_only != 0;
    if (pass > 0) {
        least = uniform(plan) >> 1;
        hopeless = uniform(plan) & 1;
    } else if (MODE == kChainsInPieces) {
        least = piece_steps<TIN>(a);
        if (a.whole_elsewhere && least == kNoPieces) {
            if (c == 0 && tid == 0) a.matched_from[slot] = 2 * kNoPieces;
            return;
        }
    }
    Piece p = MODE == kChainsWhole ? Piece{1, 0, n} : piece_of(n, a.pieces, least, c);
    if (c >= p.count || (pass == 2 && p.count == 1)) return;
    float v = LCCRF_NEG_INF, x = 0.f;  // x: -inf where a tag cannot be in front of the sequence's first edge
    double O = 0.0;
    bool last = c == p.count - 1;
    if constexpr (COMPARE) {
        if (tid < T) v = a.ends[(slot + c - 1) * T + tid];
        O = a.end_offsets[slot + c - 1];
    } else if (pass == 0) {
        if (tid < T) {
            x = Elem<TIN>::get(phib + tid);
            v = dir == 0 && c == 0 ? x * kLog2e : 0.f;
        }
    } else {
        double sum = 0.0;
        int k = 1;
        const auto add = [&](int s0, int s1) {
            for (int s = s0 + tid; s < s1; s += 64 * LG::WAVES) Oout[position(s)] += sum;
        };
        for (; k < p.count; ++k) {
            const Piece q = piece_of(n, a.pieces, least, k);
            const int from = uniform(a.matched_from[slot + k]);
            if (from == kPieceUnmatched) {
                add(q.s0, q.s1);
                p.s0 = q.s1;
                break;
            }
            add(q.s0, from);
            sum += uniform(a.deltas[slot + k]);
            add(from, q.s1 + (k == p.count - 1 ? 1 : 0));
        }
        if (k == p.count) return;
        if (tid < T) v = a.ends2[(slot + k) * T + tid];
        O = uniform(a.end_offsets2[slot + k]) + sum;
        p.s1 = n;
        last = true;
    }
    int steps = p.s0;
    LinMatch match;
    match.start = p.s0;
    LogBlocks blocks;
    if (pass == 0) {
        hopeless = hopeless || (n > 0 && linear_hopeless(phib + (size_t)(dir == 0 ? first + steps : first - steps) * T * T, T, dir == 1, x == LCCRF_NEG_INF, v));
        if (MODE == kChainsInPieces && c == 0 && tid == 0) a.matched_from[slot] = 2 * least + (hopeless ? 1 : 0);
    }
    blocks.hopeless = hopeless;
    for (;;) {
        const int before = steps;
        if (!blocks.hopeless) {
            if (dir == 0) steps = linear_run<LG, TIN, ALIGNED, false, COMPARE>(lin, {phib, T, first, p.s1, uout, Oout}, v, steps, O, match);
            else steps = linear_run<LG, TIN, ALIGNED, true, COMPARE>(lin, {phib, T, first, p.s1, uout, Oout}, v, steps, O, match);
        }
        if (steps >= p.s1 || match.hit) break;
        int m = blocks.next(steps - before, p.s1 - steps);
        if (COMPARE) m = min(m, 16);
        const LogStepsResult r = log_steps(b, dir, dir == 0 ? first + steps : first - steps, m, v, O);
        v = r.v;
        O = r.O;
        steps += m;
        if constexpr (COMPARE) {
            if (steps < p.s1) {
                look_at_row(uout + (size_t)position(steps) * T, Oout[position(steps)], T, steps, v, O, match);
                if (match.hit) break;
            }
        }
    }
    if constexpr (COMPARE) {
        if (tid == 0) {
            a.matched_from[slot + c] = match.hit ? steps : kPieceUnmatched;
            a.deltas[slot + c] = match.delta;
        }
        if (match.hit) return;
    }
    float* uend = last && !COMPARE ? uout + (size_t)end * T : (COMPARE ? a.ends2 : a.ends) + (slot + c) * T;
    double* Oend = last && !COMPARE ? Oout + end : (COMPARE ? a.end_offsets2 : a.end_offsets) + slot + c;
    if (tid < T) uend[tid] = v;
    if (tid == 0) *Oend = O;
}

}  // namespace lccrf
