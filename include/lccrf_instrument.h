/*
 * lccrf_instrument.h - benchmark instrumentation of the linear-chain CRF library.
 *
 * Not part of the query interface (include/lccrf.h): what is declared here exists so that a
 * benchmark can time the two passes of lccrf_marginals separately on the launch stream.
 */
#ifndef LCCRF_INSTRUMENT_H
#define LCCRF_INSTRUMENT_H

#include "lccrf.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * lccrf_marginals_algo (section "Computing Marginals" of the paper, Eq. 3-4) with three
 * caller-created hipEvent_t handles (passed as void*, any may be NULL) recorded on `stream`
 * before the first kernel, between the two passes of the sequential schedule (after every
 * matrix has been read once and the half-way vectors are stored, or, where lccrf_marginals_by_edges says so, twice and the
 * vectors of every position; before the pass that
 * re-reads phi and writes the marginals), and after the last kernel.  Lets a caller time the
 * passes separately with hipEventElapsedTime.  Same results and errors as lccrf_marginals_algo.
 */
int lccrf_marginals_timed(const void* phi, lccrf_dtype dt, const int32_t* lengths,
                          int B, int N, int T, float* logZ, float* marginals,
                          void* workspace, size_t workspace_bytes, void* stream, lccrf_algo algo,
                          void* ev_begin, void* ev_between, void* ev_end);

/*
 * Streaming probe: `workgroups` workgroups of 1024 threads each read a contiguous share of in[0 .. bytes)
 * in 16-byte accesses with four loads in flight per thread, the access pattern of the chain kernels
 * (one workgroup per chain, one tile per position), and, if `out` is non-NULL, write every vector to
 * the same place in out.  Timed by the caller, it gives the bandwidth that many workgroups can draw:
 * the practical ceiling for a batch with that many chains, beside the datasheet peak.
 *   in, out   device buffers of `bytes` bytes, 16-byte aligned (out may be NULL: read only)
 *   sink      one device float (keeps the reads alive; never written for real data)
 * The bytes actually covered are lccrf_stream_probe_bytes(bytes, workgroups) (whole rounds of 64 KiB per
 * workgroup; 0 if bytes is too small for one round each, which lccrf_stream_probe refuses with
 * LCCRF_EINVAL).  Enqueues one kernel on `stream`; errors as the queries.
 */
int lccrf_stream_probe(const void* in, void* out, size_t bytes, int workgroups, float* sink, void* stream);
size_t lccrf_stream_probe_bytes(size_t bytes, int workgroups);

/*
 * 1 where the default schedule of lccrf_marginals, in place of a second pass that writes the marginals as the chains go, runs
 * the chains of the first one to the far ends (two reads of phi) and writes every edge in a kernel of its own (a third).
 * 0 elsewhere, or without a device.  (At 128 tags 0, though AUTO does the same with chains that it walks in pieces.)
 */
int lccrf_marginals_by_edges(lccrf_dtype dt, int B, int T);

/*
 * How many pieces, walked by a workgroup each, the default schedule of lccrf_log_partition, lccrf_marginals, lccrf_log_prob or lccrf_sample
 * cuts a chain into at most (1: none; 65 .. 256 tags only).  *plan (may be NULL): where in the workspace a call leaves what became of
 * that, int32 [2 B][pieces], chain 2 b forward and 2 b + 1 backward.  Entry 0: twice the least steps of a piece, one more if the chain takes
 * no steps in scaled probabilities; 2^21 and more: the batch was not cut.  Entry c > 0: the step from which piece c stands as it was
 * walked without its predecessor, 2^31 - 1 if the chain was walked again from its end on.  (Sampling overwrites it.)  0 without pieces.
 * LCCRF_EINVAL for other queries and shapes that are not served.
 */
int lccrf_first_pass_pieces(lccrf_op op, lccrf_dtype dt, int B, int N, int T, size_t* plan);

/*
 * The largest row of a T x T matrix that any thread of a first pass in scaled probabilities (33 .. 256 tags) takes, by the
 * kernels' own arithmetic over every thread and item of the instance the dispatch chooses: at most T - 1, or the pass
 * reads past the matrix.  Host only; -1 for other tag counts.
 */
int lccrf_first_pass_largest_row(int T);

#ifdef __cplusplus
}
#endif
#endif /* LCCRF_INSTRUMENT_H */
