/*
 * libburstattn -- diagnostics.  Not part of the attention path: host-side views of the kernels' tile
 * logic for tests, and a matrix-core ceiling probe for benchmarks.  Conventions as in burst_attn.h.
 */
#ifndef BURST_ATTN_DIAG_H
#define BURST_ATTN_DIAG_H

#include "burst_attn.h"
#include "burst_lm_head.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Host diagnostics of the tile-level mask logic, running the very code the kernels compile (no GPU
 * involved), so that tests can hold it against a brute-force visibility matrix.
 *
 * burst_attn_tile_class: class of the block of query rows [q0, q1) against key rows [k0, k1):
 * 0 = no pair visible (the kernels skip the tile), 1 = every pair visible (no per-element predicate),
 * 2 = mixed.  method 0: the direct position-range test (launch plan); 1: the query tile [q0, q1) as a dK/dV
 * wave that owns the keys [k0, k1) classifies it while it walks (TileRanges); 2: the key tile [k0, k1) as a
 * forward or dQ wave that owns the query rows [q0, q1) does.  These three must agree.  3 and 4: as 1 and 2 with a
 * tile of 64 rows from q0 or k0 on, as the kernels have it at the end of a chunk: never 1 where rows are missing.
 * Negative burst_status_t on a bad argument.
 *
 * burst_attn_visible_rows: the rows [out[0], out[1]) of the query axis that see key row `row` (query_axis !=
 * 0), or of the key axis that query row `row` sees; the interval is empty where out[0] >= out[1].  It is what a lane compares
 * with, row by row, in a mixed tile.  The block mask is not part of it.
 *
 * burst_attn_visible_tile_runs: the tiles of `tile_rows` rows along the query axis (query_axis != 0;
 * tile_rows 64 or 256) or the key axis (tile_rows 64 or 128) that can hold a pair visible to rows
 * [r0, r1) of the other axis: one run, out = {start, length, 0, 0} in tiles. */
int burst_attn_tile_class(const burst_mask_t* mask, int64_t q0, int64_t q1, int64_t k0, int64_t k1, int32_t method);
int burst_attn_visible_rows(const burst_mask_t* mask, int32_t query_axis, int64_t row, int32_t out_lo_hi[2]);
int burst_attn_visible_tile_runs(const burst_mask_t* mask, int32_t query_axis, int32_t tile_rows, int64_t r0, int64_t r1,
                                 int32_t out_start_len[4]);

/* Diagnostic, not part of the attention path: enqueues `iterations` x 8 independent bf16 16x16x32
 * MFMAs (the kernels' shape) per wave on every SIMD (512 work-groups of 256 threads) with constant (0) or pseudo-random
 * (1) register operands, and stores the flop count of the launch in *flops_out (host, optional).
 * Timed by the caller with events, it gives the matrix-core ceiling of the chip as it is clocked under
 * that load: dense attention tiles are bounded by the random-operand figure.  sink: optional device
 * pointer to 4 bytes (never written in practice).  iterations in [1, 2^24]. */
int burst_attn_mfma_probe(int32_t random_operands, int32_t iterations, float* sink, int64_t* flops_out,
                          void* hip_stream);

/* The step kernels cut a streamed axis (keys for the forward kernel when it only updates the running state,
 * and for dQ; queries for dK / dV) that is longer than twice `rows` into ranges of about `rows` rows, one
 * launch per range (an L2-locality measure; default 32768).  Tests lower it to drive the chunked path at sizes
 * the oracle can check exhaustively.  Process-wide; values below 256 are raised to 256.  Returns the value now
 * in force. */
int burst_attn_set_chunk_rows(int32_t rows);

/* Host view of that plan (no GPU involved): the ranges of local rows the query axis (query_axis != 0: the
 * dK/dV kernel's launches) or the key axis (the dQ kernel's and the forward kernel's) of a step with this mask is cut into.  Returns
 * the number of ranges (negative burst_status_t on a bad mask) and fills, for the first max_ranges of them,
 * out[7 i ..] = {first row, end row, pieces, rows per piece, position of the first row, position period of
 * the pieces, byte offset of the range's block mask from the step's} -- the chunk the range's launch
 * describes to the kernel.  One range means one launch with the step's own mask. */
int burst_attn_chunk_plan(const burst_mask_t* mask, int32_t query_axis, int32_t max_ranges, int64_t* out);

/* Host view of the launches of step kernels that a call with these steps makes (no GPU involved): which kernel each of them takes.
 * call: 0 forward steps into the running state, 1 one forward step with a result of its own, 2 backward steps, 3 the same for dQ
 * alone, 4 for dK and dV alone.  The steps have the same query side.  Returns the number of launches (negative burst_status_t on a bad
 * argument) and fills out[i], for the first max_launches of them, with the bits below: 0 is a forward launch, DQ and DKDV say what a
 * backward launch computes. */
#define BURST_KERNEL_DQ 1
#define BURST_KERNEL_DKDV 2
#define BURST_KERNEL_DEALT 4          /* the four waves of a work-group share 32 rows and deal the walk among themselves */
#define BURST_KERNEL_SHARED_CU 8      /* head_dim 64, dK/dV: two work-groups of eight waves per CU */
#define BURST_KERNEL_KEY_TILES_64 16  /* dK/dV: key tiles of 64 rows instead of 128 */
int burst_attn_launch_plan(int32_t call, int32_t n_steps, const burst_shape_t* shapes, const burst_mask_t* masks,
                           int32_t max_launches, int32_t* out);

/* Host view of the LM head's products over the first sequence tile of a call with this shape (tile_tokens as given; no GPU involved): for
 * the logits, dH and dW the edge of an output tile (128 or 256) and the parts its contraction is split in, out = {edge, parts} x 3. */
int burst_lm_head_tile_plan(const burst_lm_head_shape_t* shape, int32_t out[6]);

#ifdef __cplusplus
}
#endif
#endif /* BURST_ATTN_DIAG_H */
