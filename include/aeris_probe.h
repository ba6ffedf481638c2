/*
 * aeris_probe.h -- aids for measuring and testing shipped with the shifted-window attention
 * library; not part of its paths and not needed by its callers.
 */
#ifndef AERIS_PROBE_H
#define AERIS_PROBE_H

#include <stdint.h>

#include "aeris_winattn.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * bench.py uses this one to report, next to the fraction of the published MFMA peak, the fraction
 * of the MFMA rate this machine sustains under its power limit.
 * Launches `blocks` workgroups of 256 threads, each wave issuing
 * 8 * iters v_mfma_f32_32x32x16_bf16 on register operands (32768 FLOP each) and nothing else.
 * random_operands != 0 fills the operands with pseudo-random bf16 values of unit scale, else
 * with small integers.  sink: device buffer of blocks * 256 floats, overwritten.
 * 1 <= blocks <= 65536, 1 <= iters.  FLOPs of a launch: blocks * 4 * iters * 8 * 32768.
 */
int aeris_mfma_loop_probe(int32_t blocks, int32_t iters, int32_t random_operands, float* sink,
                          void* hip_stream);

/*
 * How attention calls run a parameter block they accept (else its error code), with n_windows listed
 * windows, or all of them (0).  *forward: the workgroups that share the queries of a (batch, window, head)
 * whose keys and values each holds whole; 0: tiles of 128 or 256 queries with streamed keys.  *backward:
 * 0: one kernel makes dQ, dK and dV of a window and head; else a dQ kernel and one for dK and dV, which is
 * 1: the generic one, operands read first, 2: the same, operands read one block of products ahead, 3: the
 * software-pipelined one.  Launches nothing.
 */
int aeris_winattn_plan(const aeris_winattn_params* p, int32_t n_windows, int32_t* forward, int32_t* backward);

/*
 * How the projections (aeris_linear_fwd; with several samples aeris_norm_linear_fwd, gated != 0
 * aeris_norm_linear_swiglu_fwd, features = rows of the weight) are computed at a size they accept,
 * else their error code: *tile, the sides of the workgroup tiles (256, 128 or 64); *in_turn, whether
 * the XCDs take the token tiles in turn (1) or contiguous ranges of all tiles (0).
 */
int aeris_projection_plan(int64_t n_rows, int64_t rows_per_sample, int32_t channels, int32_t features,
                          int32_t gated, int32_t* tile, int32_t* in_turn);

/*
 * How aeris_linear_bwd computes dweight at a size it accepts (else its error code): *tile, the
 * sides of its square workgroup tiles (256, 128 or 64); *ranges, the row ranges whose partial
 * results are added; *steps, the steps of 64 rows in each but the last.  Launches nothing.
 */
int aeris_linear_bwd_plan(int64_t n_rows, int32_t channels, int32_t out_features, int32_t* tile,
                          int32_t* ranges, int32_t* steps);

#ifdef __cplusplus
}
#endif
#endif /* AERIS_PROBE_H */
