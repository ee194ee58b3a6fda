/*
 * Measurement probes of libqllm: no part of the method and no part of its boundary.  They exist for callers
 * (the benchmark) that price the two hot kernels against what the machine delivers, next to the data-sheet
 * peaks.  DEVICE pointers; all conventions as in qllm.h.
 */
#ifndef QLLM_PROBES_H
#define QLLM_PROBES_H

#include <stdint.h>

#include "qllm.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 *   qllm_probe_mfma    `workgroups` workgroups of 8 waves; every wave issues iters * 32 int8 matrix-core
 *                      operations (16 x 16 x 64 each, i.e. 2 * 16384 integer operations) on register
 *                      operands shaped like 4-bit codes and touches no memory.  sink: one device int32.
 *   qllm_probe_mfma_fp6  the same shape of loop with FP6 (E2M3) matrix-core operations, 16 x 16 x 128 each, on
 *                      operands whose 6-bit fields hold 4-bit codes.  sink: one device float.
 *   qllm_probe_stream  reads `bytes` (a multiple of 16) from src and writes bytes / 4 to dst: the 4 : 1
 *                      read : write mix of the fused kernel with bf16 input and 4-bit codes.
 * Errors: NULL / SHAPE / ALIGN (src 16-byte, dst 4-byte aligned) / HIP.
 */
int32_t qllm_probe_mfma(int32_t workgroups, int32_t iters, int32_t *sink, void *hip_stream);
int32_t qllm_probe_mfma_fp6(int32_t workgroups, int32_t iters, float *sink, void *hip_stream);
int32_t qllm_probe_stream(const void *src, void *dst, int64_t bytes, int32_t workgroups, void *hip_stream);

/*
 * What the fused kernel of qllm_reassembled_linear does for a map, a weight and N > 0 tokens (no launch; of the weight only O, K,
 * bits and whether tiles6 / tiles8 are NULL are read, x is taken as 16-byte aligned with rows of ldx elements).
 *   form             QLLM_FUSED_*
 *   laid_out         1: it writes the codes as the product reads them, and the workspace's packed rows stay as they were
 *   chunks_per_lane, lanes   the shape of a row's workgroup (0 where it walks the map)
 *   empty_pass       1: every workgroup puts out a row of nothing before its first one
 *   ahead_bytes      how much of the weight's re-laid copy idle CUs read ahead of the product
 * Errors: NULL / SHAPE / BITS / DTYPE / MAP / WORKSPACE.
 */
typedef struct {
    int32_t form, laid_out, chunks_per_lane, lanes, empty_pass;
    int64_t ahead_bytes;
} qllm_layer_launch;
int32_t qllm_probe_layer_launch(const qllm_map *map, int32_t x_dtype, int64_t N, int64_t ldx, int32_t norm, int32_t has_beta,
                                int32_t a_bits, const qllm_weight *w, int64_t workspace_bytes, qllm_layer_launch *out);

/*
 * The mid-size tiles, *tokens x *features, that qllm_int_gemm, or the product of the layer call, runs one round of; 0 x 0 where it
 * takes another kernel.  Arguments and errors as of qllm_gemm_kernel_choice, whose *tile does not tell them apart.  Returns QLLM_OK
 * or a QLLM_ERR_*.
 */
int32_t qllm_probe_mid_tile(const qllm_weight *w, int32_t a_bits, int64_t N, int64_t workspace_bytes, int32_t in_layer,
                            int32_t *tokens, int32_t *features);

/*
 * One half of qllm_reassembled_linear with the same arguments, to be timed by itself: 1 the fused kernel, 2 the product (the
 * workspace as half 1 left it).  Half 1 then half 2 is the layer call.  Errors: those of qllm_reassembled_linear, SHAPE for any
 * other half.
 */
int32_t qllm_probe_layer_half(int32_t half, const void *x, int32_t x_dtype, int64_t N, int64_t C, int64_t ldx, int32_t norm,
                              const float *gamma, const float *beta, float eps, const qllm_map *map, int32_t a_bits,
                              const qllm_weight *w, void *y, int32_t y_dtype, int64_t ldy, void *workspace,
                              int64_t workspace_bytes, void *hip_stream);

#ifdef __cplusplus
}
#endif
#endif /* QLLM_PROBES_H */
