/*
 * libspecvla_verify - measurement and inspection aids.  Nothing here is part of the
 * verification path (include/specvla_verify.h); benchmarks and tests use these calls to look
 * inside it.  Same conventions: plain C, [host] / [device] tags, int status, the caller owns
 * every buffer.
 */
#ifndef SPECVLA_VERIFY_AUX_H
#define SPECVLA_VERIFY_AUX_H

#include "specvla_verify.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Host-only inspection aid for tests: where an intermediate of the last sv_verify_layer call
 * lives inside the workspace.  which = SV_WS_ATTN_OUT: attention output before the output
 * projection, float32 [B*T, nh*d].  which = SV_WS_Q: rotated queries, float32 [B*T, nh*d].
 * which = SV_WS_STATUS: one int32 (bytes = 0 for SV_F32 models), zero unless the workgroups that
 * share an output along K ran on different XCDs (bit 0) or waited for each other in vain (bit 1) -
 * the placement that their exchange through one XCD's cache relies on is checked in every launch;
 * non-zero means results are suspect.  Cleared by sv_workspace_init. */
#define SV_WS_ATTN_OUT 0
#define SV_WS_Q 1
#define SV_WS_STATUS 2
int sv_workspace_region(const sv_model_cfg *cfg, int B, int T, int n_scored, int which,
                        size_t *offset, size_t *bytes);

/* Host-only inspection aid for tests and benchmarks: how a product of a bf16 model is split over a device of
 * n_xcd XCDs (1 .. 8) for n_rows rows of activations.  which: SV_PLAN_*; n_scored: rows of the packed head
 * (SV_PLAN_HEAD only).  plan: [host, out] int32[6]: kernel (0 gemm_skinny, 1 gemm_mid, 2 gemm_thin), 32-row
 * blocks of activations a workgroup multiplies (gemm_thin: half of the one), weight tiles of the kernel instance (per
 * workgroup, gemm_mid: per wave), slices along K, column groups per XCD, workgroups that share the rows of a column
 * group out.  Rows multiplied, padding included: 32 * plan[1] * plan[5], gemm_thin: 16.
 * SV_ERR_DTYPE for SV_F32, SV_ERR_SHAPE for other sizes out of range. */
#define SV_PLAN_QKV 0
#define SV_PLAN_OUT 1
#define SV_PLAN_GATE_UP 2
#define SV_PLAN_DOWN 3
#define SV_PLAN_HEAD 4
int sv_product_plan(const sv_model_cfg *cfg, int n_rows, int which, int n_scored, int n_xcd,
                    int32_t *plan);

/* Measurement aid: sv_verify_layer - the same launches - with the caller's HIP events recorded on
 * `stream` between them, so that a benchmark can read durations with hipEventElapsedTime:
 * events[0],[1] bracket the q/k/v product, [2],[3] the tree attention (with the launch that merges
 * its splits, if there are any), [3],[4] the output product, [5],[6] the gate/up product, [7],[8]
 * the down product.
 * events: [host] array of SV_N_TIMING_EVENTS hipEvent_t (created by the caller with timing
 * enabled).  SV_ERR_NULL if the array or an entry is NULL. */
#define SV_N_TIMING_EVENTS 9
int sv_verify_layer_timed(const sv_model_cfg *cfg, const void *packed, float *x,
                          const sv_kv_view *kv, const sv_tree *tree, int B, void *workspace,
                          size_t ws_bytes, void *stream, void *const *events);

/* Measurement aid, no part of the verification path: reads `bytes` of device memory once with
 * the access pattern of the weight stream (16-byte non-temporal loads, 1 KiB per wave and
 * instruction, 8 KiB per wave in flight) and discards the data.  bench.py times it to report
 * the streaming-read rate the GPU reaches next to its data-sheet HBM peak.
 *   ptr: [device], 16-byte aligned, bytes a multiple of 16;  sink: [device] 16 bytes, 16-byte
 *   aligned (written only for one data pattern in 2^96)
 * SV_ERR_SHAPE for sizes or alignments outside that. */
int sv_stream_read(const void *ptr, size_t bytes, void *sink, void *stream);

#ifdef __cplusplus
}
#endif
#endif /* SPECVLA_VERIFY_AUX_H */
