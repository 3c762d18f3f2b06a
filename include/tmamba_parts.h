/*
 * tmamba_parts.h — the training products of tmamba.h with a second scratch
 * buffer and the element types of a mixed-precision layer.
 *
 * slots: float32 scratch through which the parts of output tiles that are cut
 * along the contraction meet (16-byte aligned).  The *_slots functions give
 * its size for a shape on the current device: 0 where no tile is cut, -1 for
 * sizes the call rejects.  With NULL the parts add up by atomics in the
 * output itself (float32 outputs only; slower where an output has few tiles).
 * The scratch is free again when the call's kernels are done; nothing in it
 * outlives the call.  Everything not said here is as in tmamba.h.
 */
#ifndef TMAMBA_PARTS_H
#define TMAMBA_PARTS_H

#include "tmamba.h"

#ifdef __cplusplus
extern "C" {
#endif

/* the larger of the two tm_tgemm_fwd_scratch */
int64_t tm_tgemm_fwd_slots(int64_t M, int64_t N, int64_t K, int32_t g);
int64_t tm_tgemm_fwd_scratch(int64_t M, int64_t N, int64_t K, int32_t g, int32_t y_bf16);
int64_t tm_tgemm_bwd_dx_slots(int64_t M, int64_t N, int64_t K, int32_t exact);
int64_t tm_tgemm_bwd_dw_slots(int64_t M, int64_t N, int64_t K);

/*
 * Y = X . What^T in float32 (y_bf16 = 0) or rounded once to bfloat16
 * (y_bf16 = 1), on the tile shape and cut that suit the sizes.  workspace:
 * NULL, or that of tm_tgemm_fwd_ws (float32 only).  slots (at least
 * tm_tgemm_fwd_scratch bytes): the parts' slots, or, where two parts meet in Y,
 * the words they take turns with if there is no workspace.  With slots, or
 * where none are needed, two calls give the same bits.
 */
tm_status tm_tgemm_fwd_parts(const uint16_t* X, const uint8_t* codes, const float* scales,
                             int64_t M, int64_t N, int64_t K, int32_t g, void* Y, int32_t y_bf16,
                             void* workspace, int64_t workspace_bytes, float* slots,
                             int64_t slots_bytes, tm_stream stream);

/*
 * dX[M, K] = dY . What in float32 (dx_bf16 = 0) or rounded once to bfloat16
 * (dx_bf16 = 1; slots are then needed where a tile is cut).  exact = 0: the
 * one-pass float16 form, which needs workspace
 * (tm_tgemm_bwd_dx_f16_workspace bytes); exact = 1: the two-pass form, whose
 * workspace is NULL.  dy_f32 = 1 (exact = 0 only): dY is float32 and its
 * rounding to bfloat16 is also written to dY_bf16 [M, N]; else dY is bfloat16
 * and dY_bf16 NULL.
 */
tm_status tm_tgemm_bwd_dx_parts(const void* dY, int32_t dy_f32, uint16_t* dY_bf16,
                                const uint8_t* codes, const float* scales, int64_t M, int64_t N,
                                int64_t K, int32_t g, int32_t exact, void* dX, int32_t dx_bf16,
                                void* workspace, int64_t workspace_bytes, float* slots,
                                int64_t slots_bytes, tm_stream stream);

/* tm_tgemm_bwd_dw_ste with slots. */
tm_status tm_tgemm_bwd_dw_parts(const uint16_t* dY, const uint16_t* X, int64_t M, int64_t N,
                                int64_t K, float* dW, int32_t accumulate, float* slots,
                                int64_t slots_bytes, tm_stream stream);

#ifdef __cplusplus
}
#endif

#endif /* TMAMBA_PARTS_H */
