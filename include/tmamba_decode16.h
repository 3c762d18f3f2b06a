/*
 * tmamba_decode16.h — the three calls of a decode layer for batches of 5 to
 * 16 rows, whose normalizations need no launch of their own: a call takes the
 * partial sums of squares that the one before left, or sums the squares
 * itself.  Shapes, layouts and status codes as in tmamba.h.
 */
#ifndef TMAMBA_DECODE16_H
#define TMAMBA_DECODE16_H

#include "tmamba.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * part[b] = sum of the squares of row b of src [B, D]; dst (NULL or [B, D],
 * not overlapping src) receives a copy of src.
 */
tm_status tm_rows_sumsq(const float* src, int32_t B, int64_t D, float* dst, float* part,
                        tm_stream stream);

/*
 * x = bf16(src / sqrt(sum(part) / K + eps) * norm_w) per batch row (B <= 16,
 * part [B, nparts]; NULL with nparts = 0: the squares of src are summed by this
 * call), y [B, N] = x . What^T, or += it with accumulate = 1; g = 64, 128 or
 * 256, K <= 4096.  With B >= 9 the sums are taken in the order of tm_tgemv,
 * and the squares, with part NULL, in that of tm_residual_rmsnorm: the same
 * bits as those two calls.  part_out (NULL or [B, ceil(N / 16)]): partial sums
 * of the squares of y as written.  advance (NULL or a mixer's conv_pos): the
 * ring position moves on by one slot.
 */
tm_status tm_tgemv_rms16(const float* src, const float* part, int32_t nparts,
                         const float* norm_w, float eps, const uint8_t* codes,
                         const uint16_t* scales_f16, int32_t B, int64_t N, int64_t K, int32_t g,
                         float* y, int32_t accumulate, float* part_out, int32_t* advance,
                         tm_stream stream);

/*
 * tm_mixer_gate with the heads' sums of the squares of gated in partial
 * [B, nheads]; conv_pos is read and left as it is.
 */
tm_status tm_mixer_gate_part(const float* zxbcdt, int32_t B, int32_t nheads, int32_t headdim,
                             int32_t d_state, uint16_t* conv_state, const int32_t* conv_pos,
                             uint16_t* ssm_state, const float* conv_w, const float* conv_b,
                             const float* dt_bias, const float* A_log, const float* D,
                             float* gated, float* partial, tm_stream stream);

#ifdef __cplusplus
}
#endif

#endif /* TMAMBA_DECODE16_H */
