// C ABI of tmamba_decode16.h: argument checks, then one launcher.
#include "../../include/tmamba_decode16.h"

#include "abi_checks.hpp"

using namespace tmk_abi;

extern "C" {

tm_status tm_rows_sumsq(const float* src, int32_t B, int64_t D, float* dst, float* part,
                        tm_stream stream) {
  if (!src || !part) return TM_EINVAL;
  int64_t b;
  if (B < 1 || B > 65535 || D < 1 || !bytes_of(B, D, 4, &b)) return TM_ESHAPE;
  if (!aligned(src, 4) || !aligned(dst, 4) || !aligned(part, 4)) return TM_EALIGN;
  const Span s = span(src, b), d = span(dst, dst ? b : 0), p = span(part, (int64_t)B * 4);
  if (overlap(s, d) || overlap(s, p) || overlap(d, p)) return TM_EINVAL;
  return hip_status(tmk::launch_rows_sumsq(src, B, D, dst, part, to_hip(stream)));
}

tm_status tm_tgemv_rms16(const float* src, const float* part, int32_t nparts,
                         const float* norm_w, float eps, const uint8_t* codes,
                         const uint16_t* scales_f16, int32_t B, int64_t N, int64_t K, int32_t g,
                         float* y, int32_t accumulate, float* part_out, int32_t* advance,
                         tm_stream stream) {
  if (!src || !norm_w || !codes || !scales_f16 || !y) return TM_EINVAL;
  if (!(eps >= 0.0f) || !std::isfinite(eps) || (accumulate & ~1)) return TM_EINVAL;
  if (B < 1 || B > 16 || N < 1 || N > (int64_t(1) << 26)) return TM_ESHAPE;
  if (part ? nparts < 1 : nparts != 0) return TM_ESHAPE;
  if (tm_status st = shape_kg(K, g)) return st;
  if (g < 64 || g > 256 || K > tmk::kRms16MaxK) return TM_ESHAPE;
  int64_t xb, wb, cb, sb, yb, pb;
  if (!bytes_of(B, K, 4, &xb) || !bytes_of(1, K, 4, &wb) || !bytes_of(N, K / 4, 1, &cb) ||
      !bytes_of(N, K / g, 2, &sb) || !bytes_of(B, N, 4, &yb) || !bytes_of(B, nparts, 4, &pb))
    return TM_ESHAPE;
  if (!aligned(src, 16) || !aligned(part, 4) || !aligned(norm_w, 16) || !aligned(codes, 16) ||
      !aligned(scales_f16, 2) || !aligned(y, 4) || !aligned(part_out, 4) || !aligned(advance, 4))
    return TM_EALIGN;
  const Span ins[5] = {span(src, xb), span(part, part ? pb : 0), span(norm_w, wb), span(codes, cb),
                       span(scales_f16, sb)};
  const Span outs[3] = {span(y, yb), span(part_out, part_out ? B * ((N + 15) / 16) * 4 : 0),
                        span(advance, advance ? 4 : 0)};
  for (int i = 0; i < 3; ++i) {
    for (const Span& in : ins)
      if (overlap(outs[i], in)) return TM_EINVAL;
    for (int j = i + 1; j < 3; ++j)
      if (overlap(outs[i], outs[j])) return TM_EINVAL;
  }
  return hip_status(tmk::launch_tgemv_rms16(src, part, nparts, norm_w, eps, codes, scales_f16, B,
                                            N, K, g, y, accumulate, part_out, advance,
                                            to_hip(stream)));
}

tm_status tm_mixer_gate_part(const float* zxbcdt, int32_t B, int32_t nheads, int32_t headdim,
                             int32_t d_state, uint16_t* conv_state, const int32_t* conv_pos,
                             uint16_t* ssm_state, const float* conv_w, const float* conv_b,
                             const float* dt_bias, const float* A_log, const float* D,
                             float* gated, float* partial, tm_stream stream) {
  if (!partial) return TM_EINVAL;
  if (tm_status st = mixer_checked(zxbcdt, B, nheads, headdim, d_state, conv_state,
                                   const_cast<int32_t*>(conv_pos), ssm_state, conv_w, conv_b,
                                   dt_bias, A_log, D, nullptr, 0.f, nullptr, gated, true))
    return st;
  if (!aligned(partial, 4)) return TM_EALIGN;
  const int64_t h = nheads, di = 64 * h, cd = di + 256;
  const Span p = span(partial, B * h * 4);
  const Span others[10] = {span(zxbcdt, B * (2 * di + 256 + h) * 4), span(conv_state, B * cd * 8),
                           span(conv_pos, 4), span(ssm_state, B * di * 256),
                           span(gated, B * di * 4), span(conv_w, cd * 16), span(conv_b, cd * 4),
                           span(dt_bias, h * 4), span(A_log, h * 4), span(D, h * 4)};
  for (const Span& o : others)
    if (overlap(p, o)) return TM_EINVAL;
  return hip_status(tmk::launch_mixer_gate_part(zxbcdt, B, nheads, conv_state, conv_pos,
                                                ssm_state, conv_w, conv_b, dt_bias, A_log, D,
                                                gated, partial, to_hip(stream)));
}

}  // extern "C"
