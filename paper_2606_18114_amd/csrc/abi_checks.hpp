// Host-side argument checks shared by the C ABI's translation units.  Every
// check runs before any HIP call, so a rejected call enqueues nothing.
#pragma once

#include <cmath>
#include <cstdint>

#include "../../include/tmamba.h"
#include "launchers.hpp"

namespace tmk_abi {

struct Span {
  uintptr_t lo = 0, hi = 0;  // [lo, hi)
};

inline bool bytes_of(int64_t a, int64_t b, int64_t elem, int64_t* out) {
  int64_t t;
  if (a < 0 || b < 0) return false;
  if (__builtin_mul_overflow(a, b, &t)) return false;
  if (__builtin_mul_overflow(t, elem, &t)) return false;
  if (t > (int64_t(1) << 46)) return false;  // 64 TiB: far beyond any device
  *out = t;
  return true;
}

inline Span span(const void* p, int64_t bytes) {
  Span s;
  s.lo = reinterpret_cast<uintptr_t>(p);
  s.hi = s.lo + static_cast<uintptr_t>(bytes);
  return s;
}

inline bool overlap(Span a, Span b) {
  if (a.lo == 0 || b.lo == 0 || a.hi == a.lo || b.hi == b.lo) return false;
  return a.lo < b.hi && b.lo < a.hi;
}

inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

inline bool group_ok(int32_t g) { return g == 32 || g == 64 || g == 128 || g == 256 || g == 512; }

inline tm_status shape_kg(int64_t K, int32_t g) {
  if (!group_ok(g)) return TM_ESHAPE;
  if (K < 1 || K % g != 0 || K % 64 != 0) return TM_ESHAPE;
  return TM_OK;
}

inline tm_status hip_status(hipError_t e) { return e == hipSuccess ? TM_OK : TM_EHIP; }

inline hipStream_t to_hip(tm_stream s) { return reinterpret_cast<hipStream_t>(s); }

constexpr int64_t kMaxGridBlocks = (int64_t(1) << 31) - 1;
constexpr int64_t kFwdTicketBytes = 8 * (int64_t)tmk::kFwdMaxTicketTiles;

// Y holds es-byte elements: 4 (float32) or 2 (bfloat16 bits)
// workspace NULL: the calls without one (cut tiles add with atomics)
inline tm_status fwd_checked(const uint16_t* X, const uint8_t* codes, const float* scales,
                             int64_t M, int64_t N, int64_t K, int32_t g, const void* Y, int es,
                             const void* workspace, int64_t workspace_bytes) {
  if (!X || !codes || !scales || !Y) return TM_EINVAL;
  if (M < 1 || N < 1) return TM_ESHAPE;
  if (tm_status st = shape_kg(K, g)) return st;
  int64_t xb, cb, sb, yb;
  if (!bytes_of(M, K, 2, &xb) || !bytes_of(N, K / 4, 1, &cb) || !bytes_of(N, K / g, 4, &sb) ||
      !bytes_of(M, N, es, &yb))
    return TM_ESHAPE;
  if (((M + 255) / 256) * ((N + 255) / 256) > kMaxGridBlocks) return TM_ESHAPE;
  if (K > (int64_t(1) << 22) || N > (int64_t(1) << 26)) return TM_ESHAPE;  // 32-bit tile offsets
  if (!aligned(X, 16) || !aligned(codes, 16) || !aligned(scales, 4) || !aligned(Y, 16))
    return TM_EALIGN;
  const Span y = span(Y, yb);
  if (overlap(y, span(X, xb)) || overlap(y, span(codes, cb)) || overlap(y, span(scales, sb)))
    return TM_EINVAL;
  if (workspace) {
    if (workspace_bytes < kFwdTicketBytes) return TM_ESHAPE;
    if (!aligned(workspace, 4)) return TM_EALIGN;
    const Span w = span(workspace, kFwdTicketBytes);
    if (overlap(w, y) || overlap(w, span(X, xb)) || overlap(w, span(codes, cb)) ||
        overlap(w, span(scales, sb)))
      return TM_EINVAL;
  }
  return TM_OK;
}

// argument checks of the dX calls; workspace NULL: the two-pass call, which
// takes none.  dY holds ye-byte elements (2: bfloat16 bits, 4: float32) and
// dX xe-byte ones (4: float32, 2: bfloat16 bits)
inline tm_status bwd_dx_checked(const void* dY, const uint8_t* codes, const float* scales,
                                int64_t M, int64_t N, int64_t K, int32_t g, const void* dX,
                                const void* workspace, int64_t workspace_bytes, int ye = 2,
                                int xe = 4) {
  if (!dY || !codes || !scales || !dX) return TM_EINVAL;
  if (M < 1 || N < 1 || N % 8 != 0) return TM_ESHAPE;
  if (tm_status st = shape_kg(K, g)) return st;
  if (N > (int64_t(1) << 22) || K > (int64_t(1) << 26)) return TM_ESHAPE;
  int64_t yb, cb, sb, xb;
  if (!bytes_of(M, N, ye, &yb) || !bytes_of(N, K / 4, 1, &cb) || !bytes_of(N, K / g, 4, &sb) ||
      !bytes_of(M, K, xe, &xb))
    return TM_ESHAPE;
  if (((M + 255) / 256) * ((K + 255) / 256) > kMaxGridBlocks) return TM_ESHAPE;
  if (!aligned(dY, 16) || !aligned(codes, 16) || !aligned(scales, 4) || !aligned(dX, 16))
    return TM_EALIGN;
  const Span o = span(dX, xb);
  if (overlap(o, span(dY, yb)) || overlap(o, span(codes, cb)) || overlap(o, span(scales, sb)))
    return TM_EINVAL;
  if (workspace) {
    const int64_t need = tmk::dx_f16_workspace_bytes(M, N);
    if (workspace_bytes < need) return TM_ESHAPE;
    if (!aligned(workspace, 256)) return TM_EALIGN;
    const Span w = span(workspace, need);
    if (overlap(w, o) || overlap(w, span(dY, yb)) || overlap(w, span(codes, cb)) ||
        overlap(w, span(scales, sb)))
      return TM_EINVAL;
  }
  return TM_OK;
}

inline tm_status bwd_dw_checked(const uint16_t* dY, const uint16_t* X, int64_t M, int64_t N,
                                int64_t K, const float* dW, int32_t accumulate) {
  if (!dY || !X || !dW) return TM_EINVAL;
  if (accumulate != 0 && accumulate != 1) return TM_EINVAL;
  if (M < 1 || N < 1 || N % 8 != 0 || K < 1 || K % 64 != 0) return TM_ESHAPE;
  int64_t yb, xb, wb;
  if (!bytes_of(M, N, 2, &yb) || !bytes_of(M, K, 2, &xb) || !bytes_of(N, K, 4, &wb))
    return TM_ESHAPE;
  if (((N + 255) / 256) * ((K + 255) / 256) * ((M + 255) / 256) > kMaxGridBlocks) return TM_ESHAPE;
  if (N > (int64_t(1) << 26) || K > (int64_t(1) << 26)) return TM_ESHAPE;  // 32-bit row offsets
  if (!aligned(dY, 16) || !aligned(X, 16) || !aligned(dW, 16)) return TM_EALIGN;
  const Span o = span(dW, wb);
  if (overlap(o, span(dY, yb)) || overlap(o, span(X, xb))) return TM_EINVAL;
  return TM_OK;
}

// argument checks of the mixer step; workspace NULL: the library's own
// scratch array (no overlap check needed: no caller array can overlap it)
// gate_only: the gated float32 output of tm_mixer_gate in place of the
// normalized bfloat16 one (no norm_w, eps or workspace)
inline tm_status mixer_checked(const float* zxbcdt, int32_t B, int32_t nheads, int32_t headdim,
                        int32_t d_state, uint16_t* conv_state, int32_t* conv_pos,
                        uint16_t* ssm_state, const float* conv_w, const float* conv_b,
                        const float* dt_bias, const float* A_log, const float* D,
                        const float* norm_w, float eps, float* workspace, const void* out,
                        bool gate_only = false) {
  if (!zxbcdt || !conv_state || !conv_pos || !ssm_state || !conv_w || !conv_b || !dt_bias ||
      !A_log || !D || (!gate_only && !norm_w) || !out)
    return TM_EINVAL;
  if (!gate_only && (!(eps >= 0.0f) || !std::isfinite(eps))) return TM_EINVAL;
  if (B < 1 || B > 65535 || nheads < 1 || nheads > 4096 || headdim != 64 || d_state != 128)
    return TM_ESHAPE;
  const int64_t di = (int64_t)nheads * headdim, cd = di + 2 * (int64_t)d_state;
  const int64_t zw = 2 * di + 2 * (int64_t)d_state + nheads;
  int64_t zb, cb, sb, wb, ob;
  if (!bytes_of(B, zw, 4, &zb) || !bytes_of((int64_t)B * cd, 4, 2, &cb) ||
      !bytes_of((int64_t)B * nheads * headdim, d_state, 2, &sb) ||
      !bytes_of(B, di + nheads, 4, &wb) || !bytes_of(B, di, gate_only ? 4 : 2, &ob))
    return TM_ESHAPE;
  if (!aligned(zxbcdt, 4) || !aligned(conv_state, 8) || !aligned(conv_pos, 4) ||
      !aligned(ssm_state, 16) || !aligned(conv_w, 4) || !aligned(conv_b, 4) ||
      !aligned(dt_bias, 4) || !aligned(A_log, 4) || !aligned(D, 4) || !aligned(norm_w, 4) ||
      !aligned(workspace, 4) || !aligned(out, gate_only ? 4 : 2))
    return TM_EALIGN;
  const Span outs[5] = {span(conv_state, cb), span(conv_pos, 4), span(ssm_state, sb),
                        span(workspace, workspace ? wb : 0), span(out, ob)};
  const Span ins[7] = {span(zxbcdt, zb), span(conv_w, cd * 16), span(conv_b, cd * 4),
                       span(dt_bias, (int64_t)nheads * 4), span(A_log, (int64_t)nheads * 4),
                       span(D, (int64_t)nheads * 4), span(norm_w, norm_w ? di * 4 : 0)};
  for (int i = 0; i < 5; ++i) {
    for (int j = i + 1; j < 5; ++j)
      if (overlap(outs[i], outs[j])) return TM_EINVAL;
    for (const Span& in : ins)
      if (overlap(outs[i], in)) return TM_EINVAL;
  }
  return TM_OK;
}

}  // namespace tmk_abi
