// C ABI of tmamba_parts.h: argument checks, then one launcher.
#include "../../include/tmamba_parts.h"

#include "abi_checks.hpp"

namespace {

using namespace tmk_abi;

// the scratch buffer against its size and the other operands
tm_status slots_checked(const float* slots, int64_t bytes, int64_t need, const Span* others,
                        int n) {
  if (!slots) return TM_OK;
  if (bytes < need) return TM_ESHAPE;
  if (!aligned(slots, 16)) return TM_EALIGN;
  const Span s = span(slots, need);
  for (int i = 0; i < n; ++i)
    if (overlap(s, others[i])) return TM_EINVAL;
  return TM_OK;
}

bool sizes_ok(int64_t M, int64_t N, int64_t K) {
  int64_t b;
  return M >= 1 && N >= 1 && K >= 1 && bytes_of(M, N, 4, &b) && bytes_of(M, K, 4, &b) &&
         bytes_of(N, K, 4, &b);
}

}  // namespace

extern "C" {

int64_t tm_tgemm_bwd_dx_slots(int64_t M, int64_t N, int64_t K, int32_t exact) {
  if (!sizes_ok(M, N, K)) return -1;
  return exact ? tmk::bwd_dx_slot_bytes(M, N, K) : tmk::bwd_dx_f16_slot_bytes(M, N, K);
}

int64_t tm_tgemm_bwd_dw_slots(int64_t M, int64_t N, int64_t K) {
  if (!sizes_ok(M, N, K)) return -1;
  return tmk::bwd_dw_slot_bytes(M, N, K);
}

int64_t tm_tgemm_fwd_slots(int64_t M, int64_t N, int64_t K, int32_t g) {
  const int64_t f32 = tm_tgemm_fwd_scratch(M, N, K, g, 0);
  const int64_t b16 = tm_tgemm_fwd_scratch(M, N, K, g, 1);
  return f32 > b16 ? f32 : b16;
}

int64_t tm_tgemm_fwd_scratch(int64_t M, int64_t N, int64_t K, int32_t g, int32_t y_bf16) {
  if (!sizes_ok(M, N, K) || shape_kg(K, g) != TM_OK || (y_bf16 & ~1)) return -1;
  return tmk::fwd_scratch_bytes(M, N, K, g, y_bf16 != 0);
}

tm_status tm_tgemm_fwd_parts(const uint16_t* X, const uint8_t* codes, const float* scales,
                             int64_t M, int64_t N, int64_t K, int32_t g, void* Y, int32_t y_bf16,
                             void* workspace, int64_t workspace_bytes, float* slots,
                             int64_t slots_bytes, tm_stream stream) {
  if ((y_bf16 & ~1) || (y_bf16 && workspace)) return TM_EINVAL;
  const int es = y_bf16 ? 2 : 4;
  if (tm_status st = fwd_checked(X, codes, scales, M, N, K, g, Y, es, workspace, workspace_bytes))
    return st;
  const int64_t need = tm_tgemm_fwd_scratch(M, N, K, g, y_bf16);
  const Span ops[5] = {span(X, M * K * 2), span(codes, N * (K / 4)), span(scales, N * (K / g) * 4),
                       span(Y, M * N * es), span(workspace, workspace ? kFwdTicketBytes : 0)};
  if (tm_status st = slots_checked(slots, slots_bytes, need, ops, 5)) return st;
  return hip_status(tmk::launch_tgemm_fwd_parts(X, codes, scales, M, N, K, g, Y, y_bf16 != 0,
                                                static_cast<uint32_t*>(workspace), slots,
                                                slots != nullptr || need == 0, to_hip(stream)));
}

tm_status tm_tgemm_bwd_dx_parts(const void* dY, int32_t dy_f32, uint16_t* dY_bf16,
                                const uint8_t* codes, const float* scales, int64_t M, int64_t N,
                                int64_t K, int32_t g, int32_t exact, void* dX, int32_t dx_bf16,
                                void* workspace, int64_t workspace_bytes, float* slots,
                                int64_t slots_bytes, tm_stream stream) {
  if ((dy_f32 & ~1) || (dx_bf16 & ~1) || (exact & ~1)) return TM_EINVAL;
  if ((exact != 0) != (workspace == nullptr)) return TM_EINVAL;
  if ((dy_f32 != 0) != (dY_bf16 != nullptr) || (dy_f32 && exact)) return TM_EINVAL;
  const int ye = dy_f32 ? 4 : 2, xe = dx_bf16 ? 2 : 4;
  if (tm_status st = bwd_dx_checked(dY, codes, scales, M, N, K, g, dX, workspace,
                                    workspace_bytes, ye, xe))
    return st;
  const Span ops[6] = {span(dY, M * N * ye),
                       span(codes, N * (K / 4)),
                       span(scales, N * (K / g) * 4),
                       span(dX, M * K * xe),
                       span(workspace, workspace ? tmk::dx_f16_workspace_bytes(M, N) : 0),
                       span(dY_bf16, dY_bf16 ? M * N * 2 : 0)};
  if (dY_bf16) {
    if (!aligned(dY_bf16, 16)) return TM_EALIGN;
    for (int i = 0; i < 5; ++i)
      if (overlap(ops[5], ops[i])) return TM_EINVAL;
  }
  const int64_t need = tm_tgemm_bwd_dx_slots(M, N, K, exact);
  if (dx_bf16 && need > 0 && !slots) return TM_EINVAL;
  if (tm_status st = slots_checked(slots, slots_bytes, need, ops, 6)) return st;
  if (exact)
    return hip_status(tmk::launch_tgemm_bwd_dx_parts(static_cast<const uint16_t*>(dY), codes,
                                                     scales, M, N, K, g, dX, dx_bf16 != 0, slots,
                                                     to_hip(stream)));
  return hip_status(tmk::launch_tgemm_bwd_dx_f16_parts(dY, dy_f32 != 0, dY_bf16, codes, scales, M,
                                                       N, K, g, dX, dx_bf16 != 0, workspace,
                                                       slots, to_hip(stream)));
}

tm_status tm_tgemm_bwd_dw_parts(const uint16_t* dY, const uint16_t* X, int64_t M, int64_t N,
                                int64_t K, float* dW, int32_t accumulate, float* slots,
                                int64_t slots_bytes, tm_stream stream) {
  if (tm_status st = bwd_dw_checked(dY, X, M, N, K, dW, accumulate)) return st;
  const Span ops[3] = {span(dY, M * N * 2), span(X, M * K * 2), span(dW, N * K * 4)};
  if (tm_status st = slots_checked(slots, slots_bytes, tm_tgemm_bwd_dw_slots(M, N, K), ops, 3))
    return st;
  return hip_status(tmk::launch_tgemm_bwd_dw_parts(dY, X, M, N, K, dW, accumulate, slots,
                                                   to_hip(stream)));
}

}  // extern "C"
