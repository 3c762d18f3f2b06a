// Sums the slots of the output tiles that were cut along the contraction
// (tile_parts.hpp) into the output.
//
// HBM / cache bound: every slot is read once in 16-byte pieces, 256 threads
// on 4 KiB in a row (512 on 8), and each output element is written once.  A
// workgroup takes the piece (a, b, i4) of one tile: rows 32 a + 8 i4 .. + 7
// and columns 32 b .. + 31 of every wave's outputs, so a 256 x 256 tile
// spreads over 64 (or 32) workgroups.
#include "common.hpp"
#include "tile_parts.hpp"

namespace tmk {

// Kernel layout: WM x WN waves of 32 MA x 32 NB outputs.
template <bool BF, int MA, int NB, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) void reduce_parts_kernel(
    const float* __restrict__ slots, uint32_t rem, int parts, uint32_t tile0, uint32_t tiles_c,
    int64_t rows, int64_t cols, void* __restrict__ out, int accumulate) {
  constexpr int kBM = 32 * MA * WM, kBN = 32 * NB * WN, kThreads = 64 * WM * WN;
  constexpr uint32_t kPieces = MA * NB * 4;
  const uint32_t j = blockIdx.x / kPieces, piece = blockIdx.x % kPieces;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int a = (int)(piece / (4 * NB)), b = (int)((piece / 4) % NB), i4 = (int)(piece % 4);
  const uint32_t tile = tile0 + j;
  const int64_t r = (int64_t)(tile / tiles_c) * kBM + (wave / WN) * (32 * MA) + 32 * a + 8 * i4 +
                    4 * (lane >> 5);
  const int64_t c = (int64_t)(tile % tiles_c) * kBN + (wave % WN) * (32 * NB) + 32 * b +
                    (lane & 31);
  if (r >= rows || c >= cols) return;
  const f32x4* s = reinterpret_cast<const f32x4*>(slots + (int64_t)j * (kBM * kBN)) +
                   piece * (uint32_t)kThreads + tid;
  // part p of tile j: slot p * rem + j
  const int64_t pitch = (int64_t)rem * (kBM * kBN / 4);
  f32x4 v = s[0];
  int p = 1;
  for (; p + 4 <= parts; p += 4) {  // four loads in flight, added in part order
    f32x4 q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = s[(p + i) * pitch];
#pragma unroll
    for (int i = 0; i < 4; ++i) v += q[i];
  }
  for (; p < parts; ++p) v += s[p * pitch];
  const int n = rows - r < 4 ? (int)(rows - r) : 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i < n) {
      const int64_t o = (r + i) * cols + c;
      if constexpr (BF) {
        reinterpret_cast<uint16_t*>(out)[o] = __builtin_bit_cast(uint16_t, (__bf16)v[i]);
      } else {
        float* d = reinterpret_cast<float*>(out) + o;
        *d = accumulate ? *d + v[i] : v[i];
      }
    }
  }
}

#define TM_REDUCE(MA, NB, WM, WN)                                                               \
  do {                                                                                          \
    const dim3 grid((unsigned)(rem * (MA) * (NB) * 4)), block(64 * (WM) * (WN));                 \
    if (bf16_out)                                                                               \
      hipLaunchKernelGGL((reduce_parts_kernel<true, MA, NB, WM, WN>), grid, block, 0, stream,   \
                         slots, (uint32_t)rem, parts, (uint32_t)tile0, (uint32_t)tiles_c, rows, \
                         cols, out, 0);                                                         \
    else                                                                                        \
      hipLaunchKernelGGL((reduce_parts_kernel<false, MA, NB, WM, WN>), grid, block, 0, stream,  \
                         slots, (uint32_t)rem, parts, (uint32_t)tile0, (uint32_t)tiles_c, rows, \
                         cols, out, accumulate ? 1 : 0);                                        \
  } while (0)

hipError_t launch_reduce_parts(const float* slots, int64_t rem, int parts, int64_t tile0,
                               int64_t tiles_c, int64_t rows, int64_t cols, void* out,
                               bool bf16_out, bool accumulate, hipStream_t stream) {
  TM_REDUCE(4, 4, 2, 2);
  return hipGetLastError();
}

hipError_t launch_reduce_fwd_parts(const float* slots, int64_t rem, int parts, int64_t tile0,
                                   int64_t tiles_c, int64_t rows, int64_t cols, void* out,
                                   bool bf16_out, int bm, int bn, hipStream_t stream) {
  const bool accumulate = false;
  if (bm == 256 && bn == 256)
    TM_REDUCE(4, 2, 2, 4);
  else if (bm == 128 && bn == 128)
    TM_REDUCE(2, 2, 2, 2);
  else if (bm == 64 && bn == 128)
    TM_REDUCE(1, 2, 2, 2);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}
#undef TM_REDUCE

}  // namespace tmk
