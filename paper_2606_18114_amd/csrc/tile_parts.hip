// Sums the slots of the output tiles that were cut along the contraction
// (tile_parts.hpp) into the output.
//
// HBM / cache bound: every slot is read once in 16-byte pieces, 256 threads
// on 4 KiB in a row, and each output element is written once.  A workgroup
// takes the piece (a, b, i4) of one tile: rows 32 a + 8 i4 .. + 7 and columns
// 32 b .. + 31 of each of the four 128 x 128 quarters, so a tile spreads over
// 64 workgroups and even one leftover tile occupies a quarter of the chip.
#include "common.hpp"
#include "tile_parts.hpp"

namespace tmk {

template <bool BF>
__global__ __launch_bounds__(256) void reduce_parts_kernel(
    const float* __restrict__ slots, uint32_t rem, int parts, uint32_t tile0, uint32_t tiles_c,
    int64_t rows, int64_t cols, void* __restrict__ out, int accumulate) {
  const uint32_t j = blockIdx.x >> 6, piece = blockIdx.x & 63u;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int a = (int)(piece >> 4), b = (int)((piece >> 2) & 3u), i4 = (int)(piece & 3u);
  const uint32_t tile = tile0 + j;
  const int64_t r = (int64_t)(tile / tiles_c) * 256 + (wave >> 1) * 128 + 32 * a + 8 * i4 +
                    4 * (lane >> 5);
  const int64_t c = (int64_t)(tile % tiles_c) * 256 + (wave & 1) * 128 + 32 * b + (lane & 31);
  if (r >= rows || c >= cols) return;
  const f32x4* s = reinterpret_cast<const f32x4*>(slots + (int64_t)j * kSlotFloats) +
                   piece * 256u + tid;
  const int64_t pitch = (int64_t)rem * (kSlotFloats / 4);  // part p of tile j: slot p * rem + j
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

hipError_t launch_reduce_parts(const float* slots, int64_t rem, int parts, int64_t tile0,
                               int64_t tiles_c, int64_t rows, int64_t cols, void* out,
                               bool bf16_out, bool accumulate, hipStream_t stream) {
  const dim3 grid((unsigned)(rem * 64)), block(256);
  if (bf16_out)
    hipLaunchKernelGGL(reduce_parts_kernel<true>, grid, block, 0, stream, slots, (uint32_t)rem,
                       parts, (uint32_t)tile0, (uint32_t)tiles_c, rows, cols, out, 0);
  else
    hipLaunchKernelGGL(reduce_parts_kernel<false>, grid, block, 0, stream, slots, (uint32_t)rem,
                       parts, (uint32_t)tile0, (uint32_t)tiles_c, rows, cols, out,
                       accumulate ? 1 : 0);
  return hipGetLastError();
}

}  // namespace tmk
