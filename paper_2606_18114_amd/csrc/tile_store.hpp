// Output of a 128 x 128 wave tile held as 4 x 4 blocks of 32x32 MFMA
// accumulators: lane holds column l32 of each block, rows 8 (i/4) + 4 h + i%4.
//
// What bounds a small call here is the instruction fetch: every workgroup runs
// this straight-line code once, cold, so each way of writing (store, add,
// atomic; whole or ragged tile) has a loop of its own and a launch fetches
// only one, a few KiB.  The pointer steps row by row through an opaque pitch:
// precomputed offsets would be held in registers, which the accumulators need.
#pragma once

#include "common.hpp"

namespace tmk {

// One accumulator as a value of its own: without the opaque copy the compiler
// wants whole accumulator blocks in the vector registers the stores read
// from, and spills them there.
__device__ __forceinline__ float acc_value(float v) {
  asm volatile("" : "+v"(v));
  return v;
}

// op(ptr, value(a, b, i)) for every element inside the tile: base, the
// address of the wave tile's first element; pitch in elements; rows_left and
// cols_left, rows and columns of the output from there on.
template <bool FULL, typename T, typename Prep, typename Val, typename Op>
__device__ __forceinline__ void tile_store_as(T* base, int64_t pitch, int rows_left,
                                              int cols_left, Prep prep, Val val, Op op) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  int64_t pv = pitch;
  asm volatile("" : "+v"(pv));
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    if (!FULL && 32 * a >= rows_left) break;
    prep(a);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (FULL || 32 * b + l32 < cols_left) {
        T* p = base + (int64_t)(32 * a) * pitch + 32 * b + (4 * h * pv + l32);
        const int left = rows_left - 32 * a - 4 * h;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          if (FULL || 8 * (i / 4) + i % 4 < left) op(p, val(a, b, i));
          if (i < 15) p += i % 4 == 3 ? 5 * pv : pv;
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // one block's values live at a time
    }
  }
}

template <typename T, typename Prep, typename Val, typename Op>
__device__ __forceinline__ void tile_store(T* base, int64_t pitch, int rows_left, int cols_left,
                                           Prep prep, Val val, Op op) {
  if (rows_left >= 128 && cols_left >= 128)
    tile_store_as<true>(base, pitch, rows_left, cols_left, prep, val, op);
  else
    tile_store_as<false>(base, pitch, rows_left, cols_left, prep, val, op);
}

// The wave tile added to the output (rows_left a multiple of 8, as dW's rows
// are, so that whether a run of 8 rows is inside is the same for all lanes).  A
// block's 16 values are read before the first sum is written: a sum in place at
// a time waited for each read by itself (29 tokens x 9864 x 2560: 163 us, 46
// now; 16384 x 8512 x 2048: 550 and 496).
template <bool FULL, typename Val>
__device__ __forceinline__ void tile_add_as(float* base, int64_t pitch, int rows_left,
                                            int cols_left, Val val) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  int64_t pv = pitch;
  asm volatile("" : "+v"(pv));
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    if (!FULL && 32 * a >= rows_left) break;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (FULL || 32 * b + l32 < cols_left) {
        float* const p0 = base + (int64_t)(32 * a) * pitch + 32 * b + (4 * h * pv + l32);
        float old[16];
        float* p = p0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!FULL && 32 * a + 8 * r >= rows_left) break;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            old[4 * r + i] = *p;
            if (4 * r + i < 15) p += i == 3 ? 5 * pv : pv;
          }
        }
        p = p0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!FULL && 32 * a + 8 * r >= rows_left) break;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            *p = old[4 * r + i] + val(a, b, 4 * r + i);
            if (4 * r + i < 15) p += i == 3 ? 5 * pv : pv;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <typename Val>
__device__ __forceinline__ void tile_add(float* base, int64_t pitch, int rows_left, int cols_left,
                                         Val val) {
  if (rows_left >= 128 && cols_left >= 128)
    tile_add_as<true>(base, pitch, rows_left, cols_left, val);
  else
    tile_add_as<false>(base, pitch, rows_left, cols_left, val);
}

// The wave tile into the workgroup's slot of the parts buffer, in register
// order (the layout reduce_parts reads); blocks wholly outside the output are
// skipped.
template <typename Prep, typename Val>
__device__ __forceinline__ void slot_store(float* slot, int rows_left, int cols_left, Prep prep,
                                           Val val) {
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    if (32 * a >= rows_left) break;
    prep(a);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (32 * b >= cols_left) break;
      // a 32-bit lane offset from a uniform base, opaque per block so that
      // the compiler does not hold all 64 addresses at once
      uint32_t o = 16u * (uint32_t)threadIdx.x;
      asm volatile("" : "+v"(o));
      o += (uint32_t)(a * 4 + b) * 16384u;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4*>(reinterpret_cast<uint8_t*>(slot) + o + 4096 * i) =
            f32x4{val(a, b, 4 * i), val(a, b, 4 * i + 1), val(a, b, 4 * i + 2),
                  val(a, b, 4 * i + 3)};
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

}  // namespace tmk
