// How the persistent GEMM kernels share out their 256 x 256 output tiles, and
// how the parts of a tile that is cut along the contraction meet.
//
// Whole rounds of tiles (one per workgroup and round) come first.  The `rem`
// tiles left over, fewer than there are workgroups, are cut into `parts`
// contraction ranges of `per` stages each; part p of leftover tile j is run
// by workgroup p * rem + j, so the workgroups of one XCD share the operand
// rows of one range.  Each part writes its float32 sums to a slot of a
// caller-owned buffer, in the register layout of the kernel (16-byte pieces,
// thread-major, fully coalesced), and reduce_parts adds a tile's slots in
// part order (the same bits on every run) into the output.  Without a buffer
// the parts add into the cleared output with float32 atomics.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

namespace tmk {

struct TilePlan {
  int64_t full = 0, rem = 0;  // whole rounds; leftover tiles
  int parts = 1, per = 0;     // ranges per leftover tile, stages per range
  int64_t grid = 0;           // workgroups
  int64_t slots() const { return parts > 1 ? rem * parts : 0; }
};

constexpr int64_t kSlotFloats = 256 * 256;
constexpr int64_t kSlotBytes = kSlotFloats * 4;

// The plan of ntiles tiles of nst contraction stages on P workgroups, ranges
// a multiple of `unit` stages.  The number of parts balances the leftover
// tiles' compute time (unit_us per `unit` stages) against the slots' traffic
// (written once, read once: slot_us per slot over the whole chip) and the
// second launch (launch_us).
inline TilePlan plan_parts(int64_t ntiles, int64_t nst, int unit, int64_t P, double unit_us,
                           double slot_us, double launch_us) {
  TilePlan t;
  t.full = ntiles / P;
  t.rem = ntiles % P;
  const int64_t units = (nst + unit - 1) / unit;
  t.per = (int)(units * unit);
  if (t.rem > 0) {
    double best = (double)units * unit_us;
    const int64_t most = P / t.rem < units ? P / t.rem : units;
    for (int64_t k = 2; k <= most; ++k) {
      const int64_t pu = (units + k - 1) / k;
      const int64_t used = (units + pu - 1) / pu;  // no empty ranges
      if (used != k) continue;
      const double c = (double)pu * unit_us + (double)(k * t.rem) * slot_us + launch_us;
      if (c < best) {
        best = c;
        t.parts = (int)k;
        t.per = (int)(pu * unit);
      }
    }
  }
  t.grid = t.full > 0 ? P : t.rem * t.parts;
  return t;
}

// The plan without a buffer: at most P workgroups, the tiles beyond whole
// rounds cut into as many parts as there are workgroups for
inline TilePlan plan_atomic(int64_t ntiles, int64_t nst, int64_t cus) {
  TilePlan t;
  const int64_t P = ntiles < cus ? ntiles : cus;
  t.full = ntiles / P;
  t.rem = ntiles % P;
  int64_t k = t.rem ? P / t.rem : 1;
  if (k > nst) k = nst;
  t.per = (int)((nst + k - 1) / k);
  t.parts = (int)((nst + t.per - 1) / t.per);
  t.grid = P;
  return t;
}

// out[rows, cols] of the leftover tiles (tile0 + j, tiles_c tiles per row of
// tiles) from their slots: float32 (added to out when accumulate), or
// bfloat16 rounded once
hipError_t launch_reduce_parts(const float* slots, int64_t rem, int parts, int64_t tile0,
                               int64_t tiles_c, int64_t rows, int64_t cols, void* out,
                               bool bf16_out, bool accumulate, hipStream_t stream);
// the same for the forward kernel's bm x bn tiles (its wave layouts)
hipError_t launch_reduce_fwd_parts(const float* slots, int64_t rem, int parts, int64_t tile0,
                                   int64_t tiles_c, int64_t rows, int64_t cols, void* out,
                                   bool bf16_out, int bm, int bn, hipStream_t stream);

}  // namespace tmk
