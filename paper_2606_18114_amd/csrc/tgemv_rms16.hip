// Fused decode projection for batches of 5 to 16 rows (the batched counterpart
// of tm_tgemv_rms): x = bf16(src r w), r = 1 / sqrt(mean(src^2) + eps) per
// batch row, y = (or +=) x times one ternary matrix, on the bfloat16 matrix
// cores, with the normalization's passes taken out of the step:
//   * the rows' sums of squares arrive as partial sums that the kernel before
//     wrote on its way (the heads' sums of the mixer, or this kernel's own
//     part_out: one partial per 16 output rows of the residual it updates), so
//     no launch reads a row only to normalize it; or, without partial sums,
//     every workgroup takes them from the rows it reads anyway, one wave per
//     row;
//   * every workgroup builds the bfloat16 x of all rows in LDS (coalesced
//     loads of src, from L2 after the first workgroup of an XCD);
//   * the convolution ring's position moves on here, after every reader.
// A layer is three launches instead of five, and none of them is a norm of 16
// workgroups.
//
// The step is bound by the length of each launch's chain of waits, not by its
// bytes (6.5 MB of codes a layer): the codes are loaded before x, the batch
// rows are the 16 A rows of v_mfma_f32_16x16x32_bf16 as in tgemv_b16.hip, and
// the columns are split over 16 waves per workgroup, whose sums meet in LDS.
// (With the MFMA operand normalized straight from global memory, 16 rows at a
// time in 16-byte pieces, the address unit was the bound: 22 us for 8512 x
// 2048 and 28 us for 2048 x 4096 at batch 16, against 12.0 and 11.6; the norm
// and GEMV launches before took 19.9 and 18.2.)
//
// Order of the sums.  A rounding that falls the other way in one activation
// changes every value after it, so a token of 9 to 16 rows adds in the order
// of the unfused launches and has their bits: the groups of an output in four
// contiguous chains (tgemv_b16.hip), the squares of a row without partial sums
// as residual_rmsnorm takes them (256 chains of every 256th column, then a
// binary tree).  Below 9 rows the unfused projection is another kernel
// (tgemv.hip) whose sums this one cannot have; there the chains are 16, one
// per wave's columns, which need no products in LDS (batch 16 with them: 11.7
// and 10.8 us).
#include "common.hpp"
#include "launchers.hpp"
#include "mixer_dev.hpp"

namespace tmk {

constexpr int kR16Chunks = 4;  // most 64-column chunks of a wave (K <= 4096, 16 waves)
constexpr int kR16Quads = 8;   // 4-value pieces of src and w a thread has in flight
constexpr int kR16Waves = 16;

typedef __attribute__((ext_vector_type(2))) __bf16 r16_bf16x2;

// NB: 16-row blocks of the matrix per workgroup; KMAX: most columns (x takes
// 32 KMAX bytes of LDS).  part NULL: the rows' squares are summed here.
// quarters: an output's sum in four chains of groups, else one per wave
template <int G, int NB, int KMAX, bool ACC>
__global__ __launch_bounds__(64 * kR16Waves) void tgemv_rms16_kernel(
    const float* __restrict__ src, const float* __restrict__ part, int nparts,
    const float* __restrict__ nw, float eps, const uint8_t* __restrict__ codes,
    const uint16_t* __restrict__ s16, int B, int N, int K, int quarters, float* y,
    float* __restrict__ part_out, int* __restrict__ advance) {
  static_assert(G % 64 == 0 && kR16Chunks % (G / 64) == 0, "whole groups per wave");
  static_assert(64 * kR16Waves >= NB * 256, "a thread per output");
  static_assert(KMAX <= 64 * kR16Chunks * kR16Waves, "the waves' chunks cover a row");
  constexpr int WAVES = kR16Waves;
  constexpr int kWpg = G / 64;                // chunks per group
  constexpr int kGrp = kR16Chunks / kWpg;     // most groups of a wave
  constexpr int kT = 64 * WAVES, kPr = kT / 16;  // threads; threads per batch row (sums)
  constexpr int kRows = KMAX / 256;  // rows (or pieces of a row) that a thread normalizes
  // x: the 16-byte piece u of row n sits at u ^ (n % 8), so that the operand
  // reads of 16 rows spread over the banks; what the sums need of LDS reuses
  // its space (kRb blocks at a time)
  constexpr int kGroups = KMAX / G, kX = 32 * KMAX;
  constexpr int kBlk = kGroups * 1024 + 16 * 4 * (kGroups + 4) + 4096;
  constexpr int kRb = NB * kBlk <= 159 * 1024 ? NB : 2, kRed = kRb * kBlk;
  constexpr int kSums = WAVES * NB * 1024, kAll = kSums > kRed ? kSums : kRed;
  static_assert(kAll <= 159 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(16))) uint8_t lds[kX > kAll ? kX : kAll];
  __shared__ float rs[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, kq = lane >> 4;
  const int j0 = NB * blockIdx.x;
  const int ngr = K / G, gpw = (ngr + WAVES - 1) / WAVES, g0 = wave * gpw;
  const int gw = ngr - g0 < gpw ? (ngr - g0 > 0 ? ngr - g0 : 0) : gpw;  // groups of this wave
  const int nch = gw * kWpg;
  // the output this thread writes: batch row om (in the order of the
  // accumulators' lanes) of row orow
  const int om = 4 * kq + (wave & 3), orow = 16 * (j0 + (tid >> 8)) + n;
  const bool owner = tid < NB * 256 && om < B && orow < N;
  float base = 0.f;
  if (ACC && owner) base = y[(int64_t)om * N + orow];

  uint32_t cw[kR16Chunks][NB];
  uint16_t sc[NB][kGrp];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int row = 16 * (j0 + b) + n;
    const bool rok = row < N;
    const uint32_t* crow =
        reinterpret_cast<const uint32_t*>(codes + (int64_t)(rok ? row : 0) * (K / 4));
    const uint16_t* srow = s16 + (int64_t)(rok ? row : 0) * (K / G);
#pragma unroll
    for (int t = 0; t < kR16Chunks; ++t)
      cw[t][b] = rok && t < nch ? crow[g0 * (G / 16) + 4 * t + kq] : 0u;
#pragma unroll
    for (int r = 0; r < kGrp; ++r) sc[b][r] = rok && r < gw ? srow[g0 + r] : (uint16_t)0;
  }

  // x, rounded to bfloat16 (to nearest even); rows past B are left as they
  // are: an A row only reaches its own output row, which is not written
  const int qpr = K / 4;  // 4-value pieces per row
  auto put = [&](int row, int q, float r, const u32x4& v, const u32x4& w) {
    uint32_t o[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const r16_bf16x2 p = {
          (__bf16)(__uint_as_float(v[2 * e]) * r * __uint_as_float(w[2 * e])),
          (__bf16)(__uint_as_float(v[2 * e + 1]) * r * __uint_as_float(w[2 * e + 1]))};
      o[e] = __builtin_bit_cast(uint32_t, p);
    }
    const uint32_t u = ((uint32_t)q >> 1) ^ ((uint32_t)row & 7u);
    *reinterpret_cast<u32x2*>(lds + (uint32_t)row * (2u * K) + 16u * u + 8u * (q & 1)) =
        u32x2{o[0], o[1]};
  };
  // 1 / rms of a row from the 64 lanes' sums
  auto row_scale = [&](float s) {
    s += __uint_as_float(lane_xchg<1>(__float_as_uint(s)));
    s += __uint_as_float(lane_xchg<2>(__float_as_uint(s)));
    s += __uint_as_float(lane_xchg<4>(__float_as_uint(s)));
    s += __uint_as_float(lane_xchg<8>(__float_as_uint(s)));
    s += __uint_as_float(lane_xchg<16>(__float_as_uint(s)));
    s += __uint_as_float(lane_xchg<32>(__float_as_uint(s)));
    return 1.f / sqrtf(s / (float)K + eps);
  };
  // the rows' 1 / rms (while loads of src are in flight)
  auto row_scales = [&]() {
    const int row = tid / kPr, l = tid % kPr;
    float s = 0.f;
    if (row < B)
      for (int i = l; i < nparts; i += kPr) s += part[(int64_t)row * nparts + i];
    const float r = row_scale(s);
    if (l == 0) rs[row] = r;
    __syncthreads();
  };
  if (advance && blockIdx.x == 0 && tid == 0) *advance = (*advance + 1) & 3;
  if (part == nullptr) {
    // wave r takes row r, lane l its pieces l, l + 64, ...: four chains of
    // every 256th column, then the tree
    if (wave < B) {
      const float* row = src + (int64_t)wave * K;
      constexpr bool kEarly = kRows <= 8;  // registers for the norm weights as well
      u32x4 v[kRows], w[kEarly ? kRows : 1];
#pragma unroll
      for (int j = 0; j < kRows; ++j)
        if (lane + 64 * j < qpr) {
          v[j] = ld16(row + 4 * (lane + 64 * j));
          if constexpr (kEarly) w[j] = ld16(nw + 4 * (lane + 64 * j));
        }
      float sq[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < kRows; ++j)
        if (lane + 64 * j < qpr) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float f = __uint_as_float(v[j][e]);
            sq[e] = __builtin_fmaf(f, f, sq[e]);
          }
        }
      const float r = row_scale((sq[0] + sq[1]) + (sq[2] + sq[3]));
#pragma unroll
      for (int j = 0; j < kRows; ++j)
        if (lane + 64 * j < qpr) {
          if constexpr (kEarly)
            put(wave, lane + 64 * j, r, v[j], w[j]);
          else
            put(wave, lane + 64 * j, r, v[j], ld16(nw + 4 * (lane + 64 * j)));
        }
    }
  } else if (kT % qpr == 0) {
    // a thread's pieces all lie in the same columns, one load of the norm
    // weights; at most kRows rows, all in flight at once
    const int step = kT / qpr, row0 = tid / qpr, q = tid % qpr;
    const u32x4 w = ld16(nw + 4 * q);
    u32x4 v[kRows];
#pragma unroll
    for (int j = 0; j < kRows; ++j)
      if (row0 + j * step < B) v[j] = ld16(src + (int64_t)(row0 + j * step) * K + 4 * q);
    row_scales();
#pragma unroll
    for (int j = 0; j < kRows; ++j)
      if (row0 + j * step < B) put(row0 + j * step, q, rs[row0 + j * step], v[j], w);
  } else {
    // pieces tid, tid + kT, ... in row order, kR16Quads at a time
    const int total = B * qpr, drow = kT / qpr, dcol = kT % qpr;
    int qi = tid, row = tid / qpr, q = tid % qpr;
    u32x4 v[kR16Quads], w[kR16Quads];
    int at[kR16Quads];  // row << 16 | piece, or -1
    auto fetch = [&]() {
#pragma unroll
      for (int j = 0; j < kR16Quads; ++j) {
        at[j] = -1;
        if (qi < total) {
          v[j] = ld16(src + (int64_t)row * K + 4 * q);
          w[j] = ld16(nw + 4 * q);
          at[j] = (row << 16) | q;
        }
        qi += kT;
        row += drow;
        q += dcol;
        if (q >= qpr) {
          q -= qpr;
          ++row;
        }
      }
    };
    fetch();
    row_scales();
    for (int done = 0; done < total; done += kT * kR16Quads) {
      if (done > 0) fetch();
#pragma unroll
      for (int j = 0; j < kR16Quads; ++j)
        if (at[j] >= 0) put(at[j] >> 16, at[j] & 0xFFFF, rs[at[j] >> 16], v[j], w[j]);
    }
  }
  __syncthreads();
  // operand of 8 columns from col
  auto xop = [&](int col) {
    return as_bf16x8(*reinterpret_cast<const u32x4*>(
        lds + (uint32_t)n * (2u * K) + 16u * ((uint32_t)(col / 8) ^ (uint32_t)(n & 7))));
  };
  f32x4 acc[NB][kGrp];  // each group's products
#pragma unroll
  for (int t = 0; t < kR16Chunks; ++t) {
    if (t < nch) {  // uniform
      const int col = g0 * G + 64 * t + 16 * kq;
      const bf16x8 a0 = xop(col), a1 = xop(col + 8);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        f32x4& a = acc[b][t / kWpg];
        if (t % kWpg == 0) a = f32x4{0.f, 0.f, 0.f, 0.f};
        a = mfma16(a0, decode_half<0>(cw[t][b]), a);
        a = mfma16(a1, decode_half<1>(cw[t][b]), a);
      }
    }
  }
  // lane (kq, n) holds batch rows 4 kq + e of weight row n of each block.  In
  // LDS: the chains' sums (chain, block, e, lane)
  float* sums = reinterpret_cast<float*>(lds);
  float v = 0.f;
  if (!quarters) {
    // a chain is what a wave holds
    __syncthreads();  // x has been read
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float run = 0.f;
#pragma unroll
        for (int r = 0; r < kGrp; ++r)
          if (r < gw) run = __builtin_fmaf(acc[b][r][e], h2f(sc[b][r]), run);
        sums[((wave * NB + b) * 4 + e) * 64 + lane] = run;
      }
    __syncthreads();
    if (tid < NB * 256) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) sum += sums[w * (NB * 256) + (tid >> 6) * 64 + lane];
      v = 0.5f * sum;  // the codes decode to 2q
    }
  } else {
    // a chain is a quarter of the row's groups, from several waves: the groups'
    // products (group, block, e, lane) and scales (block, n, group) go to LDS,
    // and wave w takes the chains w, w + 16, ... (4 (4 b + e) + quarter)
    constexpr int kLd = kGroups + 4;
    float* red = sums + 4 * kRb * 256;
    float* scl = red + kGroups * kRb * 256;
    const int len = (ngr + 3) / 4;
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += kRb) {
      __syncthreads();  // x, or the blocks before, have been read
#pragma unroll
      for (int b = b0; b < b0 + kRb && b < NB; ++b)
#pragma unroll
        for (int r = 0; r < kGrp; ++r)
          if (r < gw) {
            const int at = (g0 + r) * kRb + (b - b0);
#pragma unroll
            for (int e = 0; e < 4; ++e) red[(at * 4 + e) * 64 + lane] = acc[b][r][e];
            if (kq == 0) scl[((b - b0) * 16 + n) * kLd + g0 + r] = h2f(sc[b][r]);
          }
      __syncthreads();
      float run[kRb];
#pragma unroll
      for (int i = 0; i < kRb; ++i) run[i] = 0.f;
#pragma unroll 4
      for (int g = 0; g < len; ++g) {
#pragma unroll
        for (int i = 0; i < kRb; ++i) {
          const int c = wave + 16 * i, be = c >> 2, at = (c & 3) * len + g;
          const bool in = at < ngr && b0 + (be >> 2) < NB;
          const float f = red[((in ? at : 0) * (kRb * 4) + be) * 64 + lane];
          const float c1 = scl[((be >> 2) * 16 + n) * kLd + (in ? at : 0)];
          run[i] = in ? __builtin_fmaf(f, c1, run[i]) : run[i];
        }
      }
#pragma unroll
      for (int i = 0; i < kRb; ++i) {
        const int c = wave + 16 * i;
        sums[((c & 3) * (kRb * 4) + (c >> 2)) * 64 + lane] = run[i];
      }
      __syncthreads();
      const int be = (tid >> 6) - 4 * b0;  // (block, e) of this thread's output
      if (be >= 0 && be < 4 * kRb) {
        float sum = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) sum += sums[(c * (kRb * 4) + be) * 64 + lane];
        v = 0.5f * sum;
      }
    }
  }
  if (tid < NB * 256) {
    if constexpr (ACC) v = __fadd_rn(base, v);
    if (owner) y[(int64_t)om * N + orow] = v;
    if (part_out) {
      // the block's 16 rows of this batch row
      float sq = owner ? v * v : 0.f;
      sq += __uint_as_float(lane_xchg<1>(__float_as_uint(sq)));
      sq += __uint_as_float(lane_xchg<2>(__float_as_uint(sq)));
      sq += __uint_as_float(lane_xchg<4>(__float_as_uint(sq)));
      sq += __uint_as_float(lane_xchg<8>(__float_as_uint(sq)));
      const int blk = j0 + (tid >> 8), nblk = (N + 15) / 16;
      if (n == 0 && om < B && blk < nblk) part_out[(int64_t)om * nblk + blk] = sq;
    }
  }
}

// dst[b] = src[b] (dst may be NULL) and part[b] = the row's sum of squares
__global__ __launch_bounds__(256) void rows_sumsq_kernel(const float* src, int64_t D, float* dst,
                                                         float* __restrict__ part) {
  __shared__ float wsum[4];
  const int64_t o = (int64_t)blockIdx.x * D;
  float sq = 0.f;
  for (int64_t i = threadIdx.x; i < D; i += 256) {
    const float v = src[o + i];
    if (dst) dst[o + i] = v;
    sq = __builtin_fmaf(v, v, sq);
  }
  sq += __uint_as_float(lane_xchg<1>(__float_as_uint(sq)));
  sq += __uint_as_float(lane_xchg<2>(__float_as_uint(sq)));
  sq += __uint_as_float(lane_xchg<4>(__float_as_uint(sq)));
  sq += __uint_as_float(lane_xchg<8>(__float_as_uint(sq)));
  sq += __uint_as_float(lane_xchg<16>(__float_as_uint(sq)));
  sq += __uint_as_float(lane_xchg<32>(__float_as_uint(sq)));
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = sq;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

hipError_t launch_rows_sumsq(const float* src, int B, int64_t D, float* dst, float* part,
                             hipStream_t stream) {
  hipLaunchKernelGGL(rows_sumsq_kernel, dim3((unsigned)B), dim3(256), 0, stream, src, D, dst,
                     part);
  return hipGetLastError();
}

// As many blocks per workgroup, up to four, as leave at most one workgroup per
// CU: every workgroup builds all of x, so a CU with two would do it twice.
template <int G, int KMAX, bool ACC>
static hipError_t launch_r16(const float* src, const float* part, int nparts, const float* nw,
                             float eps, const uint8_t* codes, const uint16_t* s16, int B, int N,
                             int K, float* y, float* part_out, int* advance,
                             hipStream_t stream) {
  const int nblk = (N + 15) / 16, cus = current_cu_count();
  const int quarters = tgemv_b16_takes(B, G) ? 1 : 0;
#define TM_R16(NB_)                                                                          \
  hipLaunchKernelGGL((tgemv_rms16_kernel<G, NB_, KMAX, ACC>), dim3((nblk + NB_ - 1) / NB_),  \
                     dim3(64 * kR16Waves), 0, stream, src, part, nparts, nw, eps, codes, s16, \
                     B, N, K, quarters, y, part_out, advance)
  if (nblk <= cus)
    TM_R16(1);
  else if (nblk <= 2 * cus)
    TM_R16(2);
  else if (nblk <= 3 * cus)
    TM_R16(3);
  else
    TM_R16(4);
#undef TM_R16
  return hipGetLastError();
}

template <int G>
static hipError_t launch_r16_k(const float* src, const float* part, int nparts, const float* nw,
                               float eps, const uint8_t* codes, const uint16_t* s16, int B,
                               int N, int K, float* y, int accum, float* part_out, int* advance,
                               hipStream_t stream) {
  auto go = [&](auto f) {
    return f(src, part, nparts, nw, eps, codes, s16, B, N, K, y, part_out, advance, stream);
  };
  if (K <= 2048) return accum ? go(launch_r16<G, 2048, true>) : go(launch_r16<G, 2048, false>);
  return accum ? go(launch_r16<G, 4096, true>) : go(launch_r16<G, 4096, false>);
}

hipError_t launch_tgemv_rms16(const float* src, const float* part, int nparts, const float* nw,
                              float eps, const uint8_t* codes, const uint16_t* s16, int B,
                              int64_t N, int64_t K, int g, float* y, int accum, float* part_out,
                              int* advance, hipStream_t stream) {
  if (B < 1 || B > 16 || N > 0x7FFFFFF0 || K > kRms16MaxK || K % 64 != 0 || K % g != 0)
    return hipErrorInvalidValue;
#define TM_R16_CASE(GG)                                                                        \
  case GG:                                                                                     \
    return launch_r16_k<GG>(src, part, nparts, nw, eps, codes, s16, B, (int)N, (int)K, y, accum, \
                            part_out, advance, stream);
  switch (g) {
    TM_R16_CASE(64)
    TM_R16_CASE(128)
    TM_R16_CASE(256)
    default: return hipErrorInvalidValue;
  }
#undef TM_R16_CASE
}

}  // namespace tmk
