// Decode-time ternary GEMV for batches of 9 to 16 rows (paper Sec. 8: decode
// reads every weight once per step; with more tokens per step the products
// grow and the vector ALUs of the FP8-split form become the bound).
//
// The batch rows fill the 16 A rows of v_mfma_f32_16x16x32_bf16 as they are
// (bfloat16), and the codes of 16 weight rows are the B operand, decoded to
// bfloat16 2q by one shift and one AND per two codes, so the products are
// exact and the sums float32.
//
// What bounds it is the code stream, if x stays out of its way: with the A
// operand read from global memory in 16-byte pieces of 16 rows, the address
// units were the bound (48 layers of 8512 x 2048 and 2048 x 4096, batch 16:
// 345 us, three times the batch-8 form).  So a workgroup first copies x (all
// rows, a window of at most KMAX columns) into LDS, and its waves then run
// independently: each takes whole 16-row blocks, one to four of them, with
// the codes of the next 1024 columns in flight while it works on the last.
// Two workgroups of 8 waves share a CU at K <= 2048 (64 KiB of x each), one
// of 16 waves beyond.  A lane with column n (its weight row, also its A row)
// and k quarter kq takes WPL consecutive code words of its row, 16 WPL columns
// of the step's 64 WPL (at most one group): the k index of the MFMA is any
// permutation of the columns as long as both operands use the same one, so a
// row's codes are read in runs of 16 WPL bytes.  A row's group scales are
// loaded once, a quarter of them by each kq, and passed between lanes.
#include "common.hpp"
#include "launchers.hpp"
#include "mixer_dev.hpp"

namespace tmk {

constexpr int kB16Cols = 1024;  // columns of a row in flight together

// W: waves; KMAX: columns of x in LDS
template <int G, int W, int KMAX>
__global__ __launch_bounds__(64 * W, 4) void tgemv_b16_kernel(const uint16_t* __restrict__ x,
                                                           const uint8_t* __restrict__ codes,
                                                           const uint16_t* __restrict__ s16,
                                                           int B, int N, int K, int wgs, int bpw,
                                                           float* __restrict__ y) {
  constexpr int WPL = G >= 256 ? 4 : G / 64;       // code words per lane and step
  constexpr int kStep = 64 * WPL;                  // columns per step (at most a group)
  constexpr int kSteps = kB16Cols / kStep;
  constexpr int kSpg = G / kStep;                  // steps per group
  constexpr int kGrp = kB16Cols / G;               // groups per round
  constexpr int kSc = (kGrp + 3) / 4;              // of them, loaded by one lane
  constexpr int kT = 64 * W;
  static_assert(KMAX % kB16Cols == 0 && kB16Cols % G == 0, "whole groups per round and window");
  // the 16-byte piece u of row m sits at u ^ (m % 8), so that the operand
  // reads of 16 rows spread over the banks
  __shared__ __attribute__((aligned(16))) uint8_t lds[32 * KMAX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, kq = lane >> 4;
  const int c = blockIdx.x / wgs, w0 = blockIdx.x % wgs;
  const uint16_t* xm = x + (int64_t)c * B * K;
  const uint8_t* cm = codes + (int64_t)c * N * (K / 4);
  const uint16_t* sm = s16 + (int64_t)c * N * (K / G);
  // block i of this wave
  auto row_of = [&](int i) { return 16 * ((w0 * bpw + i) * W + wave) + n; };

  struct Round {
    uint32_t cw[kSteps][WPL];
    uint16_t sc[kSc];
  };
  // columns col0 .. + 1023 of block i (zero past the row, or past the matrix)
  auto load = [&](Round& q, int i, int col0) {
    const int row = row_of(i);
    const bool ok = i < bpw && row < N;
    const uint8_t* cr = cm + (int64_t)(ok ? row : 0) * (K / 4);
    const uint16_t* sr = sm + (int64_t)(ok ? row : 0) * (K / G);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const int col = col0 + kStep * s;
#pragma unroll
      for (int j = 0; j < WPL; ++j) q.cw[s][j] = 0u;
      if (ok && col < K) {
        const uint8_t* p = cr + col / 4 + 4 * WPL * kq;
        if constexpr (WPL == 4) {
          const u32x4 v = ld16(p);
#pragma unroll
          for (int j = 0; j < 4; ++j) q.cw[s][j] = v[j];
        } else if constexpr (WPL == 2) {
          const u32x2 v = *reinterpret_cast<const u32x2*>(p);
          q.cw[s][0] = v.x;
          q.cw[s][1] = v.y;
        } else {
          q.cw[s][0] = *reinterpret_cast<const uint32_t*>(p);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kSc; ++t) {
      const int g = col0 / G + 4 * t + kq;
      q.sc[t] = ok && g < K / G && 4 * t + kq < kGrp ? sr[g] : (uint16_t)0;
    }
  };

  float tot[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) tot[i][e] = 0.f;

  for (int k0 = 0; k0 < K; k0 += KMAX) {
    const int kw = K - k0 < KMAX ? K - k0 : KMAX;  // columns of this window
    Round cur;
    load(cur, 0, k0);  // in flight during the copy of x
    if (k0 > 0) __syncthreads();  // the window before has been read
    {
      const int ppr = kw / 8;  // 16-byte pieces per row; pieces tid, tid + kT, ...
      const int drow = kT / ppr, dp = kT % ppr;
      int row = tid / ppr, p = tid % ppr;
      while (row < B) {
        u32x4 v[4];
        int r[4], u[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          r[j] = row;
          u[j] = p;
          if (row < B) v[j] = ld16(xm + (int64_t)row * K + k0 + 8 * p);
          row += drow;
          p += dp;
          if (p >= ppr) {
            p -= ppr;
            ++row;
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (r[j] < B) st16(lds + r[j] * (2 * KMAX) + 16 * (u[j] ^ (r[j] & 7)), v[j]);
      }
    }
    __syncthreads();
    // A operand of the 8 columns from col (relative to the window); rows past
    // B hold what was there: an A row only reaches its own output row
    auto xop = [&](int col) {
      return as_bf16x8(*reinterpret_cast<const u32x4*>(lds + n * (2 * KMAX) +
                                                       16 * ((col / 8) ^ (n & 7))));
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i >= bpw) break;
      float part[4][4];  // sums of every fourth group: short chains round less
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[t][e] = 0.f;
      for (int r0 = 0; r0 < kw; r0 += kB16Cols) {
        Round nxt;
        const bool last = r0 + kB16Cols >= kw;
        load(nxt, last ? i + 1 : i, last ? k0 : k0 + r0 + kB16Cols);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
          const int col = r0 + kStep * s;
          if (col >= kw) break;  // uniform
          if (s % kSpg == 0) acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < WPL; ++j) {
            const int at = col + 16 * WPL * kq + 16 * j;
            acc = mfma16(xop(at), decode_half<0>(cur.cw[s][j]), acc);
            acc = mfma16(xop(at + 8), decode_half<1>(cur.cw[s][j]), acc);
          }
          if (s % kSpg == kSpg - 1) {
            const int g = s / kSpg;
            const float sv = h2f((uint16_t)__shfl((int)cur.sc[g / 4], 16 * (g % 4) + n, 64));
#pragma unroll
            for (int e = 0; e < 4; ++e)
              part[g % 4][e] = __builtin_fmaf(acc[e], sv, part[g % 4][e]);
          }
        }
        cur = nxt;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        tot[i][e] += (part[0][e] + part[1][e]) + (part[2][e] + part[3][e]);
    }
  }
  // lane (kq, n) holds batch rows 4 kq + e of weight row n; the codes decode to 2q
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = row_of(i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = 4 * kq + e;
      if (i < bpw && m < B && row < N) y[((int64_t)c * B + m) * N + row] = 0.5f * tot[i][e];
    }
  }
}

constexpr int kB16Chunks = 8;  // 64-column chunks whose loads are in flight together

// Launches of few blocks: one workgroup of four waves per 16-row block, wave w
// on a contiguous quarter of the rows' groups with eight chunks in flight, x
// straight from L2; the four waves' totals meet in LDS in wave order.
template <int G>
__global__ __launch_bounds__(256) void tgemv_b16_few_kernel(const uint16_t* __restrict__ x,
                                                            const uint8_t* __restrict__ codes,
                                                            const uint16_t* __restrict__ s16,
                                                            int B, int N, int K, int nblk,
                                                            float* __restrict__ y) {
  constexpr int NB = 1;
  static_assert(G % 64 == 0 && kB16Chunks % (G / 64 > 0 ? G / 64 : 1) == 0,
                "groups of whole chunks, whole groups per round");
  constexpr int kWpg = G / 64;                // chunks per group
  constexpr int kScales = kB16Chunks / kWpg;  // groups per round
  __shared__ float red[4 * NB * 64 * 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, kq = lane >> 4;
  const int c = blockIdx.x / nblk, j0 = NB * (blockIdx.x % nblk);
  const bool xok = n < B;
  const int ngr = K / G, gpw = (ngr + 3) / 4, g0 = wave * gpw;
  const int gw = ngr - g0 < gpw ? (ngr - g0 > 0 ? ngr - g0 : 0) : gpw;  // groups of this wave
  const int nch = gw * kWpg;
  const uint32_t* crow[NB];
  const uint16_t* srow[NB];
  bool rok[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int row = 16 * (j0 + b) + n;
    rok[b] = row < N;
    crow[b] = reinterpret_cast<const uint32_t*>(codes +
                                                ((int64_t)c * N + (rok[b] ? row : 0)) * (K / 4));
    srow[b] = s16 + ((int64_t)c * N + (rok[b] ? row : 0)) * (K / G);
  }
  const uint16_t* xrow = x + ((int64_t)c * B + (xok ? n : 0)) * K;

  float tot[NB][4];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) tot[b][e] = 0.f;
  for (int i0 = 0; i0 < nch; i0 += kB16Chunks) {
    uint32_t cw[kB16Chunks][NB];
    u32x4 xa[kB16Chunks][2];
    uint16_t sc[NB][kScales];
#pragma unroll
    for (int t = 0; t < kB16Chunks; ++t) {
      const int i = i0 + t;
      const int col = g0 * G + 64 * i + 16 * kq;
      xa[t][0] = xa[t][1] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int b = 0; b < NB; ++b) cw[t][b] = 0u;
      if (i < nch) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (rok[b]) cw[t][b] = crow[b][col / 16];
        if (xok) {
          xa[t][0] = ld16(xrow + col);
          xa[t][1] = ld16(xrow + col + 8);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < kScales; ++r) {
        const int gi = i0 / kWpg + r;
        sc[b][r] = rok[b] && gi < gw ? srow[b][g0 + gi] : (uint16_t)0;
      }
    f32x4 acc[NB];
#pragma unroll
    for (int t = 0; t < kB16Chunks; ++t) {
      if (i0 + t < nch) {  // uniform
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          if (t % kWpg == 0) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
          const uint32_t w = cw[t][b];
          const u32x4 b0 = {(w << 14) & kPairMask, (w << 12) & kPairMask, (w << 10) & kPairMask,
                            (w << 8) & kPairMask};
          const u32x4 b1 = {(w << 6) & kPairMask, (w << 4) & kPairMask, (w << 2) & kPairMask,
                            w & kPairMask};
          acc[b] = mfma16(as_bf16x8(xa[t][0]), as_bf16x8(b0), acc[b]);
          acc[b] = mfma16(as_bf16x8(xa[t][1]), as_bf16x8(b1), acc[b]);
          if (t % kWpg == kWpg - 1) {
            const float s = h2f(sc[b][t / kWpg]);
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[b][e] = __builtin_fmaf(acc[b][e], s, tot[b][e]);
          }
        }
      }
    }
  }
  // lane (kq, n) holds batch rows 4 kq + e of weight row n of each block; the
  // waves meet in LDS
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[((wave * NB + b) * 64 + lane) * 4 + e] = tot[b][e];
  __syncthreads();
  {
    const int b = wave;  // wave b writes block b (NB <= 4)
    if (b < NB) {
      const int row = 16 * (j0 + b) + n;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = 4 * kq + e;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) sum += red[((w * NB + b) * 64 + lane) * 4 + e];
        // the codes decode to 2q
        if (m < B && row < N) y[((int64_t)c * B + m) * N + row] = 0.5f * sum;
      }
    }
  }
}

// Past four blocks per CU x goes through LDS, else each block is a workgroup of
// its own (8 matrices of 1024 x 2048, 512 blocks: 64 workgroups of the first
// form leave the chip idle).  At g = 64 a lane's codes come in 4-byte words,
// and where the 16 waves of K > 2048 take a CU each the first form pays only
// from six or seven blocks per CU on (4 matrices of 4400 x 4096, 1100 blocks: 48
// us at batch 16, 38 as workgroups of their own, 46 and 32 at batch 9; of 6400
// rows, 1600 blocks: 50 and 55, 48 and 43; at g = 128, batch 16: 27 and 34, 29
// and 46).  Blocks per wave: as many, up to four, as
// leave two rounds of workgroups on the chip (each copies x once for all its
// blocks).
template <int G>
static hipError_t launch_b16_g(const uint16_t* x, const uint8_t* codes, const uint16_t* s16,
                               int count, int B, int64_t N, int64_t K, float* y,
                               hipStream_t stream) {
  if (N > 0x7FFFFFFF || K > 0x7FFFFFFF) return hipErrorInvalidValue;
  const bool wide = K > 2048;
  const int64_t nblk = (N + 15) / 16, W = wide ? 16 : 8;
  const int64_t waves = (int64_t)current_cu_count() * 16;  // on the chip at once
  const int per_cu = G == 64 && wide ? (B < 13 ? 7 : 6) : 4;
  if (16 * count * nblk <= per_cu * waves) {
    hipLaunchKernelGGL((tgemv_b16_few_kernel<G>), dim3((unsigned)(count * nblk)), dim3(256), 0,
                       stream, x, codes, s16, B, (int)N, (int)K, (int)nblk, y);
    return hipGetLastError();
  }
  // (16 W bpw rows of a workgroup divide 2^31 where N is near it, so the row
  // numbers of the last one fit an int)
  int64_t bpw = count * nblk / (2 * waves);
  bpw = bpw < 1 ? 1 : (bpw > 4 ? 4 : bpw);
  const int64_t wgs = (nblk + W * bpw - 1) / (W * bpw), grid = count * wgs;
  if (grid < 1 || grid > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (wide)
    hipLaunchKernelGGL((tgemv_b16_kernel<G, 16, 4096>), dim3((unsigned)grid), dim3(1024), 0,
                       stream, x, codes, s16, B, (int)N, (int)K, (int)wgs, (int)bpw, y);
  else
    hipLaunchKernelGGL((tgemv_b16_kernel<G, 8, 2048>), dim3((unsigned)grid), dim3(512), 0,
                       stream, x, codes, s16, B, (int)N, (int)K, (int)wgs, (int)bpw, y);
  return hipGetLastError();
}

bool tgemv_b16_takes(int B, int g) { return B >= 9 && B <= 16 && g >= 64 && g <= 512; }

hipError_t launch_tgemv_b16(const uint16_t* x, const uint8_t* codes, const uint16_t* s16,
                            int count, int B, int64_t N, int64_t K, int g, float* y,
                            hipStream_t stream) {
  if (!tgemv_b16_takes(B, g) || K % 64 != 0 || K % g != 0) return hipErrorInvalidValue;
  switch (g) {
    case 64:  return launch_b16_g<64>(x, codes, s16, count, B, N, K, y, stream);
    case 128: return launch_b16_g<128>(x, codes, s16, count, B, N, K, y, stream);
    case 256: return launch_b16_g<256>(x, codes, s16, count, B, N, K, y, stream);
    case 512: return launch_b16_g<512>(x, codes, s16, count, B, N, K, y, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tmk
