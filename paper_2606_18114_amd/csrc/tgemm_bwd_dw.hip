// Straight-through backward w.r.t. the latent weight (paper Sec. 3.1,
// identity estimator: the gradient of What passes to W unchanged):
//   dW[N, K] = dY[M, N]^T . X[M, K],
// a plain bfloat16 contraction over the M tokens on the gfx950 matrix cores
// (v_mfma_f32_32x32x16_bf16), float32 accumulation.
//
// Both operands arrive token-major, while an MFMA operand lane needs eight
// consecutive tokens of one column.  The tiles are staged in LDS in their
// natural [token][column] order and read with the gfx950 transpose read
// ds_read_b64_tr_b16: in each group of 16 lanes, lane j passes the address of
// 4 columns (col + 4 (j % 4)) of token row j / 4, and lane i receives column
// col + i of 4 consecutive token rows.  Two such reads make one operand.
//
// Tile: 256 (N) x 256 (K) outputs per workgroup of 4 waves (2 x 2), 128 x 128
// per wave (4 x 4 MFMA blocks, accumulators in AGPRs), 32 tokens per stage.
// Stages flow through a 4-deep LDS ring filled by direct-to-LDS loads
// (global_load_lds) three stages ahead; in every token row the 32-byte units
// are XOR-permuted (dw_swz) so that transpose reads are free of bank
// conflicts.
//
// Work split (persistent, one workgroup per CU): the T output tiles are
// dealt round-robin, whole, T / P per workgroup; the T % P remaining tiles
// are cut along the tokens into parts that meet in slots of a caller's
// buffer (tile_parts.hpp), or, without one, by float32 atomics into a
// cleared dW.  Whole tiles are written with plain stores (read-add-write
// when accumulating).
//
// Bound: the matrix cores under the power cap where tiles are many (16384
// tokens of 2048 -> 8512: 464 us, 1.23 PFLOP/s; 637 us while every stage first
// waited for its own LDS reads), the slots' traffic and the reduction where
// they are few (2048 tokens: 81 + 6 us, 131 with atomics).
//
// The direct-to-LDS loads are issued from inline assembly, so the compiler
// neither tracks nor waits for them; each wave issues exactly eight per
// stage and counts them itself (vector-memory operations retire in order).
#include <type_traits>

#include "common.hpp"
#include "launchers.hpp"
#include "tile_parts.hpp"
#include "tile_store.hpp"

namespace tmk {

constexpr int kDwTN = 256, kDwTK = 256, kDwBM = 32, kDwRing = 4;
constexpr int kDwOp = kDwBM * 256 * 2;        // 16 KiB per operand per stage
constexpr int kDwSlot = 2 * kDwOp;            // dY tile, then X tile
constexpr int kDwLds = kDwRing * kDwSlot;     // 128 KiB
constexpr int kDwLoads = 8;                   // direct-to-LDS loads per wave per stage

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__global__ void fill_zero_f32(float* __restrict__ p, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i + 3 < n) {
    *reinterpret_cast<f32x4*>(p + i) = f32x4{0.f, 0.f, 0.f, 0.f};
  } else {
    for (int64_t j = i; j < n; ++j) p[j] = 0.f;
  }
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// lane i: 16 bytes at base + voff -> LDS lds_base + 16 i (lds_base wave-uniform)
__device__ __forceinline__ void dw_dma16(const void* base, uint32_t voff, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(base), "s"(lds_base) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int kVm>
__device__ __forceinline__ void dw_stage_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(kVm) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <int I, int N, typename F>
__device__ __forceinline__ void dw_static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    dw_static_for<I + 1, N>(f);
  }
}

// XOR applied to the 32-byte unit index of token row r: f = (r%4) ^ 2 (r%4)
// is distinct modulo 4 and in its two upper bits over any four consecutive
// rows, so the four rows of a transpose read land in distinct 32-byte bank
// groups, and so do the two column groups (units u, u + 1) read together
__device__ __forceinline__ int dw_swz(int r) { return (r & 3) ^ ((r & 3) << 1); }

// byte offset of (token row r, column c) inside an operand tile, c % 4 == 0
__device__ __forceinline__ uint32_t dw_off(int r, int c) {
  return (uint32_t)(r * 512 + 32 * ((c >> 4) ^ dw_swz(r)) + 2 * (c & 15));
}

// ACC: whole tiles are added to dW (accumulate), else stored; either form has
// the slots and the atomics of cut tiles.  Spills, outside the stages: 92 bytes a
// lane, 84 with ACC; with both ways of writing whole tiles in one kernel 152, a
// form without the atomics 192.  2048 tokens x 8512 x 2048: 88.5 us (91.9 in one
// kernel); 1000 x 3352 x 768: 36.2 (38.6).
template <bool ACC>
__global__ __launch_bounds__(256) void tgemm_bwd_dw_kernel(
    const uint16_t* __restrict__ dY, const uint16_t* __restrict__ X, int64_t M, int64_t N,
    int64_t K, float* __restrict__ dW, uint32_t tiles_k, uint32_t full, uint32_t rem,
    uint32_t parts, int per, float* __restrict__ slots) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kDwLds];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wy = wave >> 1, wx = wave & 1;  // 128-row (N) and 128-column (K) halves
  const int g = lane >> 4;                  // 16-lane group of the transpose reads
  const int j16 = lane & 15;
  const uint32_t P = gridDim.x;
  const uint32_t bid = xcd_remap(blockIdx.x, P);
  const int nst = (int)((M + kDwBM - 1) / kDwBM);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

  // this lane's transpose-read address inside an operand tile, for token
  // rows k0 .. k0+3 (k0 = 8 (g / 2) + 4 rd) and the 16 columns of its group
  const int trow = 8 * (g >> 1) + (j16 >> 2);
  const int tcol = 16 * (g & 1) + 4 * (j16 & 3);

  for (uint32_t item = 0;; ++item) {
    // ---- the item: a whole tile, or one token range of a remaining tile ----
    uint32_t tile;
    int s_beg, s_end;
    bool whole;
    if (item < full) {
      tile = item * P + bid;
      s_beg = 0;
      s_end = nst;
      whole = true;
    } else if (item == full && bid < rem * parts) {
      // part bid / rem of leftover tile bid % rem
      // (the quotients are computed in vector registers: the loaders need
      // them in scalar ones)
      const uint32_t part = (uint32_t)__builtin_amdgcn_readfirstlane((int)(bid / rem));
      tile = full * P + (bid - part * rem);
      s_beg = (int)part * per;
      s_end = s_beg + per < nst ? s_beg + per : nst;
      whole = parts == 1;
    } else {
      break;
    }
    const int64_t n0 = (int64_t)(tile / tiles_k) * kDwTN;
    const int64_t k0 = (int64_t)(tile % tiles_k) * kDwTK;

    // ---- loader: wave w loads dY rows 8w .. 8w+7 and X rows 8w .. 8w+7 of a
    // stage, 2 rows (1 KiB) per load; lane -> row 2J + lane/32, 16-byte piece
    // lane%32 of the LDS row, holding logical piece lp (unit-permuted)
    uint32_t ycol[4], xcol[4];  // byte offsets of this lane's columns in a row
    uint32_t yrow[4], xrow[4];  // and of its rows in a stage
    const int r_lo = lane >> 5;   // row of load i: 2 (4 wave + i) + r_lo
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 2 * (wave * 4 + i) + r_lo;
      const int p = lane & 31;
      const int lp = 2 * ((p >> 1) ^ dw_swz(r)) + (p & 1);
      int64_t cn = n0 + 8 * lp;
      cn = cn < N ? cn : N - 8;  // past N: re-read the last piece (columns unused)
      int64_t ck = k0 + 8 * lp;
      ck = ck < K ? ck : K - 8;
      ycol[i] = (uint32_t)cn * 2u;
      xcol[i] = (uint32_t)ck * 2u;
      yrow[i] = (uint32_t)r * (uint32_t)N * 2u;
      xrow[i] = (uint32_t)r * (uint32_t)K * 2u;
    }
    struct DmaStage {
      const uint8_t *yb, *xb;
      uint32_t ylast, xlast, dst;
    };
    auto dma_begin = [&](int st, int slot) {
      st = st < s_end ? st : s_end - 1;  // past the range: reload its last stage
      const int64_t m0 = (int64_t)st * kDwBM;
      // rows past M re-read row M - 1 (in bounds); those tokens are zeroed in
      // the dY operand below
      const uint32_t last = (uint32_t)(M - m0 < kDwBM ? M - m0 : kDwBM) - 1u;
      DmaStage d;
      d.yb = reinterpret_cast<const uint8_t*>(dY + m0 * N);
      d.xb = reinterpret_cast<const uint8_t*>(X + m0 * K);
      d.ylast = last * (uint32_t)N * 2u;
      d.xlast = last * (uint32_t)K * 2u;
      d.dst = lds0 + slot * kDwSlot + 4096u * wave;
      return d;
    };
    // load J of the eight of a stage: dY rows (0-3), X rows (4-7)
    auto dma_piece = [&](const DmaStage& d, auto j_tag) {
      constexpr int J = decltype(j_tag)::value, i = J % 4;
      if constexpr (J < 4)
        dw_dma16(d.yb, (yrow[i] < d.ylast ? yrow[i] : d.ylast) + ycol[i], d.dst + 1024 * i);
      else
        dw_dma16(d.xb, (xrow[i] < d.xlast ? xrow[i] : d.xlast) + xcol[i],
                 d.dst + kDwOp + 1024 * i);
    };
    auto dma = [&](int st, int slot) {
      const DmaStage d = dma_begin(st, slot);
      dw_static_for<0, kDwLoads>([&](auto j_tag) { dma_piece(d, j_tag); });
    };

    f32x16 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    // prologue: stages s_beg .. s_beg + 2 in flight, the first two landed
#pragma unroll
    for (int p = 0; p < kDwRing - 1; ++p) dma(s_beg + p, p);
    dw_stage_barrier<kDwLoads>();

    // per-lane byte offsets of the transpose reads of block a (dY) / b (X)
    // inside a stage's operand tile, token rows trow .. (the reads of token
    // group t and half rd add 16 t and 4 rd rows, i.e. constant offsets)
    uint32_t aoff[4], boff[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) aoff[a] = dw_off(trow, wy * 128 + 32 * a + tcol);
#pragma unroll
    for (int b = 0; b < 4; ++b) boff[b] = kDwOp + dw_off(trow, wx * 128 + 32 * b + tcol);
    auto frag = [&](const uint8_t* sb, uint32_t off, int t) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4*)(sb + off + 16 * t * 512));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4*)(sb + off + (16 * t + 4) * 512));
      const u32x2 l = __builtin_bit_cast(u32x2, lo), u = __builtin_bit_cast(u32x2, hi);
      return u32x4{l.x, l.y, u.x, u.y};
    };
    // operands of the two 16-token steps of a stage; read X of a step in the
    // order its MFMAs first use them
    u32x4 af[2][4], bf[2][4];
    auto read_op = [&](const uint8_t* sb, auto t_tag, auto x_tag) {
      constexpr int T = decltype(t_tag)::value, X_ = decltype(x_tag)::value;
      if constexpr (X_ == 0)
        af[T][0] = frag(sb, aoff[0], T);
      else if constexpr (X_ < 5)
        bf[T][X_ - 1] = frag(sb, boff[X_ - 1], T);
      else
        af[T][X_ - 4] = frag(sb, aoff[X_ - 4], T);
    };

    // One full stage in ring slot SLOT (a compile-time constant, so every LDS
    // address is a register plus an immediate offset).  One wave per SIMD
    // issues everything, so the order is fixed by hand, one MFMA per slot
    // fenced by sched_barrier: the first step's operands were read during
    // the stage before; its 16 MFMAs cover the reads of the second step (even
    // slots) and the eight loads of stage st + 3 (odd slots), and the second
    // step's MFMAs the first reads of stage st + 1.  No MFMA waits for an LDS
    // read issued less than two MFMAs earlier.
    auto stage = [&](auto slot_tag, int st) {
      constexpr int SLOT = decltype(slot_tag)::value;
      const uint8_t* sb = lds + SLOT * kDwSlot;
      const uint8_t* nb = lds + ((SLOT + 1) & (kDwRing - 1)) * kDwSlot;
      const DmaStage d = dma_begin(st + kDwRing - 1, (SLOT + kDwRing - 1) & (kDwRing - 1));
      dw_static_for<0, 32>([&](auto k_tag) {
        constexpr int k = decltype(k_tag)::value;
        constexpr int t = k / 16, a = (k % 16) / 4, b = k % 4;
        acc[a][b] = mfma32(as_bf16x8(af[t][a]), as_bf16x8(bf[t][b]), acc[a][b]);
        if constexpr (k % 2 == 0)
          read_op(t == 0 ? sb : nb, std::integral_constant<int, 1 - t>{},
                  std::integral_constant<int, (k % 16) / 2>{});
        else if constexpr (k < 16)
          dma_piece(d, std::integral_constant<int, k / 2>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    // the same without the overlap, for the last stages: tokens past M
    // contribute nothing (their dY values are zeroed in the operand)
    auto stage_tail = [&](auto slot_tag, int st) {
      constexpr int SLOT = decltype(slot_tag)::value;
      const uint8_t* sb = lds + SLOT * kDwSlot;
      const int64_t mvalid = M - (int64_t)st * kDwBM;
#pragma unroll
      for (int t = 0; t < kDwBM / 16; ++t) {
        u32x4 ta[4], tb[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) ta[a] = frag(sb, aoff[a], t);
#pragma unroll
        for (int b = 0; b < 4; ++b) tb[b] = frag(sb, boff[b], t);
        if (mvalid < kDwBM) {
          // this lane's tokens: 16 t + 8 (g / 2) + e, e = 0 .. 7 (pairs per dword)
          const int base = 16 * t + 8 * (g >> 1);
#pragma unroll
          for (int a = 0; a < 4; ++a) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int m_lo = base + 2 * e;
              const uint32_t keep =
                  (m_lo < mvalid ? 0x0000FFFFu : 0u) | (m_lo + 1 < mvalid ? 0xFFFF0000u : 0u);
              ta[a][e] &= keep;
            }
          }
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            acc[a][b] = mfma32(as_bf16x8(ta[a]), as_bf16x8(tb[b]), acc[a][b]);
      }
    };

    // groups of kDwRing full stages, then the rest
    const int s_full = s_end < nst || M % kDwBM == 0 ? s_end : s_end - 1;
    int st0 = s_beg;
    if (st0 + kDwRing <= s_full)
      dw_static_for<0, 8>([&](auto x_tag) {
        read_op(lds, std::integral_constant<int, 0>{}, x_tag);
      });
    for (; st0 + kDwRing <= s_full; st0 += kDwRing) {
      dw_static_for<0, kDwRing>([&](auto i_tag) {
        stage(i_tag, st0 + decltype(i_tag)::value);
        dw_stage_barrier<kDwLoads>();
      });
    }
    for (; st0 < s_end; st0 += kDwRing) {  // (the stages past s_end only load and wait)
      dw_static_for<0, kDwRing>([&](auto i_tag) {
        constexpr int i = decltype(i_tag)::value;
        const int st = st0 + i;
        dma(st + kDwRing - 1, (i + kDwRing - 1) & (kDwRing - 1));
        if (st < s_end) stage_tail(i_tag, st);
        dw_stage_barrier<kDwLoads>();
      });
    }
    // every load of this item has landed before the ring is reused
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();

    // ---- write
    auto val = [&](int a, int b, int i) { return acc_value(acc[a][b][i]); };
    auto none = [](int) {};
    const int64_t row0 = n0 + wy * 128, col0 = k0 + wx * 128;
    const int rows_left = (int)(N - row0 < 256 ? N - row0 : 256);
    const int cols_left = (int)(K - col0 < 256 ? K - col0 : 256);
    float* out = dW + row0 * K + col0;
    if (!whole && slots)
      slot_store(slots + (int64_t)bid * kSlotFloats, rows_left, cols_left, none, val);
    else if (!whole)
      tile_store(out, K, rows_left, cols_left, none, val,
                 [](float* p, float v) { atomicAdd(p, v); });
    else if constexpr (ACC)
      tile_add(out, K, rows_left, cols_left, val);
    else
      tile_store(out, K, rows_left, cols_left, none, val, [](float* p, float v) { *p = v; });
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// zeroes tiles t0 .. t0 + count - 1 of a float32 [rows, cols] array dealt in
// 256 x 256 tiles (tile t: row block t / tiles_c, column block t % tiles_c),
// skipping rows and columns past the array: one workgroup of 64 threads per
// tile row (cols % 4 == 0, 16-byte aligned base)
__global__ void zero_tiles_f32(float* __restrict__ out, int64_t rows, int64_t cols,
                               uint32_t tiles_c, uint32_t t0) {
  const uint32_t t = t0 + blockIdx.x / 256u;
  const int64_t r = (int64_t)(t / tiles_c) * 256 + blockIdx.x % 256u;
  const int64_t c = (int64_t)(t % tiles_c) * 256 + 4 * threadIdx.x;
  if (r < rows && c < cols) *reinterpret_cast<f32x4*>(out + r * cols + c) = f32x4{0.f, 0.f, 0.f, 0.f};
}

hipError_t launch_zero_tiles_f32(float* out, int64_t rows, int64_t cols, int64_t tiles_c,
                                 int64_t t0, int64_t count, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_tiles_f32, dim3((unsigned)(count * 256)), dim3(64), 0, stream, out,
                     rows, cols, (uint32_t)tiles_c, (uint32_t)t0);
  return hipGetLastError();
}

hipError_t launch_fill_zero_f32(float* dst, int64_t n, hipStream_t stream) {
  const int64_t threads = (n + 3) / 4;
  hipLaunchKernelGGL(fill_zero_f32, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream,
                     dst, n);
  return hipGetLastError();
}

// Time of one group of ring stages (four, 128 tokens) of a tile, of a slot's
// write and read, and of the reduction's launch; see plan_parts
constexpr double kDwUnitUs = 3.6, kDwSlotUs = 0.1, kDwLaunchUs = 5.0;

static TilePlan dw_plan(int64_t M, int64_t N, int64_t K) {
  const int64_t nt = ((N + kDwTN - 1) / kDwTN) * ((K + kDwTK - 1) / kDwTK);
  return plan_parts(nt, (M + kDwBM - 1) / kDwBM, kDwRing, current_cu_count(), kDwUnitUs,
                    kDwSlotUs, kDwLaunchUs);
}

int64_t bwd_dw_slot_bytes(int64_t M, int64_t N, int64_t K) {
  return dw_plan(M, N, K).slots() * kSlotBytes;
}

hipError_t launch_tgemm_bwd_dw_parts(const uint16_t* dY, const uint16_t* X, int64_t M, int64_t N,
                                     int64_t K, float* dW, int accumulate, float* slots,
                                     hipStream_t stream) {
  const int64_t tn = (N + kDwTN - 1) / kDwTN, tk = (K + kDwTK - 1) / kDwTK;
  const int64_t ntiles = tn * tk;
  TilePlan t = dw_plan(M, N, K);
  if (t.parts > 1 && !slots) {
    t = plan_atomic(ntiles, (M + kDwBM - 1) / kDwBM, current_cu_count());
    if (t.rem && t.parts > 1 && !accumulate) {  // these tiles are summed with atomics
      const hipError_t e = launch_zero_tiles_f32(dW, N, K, tk, ntiles - t.rem, t.rem, stream);
      if (e != hipSuccess) return e;
    }
  }
#define TM_DW_CASE(ACC_)                                                                          \
  hipLaunchKernelGGL(tgemm_bwd_dw_kernel<ACC_>, dim3((unsigned)t.grid), dim3(256), 0, stream, dY, \
                     X, M, N, K, dW, (uint32_t)tk, (uint32_t)t.full, (uint32_t)t.rem,             \
                     (uint32_t)t.parts, t.per, slots)
  if (accumulate)
    TM_DW_CASE(true);
  else
    TM_DW_CASE(false);
#undef TM_DW_CASE
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || t.parts == 1 || !slots) return e;
  return launch_reduce_parts(slots, t.rem, t.parts, ntiles - t.rem, tk, N, K, dW, false,
                             accumulate != 0, stream);
}

hipError_t launch_tgemm_bwd_dw(const uint16_t* dY, const uint16_t* X, int64_t M, int64_t N,
                               int64_t K, float* dW, int accumulate, hipStream_t stream) {
  return launch_tgemm_bwd_dw_parts(dY, X, M, N, K, dW, accumulate, nullptr, stream);
}

}  // namespace tmk
