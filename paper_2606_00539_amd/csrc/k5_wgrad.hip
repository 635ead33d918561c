// K5, the gradient pass fused into its producer for CDNA4 (gfx950): the
// weight-gradient GEMM of a linear layer with the sum of squares that the
// controller needs computed in its epilogue, so that the gradient is never
// read back from HBM for its norm (the norm is the only per-unit quantity
// the controller takes from the gradient, Sec. 3.3 and Alg. 1; it is cheap
// to compute from what the producer already holds, Sec. 3.1).
//
//   dw[o][i] = bf16_rne( sum_t dy[t][o] * x[t][i] )   fp32 accumulation
//   (accumulating problems: bf16_rne( fp32(dw_old[o][i] + that sum) ))
//   tile_ss[tile] = sum over the tile of float(dw)^2  fp32, fixed order
//
// dy: [tokens][out] bf16, x: [tokens][in] bf16, dw: [out][in] bf16, all
// row-major.  The contraction runs over the slow (token) index of both
// operands, so both tiles sit in LDS exactly as they arrive ([k][feature],
// features contiguous) and reach the matrix cores through the transposing
// LDS read ds_read_b64_tr_b16, which hands each lane four consecutive k of
// one feature.
//
// Tiling: one 256-lane workgroup per 256x256 output tile, four waves of
// 128x128 (4x4 v_mfma_f32_32x32x16_bf16 blocks each), K steps of 64 split
// into four slots of 16 (one matrix-core instruction per block and slot).
// Two LDS buffers and one set of staging registers form the pipeline:
// during step s the matrix cores work on buffer s%2, the staged operands of
// step s+1 go to the other buffer while the global loads of step s+2 refill
// the staging registers, so every global load has a whole step to land.
// The fragments of slot k+1 are read from LDS while slot k's matrix-core
// instructions run (two fragment register sets), and the workgroup meets at
// one barrier per step, placed before the last slot's matrix-core work so
// that the reads of the next buffer overlap it.  x is the matrix cores' A
// operand, so the four accumulator rows a lane holds per group are four
// consecutive output columns, 8 contiguous bytes once rounded.  Overwritten
// tiles that lie wholly inside dw pass through LDS and leave as full rows;
// the others store each lane's 8 bytes directly.
//
// Launches whose 256 tiles would leave most CUs idle run in 128x128 or 64x64
// tiles instead (tile_edge), and k5_tile_sums then forms the sums of the
// 256x256 tiles.  Every tile size accumulates over k in the same order, and the
// squares are added in the same order, so the results have the same bits.
// The 28 gradients of a 4-layer, d = 256 model at 2,037 tokens (52 tiles of 256):
// 93 us in 256 tiles (two launches of at most 16 problems), 26 us in 208 tiles
// of 128 (one launch of at most 32, 21 us, and the sums, 5 us).

#include <algorithm>
#include <type_traits>

#include "gnmr_internal.h"
#include "lane_ops.h"

namespace gnmr {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) u32x2 g_vec2;
typedef __attribute__((address_space(1))) u32x4 g_vec4;
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// Buffer resource word 3 for gfx9-family raw (untyped) buffers.
constexpr int kBufferWord3 = 0x00020000;
static_assert(kWgBM == kWgBN, "square tiles: one load pattern serves both operands");
static_assert(kWgBK == 64, "four slots of 16 per K step");

// Geometry of a kT x kT workgroup tile (kT = 256, 128 or 64): four waves, a
// quarter of the tile each, as kB x kB matrix-core blocks of 32x32.
template <int kT>
struct Tile {
  static constexpr int kB = kT / 64;         // blocks per wave and dimension
  static constexpr int kW = kT / 2;          // rows and columns of a wave's quarter
  static constexpr int kVec = kT / 8;        // 16-byte vectors per tile row
  static constexpr int kRow = kT + 32;       // LDS row stride: rows fall 64 B apart in the banks
  static constexpr int kStage = kWgBK * kRow;  // elements per operand and stage
  // 16-byte chunks per lane, operand and stage; tile rows the workgroup covers at once
  static constexpr int kChunks = kWgBK * kVec / kWgThreads;
  static constexpr int kPass = kWgThreads / kVec;
  static constexpr int kAhead = kT == 256 ? 1 : kT == 128 ? 2 : 4;  // K steps in staging registers
  static constexpr int kSets = kT == 64 ? 4 : 2;                    // fragment register sets
};
// sched_group_barrier instruction classes
constexpr int kSchedMfma = 0x008;
constexpr int kSchedVmemRead = 0x020;
constexpr int kSchedDsRead = 0x100;
constexpr int kSchedDsWrite = 0x200;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two fp32 values to packed bf16 (lo in the low half), round to nearest
// even, a NaN to a quiet NaN with its payload kept: one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

__device__ __forceinline__ float bf16_val(uint32_t b) { return __uint_as_float(b << 16); }

__device__ __forceinline__ bf16x8 frag(const uint16_t* p0, const uint16_t* p1) {
  const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p0);
  const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p1);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The problem that tile v of the launch belongs to; v becomes its tile there.
// (A single problem has kernels of its own: 2 KiB of arguments and this search are
// 0.5 us of the 6 to 10 that a small gradient takes.  8 x 48 of 5 tokens 6.2 and 5.7
// us, 512 x 512 of 100 9.6 and 9.0, 4096 x 4096 of 64 12.9 and 12.2.)
template <int kMost>
__device__ __forceinline__ int problem_of(const WgBatchOf<kMost>& batch, int& v) {
  int pi = 0, begin = 0;
#pragma unroll
  for (int i = 1; i < kMost; ++i) {
    const int b = batch.tile_begin[i];  // INT32_MAX past the last problem
    if (v >= b) {
      pi = i;
      begin = b;
    }
  }
  v -= begin;
  return pi;
}

// A 256x256 (or smaller) bf16 tile of dw at (m0, n0) in LDS: rows of kT
// elements without padding, chunk c of row r in slot c ^ (r % kVec), so that
// reads of 32 consecutive rows at one column spread over the banks.  Loaded by
// direct-to-LDS 16-byte loads, which need no registers: each wavefront
// instruction fills 1 KiB of consecutive rows.  Rows or columns outside dw
// read its last row or vector instead (never used).
template <int kT, int kWaves>
__device__ __forceinline__ void tile_to_lds(uint16_t* tile, const uint16_t* dw, int m0, int n0,
                                            int M, int N, int tid) {
  constexpr int kVec = Tile<kT>::kVec, kRows = 64 / kVec;  // rows per instruction
  constexpr int kLoads = kT / kRows / kWaves;              // instructions per wave
  const int row0 = __builtin_amdgcn_readfirstlane(tid >> 6) * kLoads * kRows;
  const int lane = tid & 63, lrow = lane / kVec;
#pragma unroll 1
  for (int q = 0; q < kLoads; ++q) {
    const int first = row0 + q * kRows, row = first + lrow;
    const int m = min(m0 + row, M - 1);
    const int n = min(n0 + 8 * ((lane % kVec) ^ (row & (kVec - 1))), N - 8);
    __builtin_amdgcn_global_load_lds((const void*)(dw + int64_t(m) * N + n),
                                     (__attribute__((address_space(3))) void*)(tile + first * kT),
                                     16, 0, 0);
  }
  __builtin_amdgcn_s_waitcnt(0);
}

// Address in such a tile of the four elements at (row, col .. col+3).
template <int kT>
__device__ __forceinline__ uint16_t* tile_at(uint16_t* tile, int row, int col) {
  constexpr int kVec = Tile<kT>::kVec;
  return &tile[row * kT + 8 * ((col >> 3) ^ (row & (kVec - 1))) + (col & 7)];
}

// Adds the squares of four packed bf16 values to ss, in order.
__device__ __forceinline__ void add_squares(const u32x2& p, float& ss) {
  const float q0 = __uint_as_float(p.x << 16), q1 = __uint_as_float(p.x & 0xFFFF0000u),
              q2 = __uint_as_float(p.y << 16), q3 = __uint_as_float(p.y & 0xFFFF0000u);
  ss = fmaf(q0, q0, ss);
  ss = fmaf(q1, q1, ss);
  ss = fmaf(q2, q2, ss);
  ss = fmaf(q3, q3, ss);
}

// The sum over a wave's lanes (a butterfly) to red[wave], for the first four
// waves of the workgroup.
__device__ __forceinline__ void wave_sum_to(float ss, float* red, int tid) {
  ss = wave_sum(ss);
  if ((tid & 63) == 0 && tid < kWgThreads) red[tid >> 6] = ss;
}

// kAcc: every problem of the batch accumulates into its stored dw (true) or
// overwrites it (false); a batch of both kinds takes one launch of each.
// kT: the tile edge.  256 writes the tile sums itself; the smaller tiles leave
// them to k5_tile_sums.
// kRows: accumulated tiles leave in full rows (rows_pay).
// kMost: the problems that a batch has room for.
template <bool kAcc, int kT, bool kRows, int kMost>
__global__ __launch_bounds__(kWgThreads, kT == 256 ? 1 : 2) void k5_wgrad(
    const WgBatchOf<kMost> batch) {
  using G = Tile<kT>;
  constexpr int kB = G::kB, kW = G::kW, kRow = G::kRow, kChunks = G::kChunks, kPass = G::kPass;
  constexpr int kAhead = G::kAhead, kSets = G::kSets;
  __shared__ __attribute__((aligned(16))) uint16_t lds[2][2][G::kStage];  // [stage][x, dy]

  // Workgroup -> tile: workgroups w, w+8, ... run on one XCD, so give each
  // XCD a contiguous run of the tile order (over all problems of the batch);
  // inside a problem the order walks groups of 8 tile rows column by column,
  // so that the tiles an XCD holds at once share their dy and x panels in
  // its L2.
  const int total = batch.total_tiles;
  const int w = blockIdx.x;
  const int xcd = w % kNumXcd, q = total / kNumXcd, r = total % kNumXcd;
  int v = xcd * q + (xcd < r ? xcd : r) + w / kNumXcd;
  const WgProblem& P = batch.p[problem_of(batch, v)];
  const uint16_t* __restrict__ dy = P.dy;
  const uint16_t* __restrict__ x = P.x;
  uint16_t* __restrict__ dw = P.dw;
  const int64_t K = P.K;
  const int M = P.M, N = P.N, tiles_m = P.tiles_m, tiles_n = P.tiles_n;
  const int per_group = kWgGroupRows * tiles_n;
  const int first_m = (v / per_group) * kWgGroupRows;
  const int rows = tiles_m - first_m < kWgGroupRows ? tiles_m - first_m : kWgGroupRows;
  const int tm = first_m + (v % per_group) % rows;
  const int tn = (v % per_group) / rows;
  const int m0 = tm * kT, n0 = tn * kT;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;  // this wave's quarter of the tile

  // Global -> LDS: lane tid moves 16-byte chunk (row tid/kVec + kPass*c, column
  // 8*(tid%kVec)) of each operand tile, c < kChunks, with buffer loads whose
  // resource covers the rows of one K step: rows past K and columns past M
  // or N (whose offset is pushed past the resource) read as zero in
  // hardware, so every load is issued unconditionally (M, N multiples of 8:
  // a chunk is all in or all out).  Steps past the end get an empty
  // resource: their loads read zeros without touching memory, and the
  // buffers they fill are never read, which keeps the loop body free of
  // branches.
  const int lrow = tid / G::kVec, lcol = (tid % G::kVec) * 8;
  const uint32_t kOut = 0x80000000u;  // beyond any resource of this kernel
  const uint32_t xo = n0 + lcol < N ? uint32_t((lrow * N + n0 + lcol) * 2) : kOut;
  const uint32_t yo = m0 + lcol < M ? uint32_t((lrow * M + m0 + lcol) * 2) : kOut;
  u32x4 rx[kAhead][kChunks], ry[kAhead][kChunks];
  __amdgpu_buffer_rsrc_t xr, yr;
  auto rsrc = [&](int64_t k0) {
    const int64_t kb = k0 < K ? k0 : 0;
    const int rws = k0 >= K ? 0 : (K - k0 < kWgBK ? int(K - k0) : kWgBK);
    xr = __builtin_amdgcn_make_buffer_rsrc((void*)(x + kb * N), 0, rws * N * 2, kBufferWord3);
    yr = __builtin_amdgcn_make_buffer_rsrc((void*)(dy + kb * M), 0, rws * M * 2, kBufferWord3);
  };
  constexpr int kPairs = 2 * kChunks;
  // A step is staged in kPairs pairs p = 2 * chunk + operand (0: x, 1: dy).
  auto gload = [&](int a, int lo, int hi) {
#pragma unroll
    for (int p = lo; p < hi; ++p) {
      const int c = p >> 1;
      if ((p & 1) == 0)
        rx[a][c] = __builtin_bit_cast(
            u32x4,
            __builtin_amdgcn_raw_buffer_load_b128(xr, xo + uint32_t(c * 2 * kPass * N), 0, 0));
      else
        ry[a][c] = __builtin_bit_cast(
            u32x4,
            __builtin_amdgcn_raw_buffer_load_b128(yr, yo + uint32_t(c * 2 * kPass * M), 0, 0));
    }
  };
  auto lstore = [&](int buf, int a, int lo, int hi) {
#pragma unroll
    for (int p = lo; p < hi; ++p) {
      const int c = p >> 1;
      *(u32x4*)&lds[buf][p & 1][(lrow + kPass * c) * kRow + lcol] = p & 1 ? ry[a][c] : rx[a][c];
    }
  };

  // Fragment addressing for ds_read_b64_tr_b16: within each 16-lane group the
  // read hands lane i column i of the 4x16 block that the group's 8-byte
  // chunks form (chunk of lane 4j + c = row j, columns 4c..4c+3).  Lane l
  // then holds feature l%32 of a 32-wide block and k = 8*(l/32) + 4h + j for
  // the two reads h = 0, 1: the same k order for both operands.
  const int f_row = 8 * (lane >> 5) + ((lane & 15) >> 2);
  const int f_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  bf16x8 fx[kSets][kB], fy[kSets][kB];  // [register set][block]
  auto rfrag = [&](int set, int buf, int kk) {
    const uint16_t* lx = &lds[buf][0][f_row * kRow + wn * kW + f_col];
    const uint16_t* ly = &lds[buf][1][f_row * kRow + wm * kW + f_col];
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const int o = kk * 16 * kRow + 32 * b;
      fx[set][b] = frag(lx + o, lx + o + 4 * kRow);
      fy[set][b] = frag(ly + o, ly + o + 4 * kRow);
    }
  };

  f32x16 acc[kB][kB];
#pragma unroll
  for (int i = 0; i < kB; ++i)
#pragma unroll
    for (int j = 0; j < kB; ++j) acc[i][j] = f32x16{};
  auto mfma = [&](int set) {
#pragma unroll
    for (int i = 0; i < kB; ++i)
#pragma unroll
      for (int j = 0; j < kB; ++j)
        acc[i][j] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[set][j], fy[set][i], acc[i][j], 0, 0, 0);
  };
  const int64_t nk = (K + kWgBK - 1) / kWgBK;  // 0 steps for an empty batch: dw = 0
  if constexpr (kT >= 128) {
    // Instruction order inside a slot (scheduling hints only): the fragment reads
    // for the next slot first, three to a matrix-core instruction (four in the 128
    // tile), then the staged pairs' stores and loads, spaced out.  A wave that
    // finds the LDS queue full holds up the matrix cores, with one wave per SIMD.
    // 256 tile, 4096^3 and the gradients of a layer (d = 5,120, 4,096 tokens):
    // 112.6 and 2,167 us; two reads each, then a pair behind each of the next:
    // 114.8 and 2,195; reads and stores mixed over the slot: 118 to 121 and 2,370
    // to 2,470.  128 tile, 1024 x 2048 and 2048 x 2048 gradients of 8,192 and 4,096
    // tokens: 66.6 and 44.8 us, mixed and in two slots 75.0 and 47.1.
    auto order = [](auto stores) {
      constexpr int kStores = decltype(stores)::value;
      if constexpr (kT == 128) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
          __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 4, 0);
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          if (i < 2) __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
          if (i < kStores) {
            __builtin_amdgcn_sched_group_barrier(kSchedDsWrite, 1, 0);
            __builtin_amdgcn_sched_group_barrier(kSchedVmemRead, 1, 0);
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
          __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
          __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 3, 0);
        }
        __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 1, 0);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          if (i < kStores) {
            __builtin_amdgcn_sched_group_barrier(kSchedDsWrite, 1, 0);
            __builtin_amdgcn_sched_group_barrier(kSchedVmemRead, 1, 0);
          }
          if (i < 5) __builtin_amdgcn_sched_group_barrier(kSchedMfma, 2, 0);
        }
      }
    };
    // Pairs staged by the end of slots 0, 1 and 2.  In 256 tiles a slot's 16
    // matrix-core instructions take 512 cycles of a CU and its 16 reads and 8
    // stores per wave 529 cycles of LDS, so 8/8/0 pairs left the first two slots
    // waiting for LDS; 6/5/5 fit all three.  The gradients of a layer (d = 5,120)
    // at 4,096 tokens: 2,133 us at 8/8/0, 2,087 us at 6/5/5 (2,091-2,094 us at
    // 6/6/4, 5/5/6 and 4/6/6).  The 128 tile's eight pairs: 3/3/2.
    constexpr int kCut0 = kT == 256 ? 6 : 3, kCut1 = kT == 256 ? 11 : 6;
    using std::integral_constant;

    // Prologue: step 0 in buffer 0, steps 1 .. kAhead in the staging
    // registers (step s in set s % kAhead), the first slot's fragments read.
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      rsrc(int64_t(a) * kWgBK);
      gload(a, 0, kPairs);
    }
    lstore(0, 0, 0, kPairs);
    rsrc(int64_t(kAhead) * kWgBK);
    gload(0, 0, kPairs);
    __syncthreads();
    rfrag(0, 0, 0);
    for (int64_t s0 = 0; s0 < nk; s0 += kAhead) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int64_t s = s0 + u;
        if (u > 0 && s >= nk) break;
        const int buf = kAhead > 1 ? u & 1 : int(s & 1), a = (u + 1) % kAhead;
        // slot 0: stage part of step s+1, load the same part of step s+1+kAhead
        rfrag(1, buf, 1);
        lstore(buf ^ 1, a, 0, kCut0);
        rsrc((s + 1 + kAhead) * kWgBK);
        gload(a, 0, kCut0);
        mfma(0);
        order(integral_constant<int, kCut0>{});
        // slot 1
        rfrag(0, buf, 2);
        lstore(buf ^ 1, a, kCut0, kCut1);
        gload(a, kCut0, kCut1);
        mfma(1);
        order(integral_constant<int, kCut1 - kCut0>{});
        // slot 2
        rfrag(1, buf, 3);
        lstore(buf ^ 1, a, kCut1, kPairs);
        gload(a, kCut1, kPairs);
        mfma(0);
        order(integral_constant<int, kPairs - kCut1>{});
        // slot 3: every wave has stored its part of step s+1 and read its last
        // fragments of buffer s%2 (the barrier waits for both), so buffer
        // (s+1)%2 is complete and buffer s%2 free for step s+2
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        rfrag(0, buf ^ 1, 0);
        mfma(1);
        order(integral_constant<int, 0>{});
      }
    }
  } else {
    // The 64 tile: a step has four matrix-core instructions per wave, less
    // than the latency of one LDS read, so it reads all its fragments at once
    // behind its one barrier.
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      rsrc(int64_t(a) * kWgBK);
      gload(a, 0, kPairs);
    }
    lstore(0, 0, 0, kPairs);
    rsrc(int64_t(kAhead) * kWgBK);
    gload(0, 0, kPairs);
    for (int64_t s0 = 0; s0 < nk; s0 += kAhead) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int64_t s = s0 + u;
        if (s >= nk) break;
        const int buf = u & 1, a = (u + 1) % kAhead;
        // Buffer s%2 is complete, and every wave has its fragments of step
        // s-1, so buffer (s+1)%2 is free.
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kSets; ++kk) rfrag(kk, buf, kk);
        lstore(buf ^ 1, a, 0, kPairs);
        rsrc((s + 1 + kAhead) * kWgBK);
        gload(a, 0, kPairs);
#pragma unroll
        for (int kk = 0; kk < kSets; ++kk) mfma(kk);
        // Reads first, then a pair behind each matrix-core instruction (left to
        // the compiler the stores mixed with the reads: 512 x 512 of 4,096 tokens
        // 29.7 us, now 25.2; 1024 x 1024 of 8,192 51.1 and 42.4).
        __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 12, 0);
        __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 4, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (i < 3) __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
          __builtin_amdgcn_sched_group_barrier(kSchedDsWrite, 1, 0);
          __builtin_amdgcn_sched_group_barrier(kSchedVmemRead, 1, 0);
        }
      }
    }
  }

  // Epilogue: accumulator register r of block (i, j) holds output row
  // m = m0 + kW*wm + 32*i + lane%32 and column
  // n = n0 + kW*wn + 32*j + 8*(r/4) + 4*(lane/32) + r%4.  When the problem
  // accumulates, the stored gradient is first widened and added in fp32 (one
  // rounding), then the sum is rounded to bf16 once.  The stored tile comes
  // through the LDS buffers, which are free once the loop is done.
  // Squares are summed along a lane's row of blocks i first, then over i; the
  // rows' sums wait in LDS past the tile (no register is free for them).
  float ss = 0.0f;
  const int m_lane = m0 + wm * kW + (lane & 31);
  const int n_lane = n0 + wn * kW + 4 * (lane >> 5);
  uint16_t* const tile = &lds[0][0][0];
  static_assert(kT * kT <= 2 * 2 * G::kStage, "the stored tile fits in the LDS buffers");
  // Rounds one group of four accumulator values (row m, columns n .. n+3)
  // and adds their squares to ss in a fixed order; returns them packed.
  auto round_group = [&](int i, int j, int g, int m, int n) {
    float v0 = acc[i][j][4 * g + 0], v1 = acc[i][j][4 * g + 1], v2 = acc[i][j][4 * g + 2],
          v3 = acc[i][j][4 * g + 3];
    if constexpr (kAcc) {
      const u32x2 old = *(const u32x2*)tile_at<kT>(tile, m - m0, n - n0);
      v0 += bf16_val(old.x & 0xFFFFu);
      v1 += bf16_val(old.x >> 16);
      v2 += bf16_val(old.y & 0xFFFFu);
      v3 += bf16_val(old.y >> 16);
    }
    const u32x2 p{pack_bf16(v0, v1), pack_bf16(v2, v3)};
    if constexpr (kT == 256) add_squares(p, ss);
    return p;
  };
  float* const row_sums = (float*)(tile + kT * kT);
  static_assert(kT != 256 || kT * kT * 2 + kB * kWgThreads * 4 <= 2 * 2 * G::kStage * 2, "LDS");
  auto end_row = [&](int i) {
    if constexpr (kT == 256) {
      row_sums[i * kWgThreads + int(threadIdx.x)] = ss;
      ss = 0.0f;
    }
  };
  __syncthreads();  // every wave is done with the operand buffers
  if constexpr (kAcc) {
    tile_to_lds<kT, 4>(tile, dw, m0, n0, M, N, tid);
    __syncthreads();
  }
  if ((!kAcc || kRows) && m0 + kT <= M && n0 + kT <= N) {
    // A tile wholly inside dw (uniform): the rounded tile goes
    // to the free LDS buffers first, in the swizzled layout of the stored
    // tile, then leaves in full rows: each wavefront store covers whole rows
    // (1 KiB of them), where a lane's own accumulator layout would touch 32
    // rows with 16 bytes each.  Accumulating, it goes where the stored values
    // were read.  (That spills eight registers in the 256 tile, so it is done
    // only where it pays.)
#pragma unroll
    for (int i = 0; i < kB; ++i) {
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        // one block at a time: its conversions and LDS accesses stay next
        // to their use, within the registers the accumulators leave free
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int m = m_lane + 32 * i, n = n_lane + 32 * j + 8 * g;
          *(u32x2*)tile_at<kT>(tile, m - m0, n - n0) = round_group(i, j, g, m, n);
        }
      }
      end_row(i);
    }
    __syncthreads();
    int row = lrow;
    uint16_t* out = dw + int64_t(m0 + row) * N + n0 + lcol;
#pragma unroll 4
    for (int p = 0; p < kT / kPass; ++p) {
      *(g_vec4*)out = *(const u32x4*)tile_at<kT>(tile, row, lcol);
      row += kPass;
      out += int64_t(kPass) * N;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const int m = m_lane + 32 * i;
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n = n_lane + 32 * j + 8 * g;
          if (m < M && n < N) *(g_vec2*)(dw + int64_t(m) * N + n) = round_group(i, j, g, m, n);
        }
      }
      end_row(i);
    }
  }
  if constexpr (kT == 256) {
    __shared__ float red[kWgThreads / 64];
    ss = row_sums[tid];
#pragma unroll
    for (int i = 1; i < kB; ++i) ss += row_sums[i * kWgThreads + tid];
    wave_sum_to(ss, red, tid);
    __syncthreads();
    if (tid == 0) P.tile_ss[tm * tiles_n + tn] = ((red[0] + red[1]) + red[2]) + red[3];
  }
}

constexpr int kSumsThreads = 1024;

// The tile sums of problems whose GEMM ran in smaller tiles: one workgroup per
// 256x256 tile reads the stored tile back (at most 128 KiB, just written).
// Sixteen waves, each with the part of one 256-tile wave that its row of
// blocks i makes, add the squares in that kernel's order, so a tile sum has
// the same bits on either path.
template <int kMost>
__global__ __launch_bounds__(kSumsThreads) void k5_tile_sums(const WgBatchOf<kMost> batch) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[256 * 256];
  __shared__ float part[4][256];  // [block row i][lane of the 256-tile kernel]
  __shared__ float red[kWgThreads / 64];
  int v = blockIdx.x;
  const WgProblem& P = batch.p[problem_of(batch, v)];
  const int M = P.M, N = P.N, m0 = v / P.tiles_n * 256, n0 = v % P.tiles_n * 256;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  tile_to_lds<256, kSumsThreads / 64>(tile, P.dw, m0, n0, M, N, tid);
  __syncthreads();
  const int i = wave >> 2, quarter = wave & 3;
  const int row = 128 * (quarter >> 1) + 32 * i + (lane & 31);
  const int col0 = 128 * (quarter & 1) + 4 * (lane >> 5);
  float ss = 0.0f;
#pragma unroll
  for (int jg = 0; jg < 16; ++jg) {
    const int col = col0 + 8 * jg;
    if (m0 + row < M && n0 + col < N) add_squares(*(const u32x2*)tile_at<256>(tile, row, col), ss);
  }
  part[i][64 * quarter + lane] = ss;
  __syncthreads();
  if (tid < kWgThreads)
    ss = ((part[0][tid] + part[1][tid]) + part[2][tid]) + part[3][tid];
  wave_sum_to(ss, red, tid);
  __syncthreads();
  if (tid == 0) P.tile_ss[v] = ((red[0] + red[1]) + red[2]) + red[3];
}

}  // namespace

int64_t wgrad_tiles(int32_t M, int32_t N) {
  return int64_t((M + kWgBM - 1) / kWgBM) * int64_t((N + kWgBN - 1) / kWgBN);
}

namespace {

// `batch`'s problems of one kind (accumulate == acc), cut into kT tiles.
template <int kT>
WgBatch tiled(const WgBatch& batch, int acc) {
  WgBatch b{};
  for (int32_t& t : b.tile_begin) t = INT32_MAX;
  for (int i = 0; i < batch.num; ++i) {
    if (batch.p[i].accumulate != acc) continue;
    WgProblem P = batch.p[i];
    P.tiles_m = (P.M + kT - 1) / kT;
    P.tiles_n = (P.N + kT - 1) / kT;
    b.tile_begin[b.num] = b.total_tiles;
    b.total_tiles += P.tiles_m * P.tiles_n;
    b.p[b.num++] = P;
  }
  return b;
}

// Whether accumulated tiles leave in full rows: where most of them have rows a
// multiple of 4,096 bytes apart.  There a wavefront's store of 16 bytes to each of
// 32 rows meets few memory channels: four 2048 x 2048 gradients, two 5504 x 2048
// and one 2048 x 5504 of 64 and 1,024 tokens take 95 and 159 us stored directly
// and 73 and 146 in rows, 4096 x 4096 of 64 and 4,096 tokens 24.2 and 121 against
// 21.4 and 119.  Other strides are as fast directly, or up to 4% faster.
bool rows_pay(const WgBatch& b) {
  int64_t strided = 0;
  for (int i = 0; i < b.num; ++i)
    if (b.p[i].N % 2048 == 0) strided += int64_t(b.p[i].tiles_m) * b.p[i].tiles_n;
  return 2 * strided > b.total_tiles;
}

template <int kT, bool kAcc, bool kRows, int kMost>
void launch_tiles(const WgBatchOf<kMost>& b, hipStream_t s) {
  hipLaunchKernelGGL((k5_wgrad<kAcc, kT, kRows, kMost>), dim3(unsigned(b.total_tiles)),
                     dim3(kWgThreads), 0, s, b);
}

template <int kT, int kMost>
void launch_tiled(const WgBatchOf<kMost>& b, bool acc, bool rows, hipStream_t s) {
  if (acc && rows) launch_tiles<kT, true, true>(b, s);
  else if (acc) launch_tiles<kT, true, false>(b, s);
  else launch_tiles<kT, false, false>(b, s);
}

WgBatchOf<1> single(const WgBatch& b) { return {1, b.total_tiles, {0}, {b.p[0]}}; }

template <int kT>
void launch_tiled(const WgBatch& batch, int acc, hipStream_t s) {
  const WgBatch b = tiled<kT>(batch, acc);
  const bool rows = acc && rows_pay(b);
  if (b.num == 1) launch_tiled<kT>(single(b), acc, rows, s);
  else launch_tiled<kT>(b, acc, rows, s);
}

template <int kMost>
void launch_sums(const WgBatchOf<kMost>& b, hipStream_t s) {
  hipLaunchKernelGGL(k5_tile_sums<kMost>, dim3(unsigned(b.total_tiles)), dim3(kSumsThreads), 0, s,
                     b);
}

// The tile edge for one launch.  A 256 tile does the most work per LDS byte
// and writes its own sum, but takes 6.4 us plus 1.0 us per K step of 64
// however few of the 256 CUs have one; the smaller tiles add the k5_tile_sums
// launch (about 5 us) and spread the same steps over 4 or 16 times the
// workgroups.  Measured on square problems, call to call, 256 / 128 / 64 tile, us
// (G: number of 256 tiles):
//   tokens      256              512              1024             2048             4096
//   G = 1       10.7  9.3  7.9   14.7 11.0  8.9   22.5 14.6 10.8   38.2 21.6 14.8   70  35  23
//   G = 16      11.1 10.3  8.6   15.1 12.1  9.7   22.9 15.6 11.7   38.7 22.6 16.0   71  37  26
//   G = 25      11.3 11.0 10.7   15.2 12.7 12.4   23.3 16.4 15.8   39.1 23.3 22.4   71  38  36
//   G = 36      11.4 11.9 12.3   15.4 13.8 14.7   23.4 17.5 19.8   39.5 24.1 28.1   71  39  47
//   G = 64      12.0 13.9 15.7   16.0 15.8 18.3   24.2 20.0 22.8   40.1 26.8 36.1   72  45  67
//   G = 81      12.3 16.7 18.2   16.4 19.8 21.4   24.5 24.0 28.8   40.4 37.1 48.0   72  64  86
//   G = 100     12.9 17.6 20.3   17.1 20.2 23.8   25.2 24.8 33.3   41.4 39.0 57.1   73  68 107
//   G = 121     13.1 19.2 21.5   17.3 21.2 25.8   25.5 26.3 37.1   41.2 41.8 61.8   74  73 116
//   G = 144     13.5 21.4 22.7   17.7 24.5 28.1   25.9 33.4 40.6   42.2 54.6 68.2   76  99 126
// and at 8,192 tokens G = 81: 139 / 120, G = 100: 138 / 126, G = 121: 151 / 141,
// G = 144: 145 / 186.  So: the 64 tile while every CU gets at most one and there are
// 4 steps to share, or at most two and 16 steps; the 128 tile while every CU gets at
// most one and the steps outweigh the second launch (4 plus one per 64 tiles more),
// or at most two and 32 steps; otherwise the 256 tile.  Two of the smaller tiles to a
// CU do not pay where the problems are no higher or wider than one: the larger tile
// then has as many, one to a CU.  64 x 32768 of 2,048, 4,096 and 8,192 tokens in 128
// and 64 tiles: 28.2 and 29.4, 46.6 and 52.4, 96 and 118 us; 128 x 38400 in 256 and 128
// tiles: 41.2 and 42.1, 90 and 98, 176 and 189.  (With a 256 tile on most CUs the chip's
// power evens that out: 128 x 65536 57.3 and 56.5, 111 and 116, accumulating 63.2 and
// 59.4, 119 and 120.)
int tile_edge(const WgBatch& batch, int acc) {
  int64_t n64 = 0, n128 = 0, n256 = 0, steps = 0;
  for (int i = 0; i < batch.num; ++i) {
    const WgProblem& p = batch.p[i];
    if (p.accumulate != acc) continue;
    const auto tiles = [&p](int t) { return int64_t((p.M + t - 1) / t) * ((p.N + t - 1) / t); };
    n64 += tiles(64);
    n128 += tiles(128);
    n256 += tiles(256);
    steps = std::max(steps, (p.K + kWgBK - 1) / kWgBK);
  }
  if (n64 <= 256 && steps >= 4) return 64;
  if (n64 <= 512 && steps >= 16 && n64 > 2 * n128) return 64;
  if (n128 <= 256 && steps >= 4 + n128 / 64) return 128;
  if (n128 <= 512 && steps >= 32 && (n128 > 2 * n256 || n256 > 192)) return 128;
  return 256;
}

}  // namespace

hipError_t launch_wgrad(const WgBatch& batch, hipStream_t s) {
  // one launch per epilogue kind: the problems that overwrite dw, then those
  // that accumulate into it, each launch with its own tile order
  for (const int acc : {0, 1}) {
    const WgBatch b = tiled<256>(batch, acc);
    if (b.total_tiles == 0) continue;
    const int t = tile_edge(batch, acc);
    if (t == 256) {
      launch_tiled<256>(batch, acc, s);
    } else {
      if (t == 128) launch_tiled<128>(batch, acc, s);
      else launch_tiled<64>(batch, acc, s);
      if (b.num == 1) launch_sums(single(b), s);
      else launch_sums(b, s);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace gnmr
