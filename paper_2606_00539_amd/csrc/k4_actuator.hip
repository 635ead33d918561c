// K4, the recovery actuator for CDNA4 (gfx950): per-token fake quantisation
// of saved activations, the format chosen per unit by the controller's mask
// (App. E.2 quantisation-simulated operators: each token is scaled into the
// format's representable range, rounded to the nearest representable value
// and rescaled; Sec. 5.1 / App. E.4: token-wise low-bit saved activations;
// Sec. 5.3 / App. E.3: the INT8 low-cost path).
//
// A token row is held in the registers of part of a wavefront (up to 512
// features), a wavefront (up to 3,072) or a workgroup of 256 or 512 lanes (up
// to 16,384): amax by a max-reduction, one fp32 division each for the scale and
// its reciprocal, then per element y = x * inv, round to the format (ties to
// the even significand, saturating), out = bf16_rne(q * s).  A row whose unit
// takes the BF16 path in place is left untouched without reading it.  The rows
// come from a table built once over many segments (k4_actuate), or from one
// matrix passed by value (k4_matrix, no table).
//
// Bound by memory: every byte is read and written once.  The lanes per row and
// the vectors per lane (for_class) keep few registers idle, so that enough rows
// are in flight per CU; rows are dealt to the eight XCDs in contiguous runs.
// Stores are non-temporal.  So are the loads of large sets; up to kK4CachedBytes
// of input the loads are ordinary ones, since such an input was often written
// just before and is in the memory-side cache (256 MB), which ordinary loads
// leave it in.  Measured (read + write; before: one wavefront per row up to
// 4,096 features and a workgroup above, room for 8 vectors per lane always,
// non-temporal loads; copy: a plain copy with non-temporal loads and stores):
//   4096 x 5120    14.8 us (5.7 TB/s)   before 19.5   copy 16.2
//   4096 x 4096    12.4 us              before 14.1   copy 13.3
//   2048 x 11008   15.8 us              before 21.1   copy 17.2
//   4096 x 1024     4.6 us              before  6.0   copy  5.0
//   16384 x 4096   51.3 us (5.2 TB/s)   before 54.9   copy 50.3   (non-temporal)
#include <algorithm>

#include "gnmr_internal.h"
#include "lane_ops.h"

namespace gnmr {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 g_cvec;
typedef __attribute__((address_space(1))) u32x4 g_vec;

struct Format {
  int mbits;    // significand bits
  int emin;     // exponent of the smallest normal binade
  float fmax;   // largest finite value
};

// E2M1, E3M2, E4M3 (OCP, 448 max), E5M2 (57344 max); no inf/NaN produced.
// The symmetric INT8 grid {0, 1, ..., 127} is the same rounding with the
// lowest binade at 2^6 and 6 fraction bits: a step of 1 below 128 and
// saturation at 127.
__device__ __forceinline__ Format format_of(int fmt) {
  switch (fmt) {
    case GNMR_FMT_INT8: return Format{6, 6, 127.0f};
    case GNMR_FMT_E2M1: return Format{1, 0, 6.0f};
    case GNMR_FMT_E3M2: return Format{2, -2, 28.0f};
    case GNMR_FMT_E4M3: return Format{3, -6, 448.0f};
    default: return Format{2, -14, 57344.0f};  // GNMR_FMT_E5M2
  }
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two fp32 values to packed bf16, round to nearest even (one
// v_cvt_pk_bf16_f32; the values here are finite).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// Nearest representable value of the format to y, ties to the even
// significand, saturating at fmax.  All steps but rintf are exact.
__device__ __forceinline__ float round_to_format(float y, const Format& f) {
  const float a = fabsf(y);
  int e = int((__float_as_uint(a) >> 23) & 0xFFu) - 127;  // binade of a (any e < emin clamps)
  e = e < f.emin ? f.emin : e;
  const float step = __uint_as_float(uint32_t(e - f.mbits + 127) << 23);
  const float inv_step = __uint_as_float(uint32_t(f.mbits - e + 127) << 23);
  float q = __fmul_rn(rintf(__fmul_rn(a, inv_step)), step);
  q = q < f.fmax ? q : f.fmax;
  return copysignf(q, y);
}

__device__ __forceinline__ uint32_t quant_pair(uint32_t w, float inv, float s, const Format& f) {
  const float lo = __fmul_rn(round_to_format(__fmul_rn(bf16_lo(w), inv), f), s);
  const float hi = __fmul_rn(round_to_format(__fmul_rn(bf16_hi(w), inv), f), s);
  return pack_bf16(lo, hi);
}

__device__ __forceinline__ float max_abs_pair(uint32_t w, float m) {
  return fmaxf(m, fmaxf(fabsf(bf16_lo(w)), fabsf(bf16_hi(w))));
}

__device__ __forceinline__ void store(g_vec* p, const u32x4& v) {
  __builtin_nontemporal_store(v, p);
}

template <bool kCached>
__device__ __forceinline__ u32x4 load(const g_cvec* p) {
  if constexpr (kCached) return *p;
  else return __builtin_nontemporal_load(p);
}

// Row `row` of segment sg (none when !valid) by LANES lanes of kVpt vectors
// each; kUniform: a wavefront's rows are of one unit.  Every lane of the workgroup
// calls it, and a row of more than 64 lanes has the workgroup to itself; `red` is
// then LDS of LANES / 64 floats.
template <int LANES, int kVpt, bool kCached, bool kUniform>
__device__ __forceinline__ void actuate_row(const ActSeg sg, int64_t row, bool valid,
                                            const uint8_t* __restrict__ mask, int fmt_low,
                                            int fmt_rec, int lane, float* red) {
  const int64_t row_off = row * sg.cols * 2;
  const g_cvec* in = (const g_cvec*)(sg.in + row_off);
  g_vec* out = (g_vec*)(sg.out + row_off);
  int nvec = valid ? sg.cols >> 3 : 0;
  // The unit's mask entry is on its way while the row is read; only where the
  // BF16 path in place may leave the row unread is it waited for first.  The
  // zero offset is opaque: the compiler would move a wave-uniform entry to a
  // scalar register, and wait for it, at once.
  const uint8_t* const entry = mask + sg.unit + __builtin_amdgcn_mbcnt_lo(0u, 0u);
  const uint8_t on = *entry;
  if (sg.in == sg.out && (fmt_low == GNMR_FMT_BF16 || fmt_rec == GNMR_FMT_BF16) &&
      (on ? fmt_rec : fmt_low) == GNMR_FMT_BF16)
    nvec = 0;

  u32x4 v[kVpt];
#pragma unroll
  for (int k = 0; k < kVpt; ++k) {
    const int i = lane + k * LANES;
    v[k] = i < nvec ? load<kCached>(in + i) : u32x4{0u, 0u, 0u, 0u};
  }
  __builtin_amdgcn_sched_barrier(0);
  int fmt = on ? fmt_rec : fmt_low;
  if constexpr (kUniform) fmt = __builtin_amdgcn_readfirstlane(fmt);
  if (fmt == GNMR_FMT_BF16) {  // BF16 path out of place: a copy
#pragma unroll
    for (int k = 0; k < kVpt; ++k) {
      const int i = lane + k * LANES;
      if (i < nvec) store(out + i, v[k]);
    }
    nvec = 0;
  }

  // amax over the row (max is exact, so the reduction order is immaterial)
  float m = 0.0f;
#pragma unroll
  for (int k = 0; k < kVpt; ++k) {
    m = max_abs_pair(v[k].x, m);
    m = max_abs_pair(v[k].y, m);
    m = max_abs_pair(v[k].z, m);
    m = max_abs_pair(v[k].w, m);
  }
  m = lanes_max<(LANES > 64 ? 64 : LANES)>(m);
  float amax = m;
  if constexpr (LANES > 64) {
    if ((lane & 63) == 0) red[lane >> 6] = m;
    __syncthreads();
    amax = red[0];
#pragma unroll
    for (int w = 1; w < LANES / 64; ++w) amax = fmaxf(amax, red[w]);
  }

  const Format f = format_of(fmt);
  if (amax == 0.0f) {  // an all-zero token stays zero
#pragma unroll
    for (int k = 0; k < kVpt; ++k) {
      const int i = lane + k * LANES;
      if (i < nvec) store(out + i, u32x4{0u, 0u, 0u, 0u});
    }
    return;
  }
  const float inv = __fdiv_rn(f.fmax, amax);  // scale into the format's range
  const float s = __fdiv_rn(amax, f.fmax);    // and back
#pragma unroll
  for (int k = 0; k < kVpt; ++k) {
    const int i = lane + k * LANES;
    if (i < nvec) {
      u32x4 o;
      o.x = quant_pair(v[k].x, inv, s, f);
      o.y = quant_pair(v[k].y, inv, s, f);
      o.z = quant_pair(v[k].z, inv, s, f);
      o.w = quant_pair(v[k].w, inv, s, f);
      store(out + i, o);
    }
  }
}

// Workgroup w runs on XCD w % 8: give each XCD a contiguous run of [0, n).
__device__ __forceinline__ uint32_t xcd_order(uint32_t w, uint32_t n) {
  const uint32_t x = w % kNumXcd, j = w / kNumXcd, q = n / kNumXcd, r = n % kNumXcd;
  return x * q + (x < r ? x : r) + j;
}

// Workgroups of 256 lanes, or of one row where that takes more.
constexpr int block_of(int lanes) { return lanes > kK4Block ? lanes : kK4Block; }

// Waves per SIMD: eight (64 VGPRs) while a lane holds few vectors, six where it
// holds four or more in a wide row or six: more rows in flight per CU than that
// cost bandwidth (6103 x 8192: 37.4 us with six, 40.5 with eight; 4066 x 12296:
// 37.6 and 39.3; but 42207 x 3080, two per lane: 105 and 92).
#define GNMR_K4_KERNEL                                         \
  __global__ __launch_bounds__(block_of(LANES)) __attribute__( \
      (amdgpu_waves_per_eu(waves_of(LANES, kVpt), waves_of(LANES, kVpt))))
constexpr int waves_of(int lanes, int vpt) { return vpt >= 6 || (vpt >= 4 && lanes > 64) ? 6 : 8; }

// Rows [0, num_rows) of the table.
template <int LANES, int kVpt, bool kCached>
GNMR_K4_KERNEL void k4_actuate(const RowItem* __restrict__ items, uint32_t num_rows,
                               const ActSeg* __restrict__ segs,
                               const uint8_t* __restrict__ mask, int fmt_low, int fmt_rec) {
  constexpr int kRows = block_of(LANES) / LANES;  // per workgroup
  __shared__ float red[block_of(LANES) / 64];
  const uint32_t sub = kRows > 1 ? threadIdx.x / LANES : 0;
  const uint32_t r = xcd_order(blockIdx.x, gridDim.x) * kRows + sub;
  const bool valid = r < num_rows;
  const RowItem it = items[valid ? r : num_rows - 1];
  const ActSeg sg = segs[it.seg];
  __builtin_amdgcn_sched_barrier(0);  // the whole entry at once, not the pointers after the mask
  actuate_row<LANES, kVpt, kCached, LANES >= 64>(sg, it.row, valid, mask, fmt_low, fmt_rec,
                                                 int(threadIdx.x) % LANES, red);
}

// One matrix without a row table (the segment passed by value).
template <int LANES, int kVpt, bool kCached>
GNMR_K4_KERNEL void k4_matrix(const ActSeg sg, uint32_t num_rows,
                              const uint8_t* __restrict__ mask, int fmt_low, int fmt_rec) {
  constexpr int kRows = block_of(LANES) / LANES;
  __shared__ float red[block_of(LANES) / 64];
  const uint32_t sub = kRows > 1 ? threadIdx.x / LANES : 0;
  const uint32_t r = xcd_order(blockIdx.x, gridDim.x) * kRows + sub;
  actuate_row<LANES, kVpt, kCached, true>(sg, r, r < num_rows, mask, fmt_low, fmt_rec,
                                          int(threadIdx.x) % LANES, red);
}

// Calls f.template operator()<LANES, kVpt>() for a row class.  The lanes and
// vectors are the fewest that hold its widest row; where several do, the split
// that was the fastest or within 3% of it over 512 to 16,384 rows, from the
// table and as a matrix (us, with its rival):
//   2048 features, 4,096 rows: 64 x 4  7.9   (128 x 2 7.5, but 11% slower than
//                                             64 x 4 from the table at 260 MB)
//   3072, 4,096 rows:          64 x 6 10.2   (128 x 3 9.5, the same)
//   4096, 2,048 rows:         256 x 2  7.5   (128 x 4 8.3, 64 x 8 8.6)
//   6144, 1,024 rows:         256 x 3  6.4   (128 x 6 7.0)
//  11008,   512 rows:         512 x 3  6.0   (256 x 6 6.4; 2,048 rows: 16.1, 15.8)
//  16384, 1,024 rows:         512 x 4 13.1   (256 x 8 14.1)
struct RowClass {
  int lanes, vpt;
};
constexpr RowClass kClasses[kK4Classes] = {{8, 2},   {16, 2},  {32, 2},  {64, 2},
                                           {64, 3},  {64, 4},  {64, 6},  {256, 2},
                                           {256, 3}, {256, 4}, {512, 3}, {512, 4}};
static_assert(kClasses[kK4Classes - 1].lanes * kClasses[kK4Classes - 1].vpt * 8 == kK4MaxCols, "");

template <int kClass = 0, typename F>
void for_class(int cls, const F& f) {
  if (cls == kClass) f.template operator()<kClasses[kClass].lanes, kClasses[kClass].vpt>();
  else if constexpr (kClass + 1 < kK4Classes) for_class<kClass + 1>(cls, f);
}

// Rows of several classes in one launch of workgroups of kK4Block lanes:
// workgroups [block[c], block[c + 1]) take rows [row[c], row[c + 1]) of the table.
struct MixedRows {
  uint32_t block[kK4Classes + 1], row[kK4Classes + 1];
};

constexpr RowClass mixed_class(int c) {
  return kClasses[c].lanes <= kK4Block
             ? kClasses[c]
             : RowClass{kK4Block, kClasses[c].vpt * (kClasses[c].lanes / kK4Block)};
}

template <bool kCached, int kClass = 0>
__device__ __forceinline__ void mixed_row(int cls, uint32_t w, const MixedRows& rows,
                                          const RowItem* items, const ActSeg* segs,
                                          const uint8_t* mask, int fmt_low, int fmt_rec,
                                          float* red) {
  if (cls == kClass) {
    constexpr int kLanes = mixed_class(kClass).lanes;
    const uint32_t sub = kLanes < kK4Block ? threadIdx.x / kLanes : 0;
    // (each class over all XCDs: its workgroups have less or more to do than others)
    const uint32_t at =
        xcd_order(w - rows.block[kClass], rows.block[kClass + 1] - rows.block[kClass]);
    const uint32_t r = rows.row[kClass] + at * (kK4Block / kLanes) + sub;
    const bool valid = r < rows.row[kClass + 1];
    const RowItem it = items[valid ? r : rows.row[kClass + 1] - 1];
    const ActSeg sg = segs[it.seg];
    __builtin_amdgcn_sched_barrier(0);
    actuate_row<kLanes, mixed_class(kClass).vpt, kCached, kLanes >= 64>(
        sg, it.row, valid, mask, fmt_low, fmt_rec, int(threadIdx.x) % kLanes, red);
  } else if constexpr (kClass + 1 < kK4Classes) {
    mixed_row<kCached, kClass + 1>(cls, w, rows, items, segs, mask, fmt_low, fmt_rec, red);
  }
}

template <bool kCached>
__global__ __launch_bounds__(kK4Block) __attribute__((amdgpu_waves_per_eu(6, 6))) void k4_mixed(
    const RowItem* __restrict__ items, const MixedRows rows, const ActSeg* __restrict__ segs,
    const uint8_t* __restrict__ mask, int fmt_low, int fmt_rec) {
  __shared__ float red[kK4Block / 64];
  const uint32_t w = blockIdx.x;
  int cls = 0;
#pragma unroll
  for (int c = 1; c < kK4Classes; ++c) cls = w >= rows.block[c] ? c : cls;
  mixed_row<kCached>(cls, w, rows, items, segs, mask, fmt_low, fmt_rec, red);
}

struct TableLaunch {
  const RowItem* items;
  int64_t rows;
  const ActSeg* segs;
  const uint8_t* mask;
  int fmt_low, fmt_rec;
  bool cached;
  hipStream_t s;
  template <int LANES, int kVpt>
  void operator()() const {
    constexpr int kBlock = block_of(LANES);
    constexpr int64_t kRows = kBlock / LANES, kMost = kRows * (int64_t(UINT32_MAX) / kBlock);
    // a grid holds fewer than 2^32 lanes
    for (int64_t r = 0; r < rows; r += kMost) {
      const int64_t n = std::min(rows - r, kMost);
      const dim3 grid(unsigned((n + kRows - 1) / kRows));
      if (cached)
        hipLaunchKernelGGL((k4_actuate<LANES, kVpt, true>), grid, dim3(kBlock), 0, s, items + r,
                           uint32_t(n), segs, mask, fmt_low, fmt_rec);
      else
        hipLaunchKernelGGL((k4_actuate<LANES, kVpt, false>), grid, dim3(kBlock), 0, s, items + r,
                           uint32_t(n), segs, mask, fmt_low, fmt_rec);
    }
  }
};

struct MatrixLaunch {
  ActSeg sg;
  int64_t rows;
  const uint8_t* mask;
  int fmt_low, fmt_rec;
  bool cached;
  hipStream_t s;
  template <int LANES, int kVpt>
  void operator()() const {
    constexpr int kBlock = block_of(LANES);
    constexpr int64_t kRows = kBlock / LANES, kMost = kRows * (int64_t(UINT32_MAX) / kBlock);
    for (int64_t r = 0; r < rows; r += kMost) {
      const int64_t n = std::min(rows - r, kMost);
      const dim3 grid(unsigned((n + kRows - 1) / kRows));
      ActSeg part = sg;
      part.in += r * sg.cols * 2;
      part.out += r * sg.cols * 2;
      if (cached)
        hipLaunchKernelGGL((k4_matrix<LANES, kVpt, true>), grid, dim3(kBlock), 0, s, part,
                           uint32_t(n), mask, fmt_low, fmt_rec);
      else
        hipLaunchKernelGGL((k4_matrix<LANES, kVpt, false>), grid, dim3(kBlock), 0, s, part,
                           uint32_t(n), mask, fmt_low, fmt_rec);
    }
  }
};

}  // namespace

int k4_class(int cols) {
  int c = 0;
  while (cols > kClasses[c].lanes * kClasses[c].vpt * 8) ++c;  // cols <= kK4MaxCols
  return c;
}

namespace {

// Whether all classes of a table take one launch, which the longest row's registers
// then limit to six waves per SIMD, or a launch each, each with a start and a tail
// of its own.  With cached loads one launch: the inputs of layers' projections, two
// widths, a launch each and one, 7.4 and 4.7 us (5120 and 13824 features, 0.9 MB),
// 8.3 and 5.6 (3.9 MB), 24.3 and 21.6 (63 MB), twelve widths 41 and 4.9 (0.9 MB),
// 62 and 24.6 (63 MB).  (A workgroup of 256 lanes with eight vectors each for every
// row: 5.0, 5.6 and 28.0 of the first three.)  Past that, rows of two vectors a lane,
// or three in a wavefront, want eight waves and lose about 0.03 to 0.05 us a MB, against
// 2 us for each further launch.  With none of them one launch: 2048 and 5504 at 100 MB
// 38.7 and 36.2, 12288 and 16384 at 68 MB 29.5 and 26.7.  With many a launch each: 1064
// and 3104 at 250 MB 101 and 108, 1112 and 3032 at 94 MB 42.0 and 43.6 (64 MB of them).
// Twelve widths, half of them such: 73.8 and 41.8 at 100 MB, 186 and 149 at 400.  A
// large table's launches are long beside what they cost: 4096 and 11008 at 500 MB 162
// and 165, 1 GB 322 and 323.
constexpr int64_t kMixedBytes = int64_t(384) << 20, kMixedFew = int64_t(32) << 20;
bool one_launch(const int64_t* class_off, int64_t bytes) {
  int present = 0;
  int64_t few = 0;  // at most these bytes are of rows that want eight waves
  for (int c = 0; c < kK4Classes; ++c) {
    const int64_t rows = class_off[c + 1] - class_off[c];
    const int lanes = kClasses[c].lanes, vpt = kClasses[c].vpt;
    present += rows > 0 ? 1 : 0;
    if (vpt == 2 || (vpt == 3 && lanes == 64)) few += rows * lanes * vpt * 16;
  }
  if (present < 2 || bytes > kMixedBytes) return false;
  return bytes <= kK4CachedBytes || few <= kMixedFew * (present - 1);
}

template <bool kCached>
void launch_mixed(const RowItem* items, const int64_t* class_off, const ActSeg* segs,
                  const uint8_t* mask, int fmt_low, int fmt_rec, hipStream_t s) {
  MixedRows m{};
  uint32_t blocks = 0;
  for (int c = 0; c <= kK4Classes; ++c) {
    m.block[c] = blocks;
    m.row[c] = uint32_t(class_off[c]);
    if (c == kK4Classes) break;
    const int64_t per = kK4Block / mixed_class(c).lanes;
    blocks += uint32_t((class_off[c + 1] - class_off[c] + per - 1) / per);
  }
  hipLaunchKernelGGL(k4_mixed<kCached>, dim3(blocks), dim3(kK4Block), 0, s, items, m, segs, mask,
                     fmt_low, fmt_rec);
}

}  // namespace

hipError_t launch_actuate(const RowItem* items, const int64_t* class_off, int64_t bytes,
                          const ActSeg* segs, const uint8_t* mask, int fmt_low, int fmt_rec,
                          hipStream_t s) {
  const bool cached = bytes <= kK4CachedBytes;
  if (one_launch(class_off, bytes)) {
    if (cached) launch_mixed<true>(items, class_off, segs, mask, fmt_low, fmt_rec, s);
    else launch_mixed<false>(items, class_off, segs, mask, fmt_low, fmt_rec, s);
    return hipGetLastError();
  }
  for (int c = 0; c < kK4Classes; ++c)
    if (class_off[c + 1] > class_off[c])
      for_class(c, TableLaunch{items + class_off[c], class_off[c + 1] - class_off[c], segs, mask,
                               fmt_low, fmt_rec, cached, s});
  return hipGetLastError();
}

hipError_t launch_actuate_matrix(const ActSeg& sg, int64_t rows, const uint8_t* mask,
                                 int fmt_low, int fmt_rec, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  for_class(k4_class(sg.cols), MatrixLaunch{sg, rows, mask, fmt_low, fmt_rec,
                                            rows * sg.cols * 2 <= kK4CachedBytes, s});
  return hipGetLastError();
}

}  // namespace gnmr
