// Butterflies over the lanes of a wavefront without LDS: swaps of half and
// quarter waves, rotations inside rows of 16 lanes and permutations inside quads
// cost a few cycles each, where a lane permute through LDS (what __shfl_xor
// becomes) takes about 100.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace gnmr {

// op(x of this lane, x of lane ^ kMask) for a symmetric op, kMask 32, 16, 8, 4,
// 2 or 1.  Mask 4 rotates by four in a row of 16, which is lane ^ 4 once lanes 8
// apart hold the same: after mask 8, as in the butterflies below.
template <int kMask, typename Op>
__device__ __forceinline__ uint32_t with_other(uint32_t x, Op op) {
  if constexpr (kMask == 32) {
    // both halves get (lower half, upper half)
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return op(r[0], r[1]);
  } else if constexpr (kMask == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return op(r[0], r[1]);
  } else {
    constexpr int kCtrl = kMask == 8 ? 0x128 : kMask == 4 ? 0x124 : kMask == 2 ? 0x4E : 0xB1;
    return op(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), kCtrl, 0xF, 0xF, false)));
  }
}

template <int kMask>
__device__ __forceinline__ float add_other(float v) {
  return __uint_as_float(with_other<kMask>(__float_as_uint(v), [](uint32_t a, uint32_t b) {
    return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
  }));
}

template <int kMask>
__device__ __forceinline__ double add_other(double v) {
  // the halves of the two operands; either order gives the same sum
  const uint64_t x = __builtin_bit_cast(uint64_t, v);
  uint32_t lo[2], hi[2];
  with_other<kMask>(uint32_t(x), [&](uint32_t a, uint32_t b) {
    lo[0] = a;
    lo[1] = b;
    return 0u;
  });
  with_other<kMask>(uint32_t(x >> 32), [&](uint32_t a, uint32_t b) {
    hi[0] = a;
    hi[1] = b;
    return 0u;
  });
  return __builtin_bit_cast(double, uint64_t(hi[0]) << 32 | lo[0]) +
         __builtin_bit_cast(double, uint64_t(hi[1]) << 32 | lo[1]);
}

// The sum over the 64 lanes, pairs 32 apart first; every lane ends with it.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  v = add_other<32>(v);
  v = add_other<16>(v);
  v = add_other<8>(v);
  v = add_other<4>(v);
  v = add_other<2>(v);
  return add_other<1>(v);
}

// The largest of every LANES consecutive lanes' values (8, 16, 32 or 64), in
// each of them.
template <int LANES>
__device__ __forceinline__ float lanes_max(float v) {
  const auto larger = [](uint32_t a, uint32_t b) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  };
  uint32_t x = __float_as_uint(v);
  if constexpr (LANES >= 64) x = with_other<32>(x, larger);
  if constexpr (LANES >= 32) x = with_other<16>(x, larger);
  if constexpr (LANES >= 16) {
    x = with_other<8>(x, larger);
    x = with_other<4>(x, larger);
  } else {
    // eight lanes, mirrored: the quads then hold the same four values
    x = larger(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x141, 0xF, 0xF, false)));
  }
  x = with_other<2>(x, larger);
  x = with_other<1>(x, larger);
  return __uint_as_float(x);
}

// Scans and reductions of 32-bit values over a wavefront by data-parallel
// primitives: four shifts inside the rows of 16 lanes, then the rows' last
// lanes passed on (about 50 cycles, where six dependent lane permutes through
// LDS take several hundred).
template <typename Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t identity, Op op) {
  auto step = [&](auto ctrl, auto rows) {
    x = op(x, uint32_t(__builtin_amdgcn_update_dpp(int(identity), int(x), decltype(ctrl)::value,
                                                   decltype(rows)::value, 0xF, false)));
  };
  constexpr int kShr = 0x110, kBcast15 = 0x142, kBcast31 = 0x143;
  using std::integral_constant;
  step(integral_constant<int, kShr + 1>{}, integral_constant<int, 0xF>{});
  step(integral_constant<int, kShr + 2>{}, integral_constant<int, 0xF>{});
  step(integral_constant<int, kShr + 4>{}, integral_constant<int, 0xF>{});
  step(integral_constant<int, kShr + 8>{}, integral_constant<int, 0xF>{});
  step(integral_constant<int, kBcast15>{}, integral_constant<int, 0xA>{});
  step(integral_constant<int, kBcast31>{}, integral_constant<int, 0xC>{});
  return x;
}

// Inclusive prefix sum over the lanes; the last lane holds the total.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x) {
  return wave_scan(x, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}

// The same inside each row of 16 lanes.
template <typename Op>
__device__ __forceinline__ uint32_t row_scan(uint32_t x, uint32_t identity, Op op) {
  auto step = [&](auto ctrl) {
    x = op(x, uint32_t(__builtin_amdgcn_update_dpp(int(identity), int(x), decltype(ctrl)::value,
                                                   0xF, 0xF, false)));
  };
  step(std::integral_constant<int, 0x111>{});
  step(std::integral_constant<int, 0x112>{});
  step(std::integral_constant<int, 0x114>{});
  step(std::integral_constant<int, 0x118>{});
  return x;
}

__device__ __forceinline__ uint32_t row_prefix(uint32_t x) {
  return row_scan(x, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}

__device__ __forceinline__ uint32_t lane_of(uint32_t x, int lane) {
  return uint32_t(__builtin_amdgcn_readlane(int(x), lane));
}

}  // namespace gnmr
