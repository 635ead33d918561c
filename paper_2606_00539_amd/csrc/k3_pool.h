// The walk of K3's workgroup over the places that K2's workgroups may fill.
#pragma once

#include <stdint.h>

namespace gnmr {

// Places of num_wgs K2 workgroups of 1 << shift units each.  2^31 - 1 units are
// 2^23 workgroups of 256: 2^31 places, one more than an int32 holds.
constexpr uint32_t pool_places(int32_t num_wgs, int32_t shift) {
  return uint32_t(num_wgs) << shift;
}

// Rounds of `block` places each.  (A loop over the places themselves would have to
// pass the last of them to end.)
constexpr uint32_t pool_rounds(uint32_t places, uint32_t block) {
  return places / block + (places % block != 0 ? 1 : 0);
}

}  // namespace gnmr
