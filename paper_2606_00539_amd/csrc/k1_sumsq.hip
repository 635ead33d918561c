// K1 of the GNMR controller pass for CDNA4 (gfx950): the sum of squares of
// every gradient element, one fp32 partial per 64 KiB work item (Sec. 2,
// local-gradient equation: n = ||g||_2 over all of a unit's parameters).
//
// Deterministic: fixed work items, a fixed reduction tree, no floating-point
// atomics; the result does not depend on the grid or on scheduling.
#include <string.h>

#include "gnmr_internal.h"
#include "k1_item.h"

namespace gnmr {
namespace {

template <typename Bases>
__global__ __launch_bounds__(kK1Block) void k1_sumsq(const Item* __restrict__ items,
                                                     uint32_t num_items, const Bases seg_base,
                                                     const int32_t* __restrict__ seg_dtype,
                                                     float* __restrict__ partial) {
  const uint32_t item = xcd_item(blockIdx.x, num_items);
  const Item it = items[item];
  if (blockIdx.x == 0) seg_base.keep();
  __shared__ float red[kK1Block / 64];
  const float s = item_sumsq(it, seg_base.of(it.seg), seg_dtype[it.seg], red);
  if (threadIdx.x == 0) partial[item] = s;
}

}  // namespace

namespace {

template <int kMost>
void launch_passed(const Item* items, int64_t num_items, const char** table,
                   const void* const* ptrs, int64_t num_segs, const int32_t* seg_dtype,
                   float* partial, hipStream_t s) {
  PassedBases<kMost> b;
  b.table = table;
  b.num = int32_t(num_segs);
  memcpy(b.base, ptrs, size_t(num_segs) * sizeof(void*));
  hipLaunchKernelGGL(k1_sumsq<PassedBases<kMost>>, dim3(unsigned(num_items)), dim3(kK1Block), 0, s,
                     items, uint32_t(num_items), b, seg_dtype, partial);
}

}  // namespace

hipError_t launch_sumsq(const Item* items, int64_t num_items, const char** seg_base,
                        const void* const* ptrs, int64_t num_segs, const int32_t* seg_dtype,
                        float* partial, hipStream_t s) {
  if (num_items <= 0) return hipSuccess;
  if (ptrs == nullptr)
    hipLaunchKernelGGL(k1_sumsq<TableBases>, dim3(unsigned(num_items)), dim3(kK1Block), 0, s, items,
                       uint32_t(num_items), TableBases{seg_base}, seg_dtype, partial);
  else if (num_segs <= kK1FewPassed)
    launch_passed<kK1FewPassed>(items, num_items, seg_base, ptrs, num_segs, seg_dtype, partial, s);
  else
    launch_passed<kK1MostPassed>(items, num_items, seg_base, ptrs, num_segs, seg_dtype, partial, s);
  return hipGetLastError();
}

}  // namespace gnmr
