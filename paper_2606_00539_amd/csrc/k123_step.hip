// A small workload's whole step in one launch for CDNA4 (gfx950): K1's work items
// and, in workgroup 0, K2 and K3 over them.
//
// Two launches of a few microseconds each spend most of their time before and
// after their work: the second waits for the first to drain, starts, loads the
// state of the units and fetches its instructions.  Here workgroup 0 does all of
// that while the others read gradients.
//
// How the partials arrive without a fence: a device-scope release writes back an
// XCD's whole L2 (a version with a ticket and fences took 12 us where two
// launches took 8).  Instead each item's partial and a tag travel in one 64-bit
// word, written and read by relaxed device-scope atomics, so that the word is its
// own notice.  The tag is the number of the launch, kept on the device (a captured
// launch replays with the next one), so a word of an earlier launch is never taken
// for one of this.  Only workgroup 0 waits, and only for workgroups that wait for
// nothing; they find room beside it, since it fills a fraction of one CU.
//
// The same partials, orders and arithmetic as K1, K2 and K3: the same results.
#include <string.h>

#include <algorithm>

#include "gnmr_internal.h"
#include "k1_item.h"
#include "launch_tag.h"
#include "unit_step.h"

namespace gnmr {
namespace {

constexpr int kStepUnits = kK1Block;  // one thread per unit

// About a microsecond each: minutes, against a step's microseconds.  A workload
// whose items do not arrive by then ends with NaN norms, not in a hang; so do its
// later steps, whose words could not be told from those still to come.
constexpr uint32_t kPolls = 1u << 28;

// The last items by workgroup number, collected after everything else has been
// done for the units whose items all came before them: about what is in flight
// when the last workgroup starts.  84 units in 6,048 items: 62.9 us a step; 512:
// 64.9, 256: 65.7, 2,048: 62.9.
constexpr uint32_t kLate = 1024;

struct StepShared {
  uint64_t counts[kK1Block / 64];
  uint64_t key[kStepUnits];
  double ss[kStepUnits];
  int32_t off[kStepUnits + 1];
  int32_t unit[kStepUnits];   // units with late items first
  int32_t late[kK1Block / 64];
  int32_t lost[kK1Block / 64];  // whether a word of the wave's has not arrived
};

// Waits for the words of workgroups [from, to); the partials go to part[item].
__device__ __forceinline__ void collect(const uint64_t* words, uint32_t num, uint32_t from,
                                        uint32_t to, uint32_t tag, float* part, int32_t* lost) {
  constexpr int kAtOnce = 4;  // words in flight per lane
  const uint32_t most = words_lost(tag) ? 1 : kPolls;
  for (uint32_t first = from + threadIdx.x; first < to; first += kAtOnce * kK1Block) {
    uint64_t v[kAtOnce];
    uint32_t polls = 0;
#pragma unroll 1
    for (; polls < most; ++polls) {
      bool all = true;
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        const uint32_t w = first + k * kK1Block;
        v[k] = __hip_atomic_load(words + (w < to ? w : first), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) all = all && uint32_t(v[k] >> 32) == tag;
      if (all) break;
      __builtin_amdgcn_s_sleep(1);
    }
    if (polls == most) *lost = 1;
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) {
      const uint32_t w = first + k * kK1Block;
      const bool here = uint32_t(v[k] >> 32) == tag;
      if (w < to) part[xcd_item(w, num)] = here ? __uint_as_float(uint32_t(v[k])) : NAN;
    }
  }
}

// sh.ss of the n units listed, with the sums of lane_ss<L> and the cross-lane
// orders of k2_update<L>.  A wavefront takes four units (L = 64) or the four
// quarters of one (L = 256) at a time, without branches, so that their loads and
// butterflies overlap.
template <int L>
__device__ __forceinline__ void sum_units(const float* part, const int32_t* unit, int n,
                                          StepShared& sh) {
  constexpr int kUnits = L == 64 ? 4 : 1;
  const int l = int(threadIdx.x) & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  for (int first = kUnits * wave; first < n; first += kUnits * (kK1Block / 64)) {
    int i[4], hi[4], longest = 0;
    double s[4][4] = {};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int at = L == 64 ? first + k : first;
      const int x = unit[at < n ? at : first];
      i[k] = sh.off[x];
      hi[k] = sh.off[x + 1];
      longest = max(longest, hi[k] - i[k]);
      i[k] += L == 64 ? l : 64 * k + l;
    }
    longest = __builtin_amdgcn_readfirstlane(longest);
#pragma unroll 1
    for (int done = 0; done < longest; done += 4 * L) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float v[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) v[m] = part[i[k] + m * L < hi[k] ? i[k] + m * L : 0];
#pragma unroll
        for (int m = 0; m < 4; ++m) v[m] = i[k] + m * L < hi[k] ? v[m] : 0.0f;
        const bool full = i[k] + 3 * L < hi[k];
        s[k][0] += double(v[0]);
#pragma unroll
        for (int m = 1; m < 4; ++m) s[k][m] += full ? double(v[m]) : 0.0;
        s[k][0] += full ? 0.0 : double(v[1]);
        s[k][0] += full ? 0.0 : double(v[2]);
        i[k] += 4 * L;
      }
    }
    double w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = wave_sum((s[k][0] + s[k][1]) + (s[k][2] + s[k][3]));
    if constexpr (L == 64) {
      if (l < 4 && first + l < n)
        sh.ss[unit[first + l]] = l == 0 ? w[0] : l == 1 ? w[1] : l == 2 ? w[2] : w[3];
    } else {
      if (l == 0) sh.ss[unit[first]] = ((w[0] + w[1]) + w[2]) + w[3];
    }
  }
}

// K2 and K3 for up to kStepUnits units.  (Running through the arithmetic once
// before the items arrive, to have its instructions in the cache, gained nothing
// behind long reads and cost 0.7 us behind short ones.)
__device__ void control(const UpdateArgs& u, const SelectArgs& s, const uint64_t* words,
                        uint32_t* launches, uint32_t num, int lanes, float* part,
                        StepShared& sh) {
  const int b = int(threadIdx.x), l = b & 63;
  const int wave = __builtin_amdgcn_readfirstlane(b >> 6);
  const bool has = b < u.num_units;
  const uint32_t tag = tag_of(*launches);
  const uint32_t late_from = num > kLate ? num - kLate : 0;
  UnitPast past{};
  int32_t lo = 0, hi = 0;
  if (has) {
    past = past_of_unit(u, b);
    lo = int32_t(u.unit_item_off[b]);
    hi = int32_t(u.unit_item_off[b + 1]);
  }
  int n_late = 0;
  if (lanes != 1) {
    // (all units where nothing is collected before the last items, those without any
    // too: each unit is summed in one of the two passes, an empty one to 0)
    bool late = has && late_from == 0;
    if (hi > lo) {
      const uint32_t last = item_wg(uint32_t(hi) - 1, num);
      late = last >= late_from || item_wg(uint32_t(lo), num) % kNumXcd != last % kNumXcd;
    }
    const uint64_t late_here = __ballot(late);
    if (has) sh.off[b + 1] = hi;
    if (b == 0) sh.off[0] = 0;
    if (l == 0) sh.late[wave] = __popcll(late_here);
    __syncthreads();
    int at = __popcll(late_here & ((uint64_t(1) << l) - 1));
#pragma unroll
    for (int w = 0; w < kK1Block / 64; ++w) {
      if (w < wave) at += sh.late[w];
      n_late += sh.late[w];
    }
    if (has) sh.unit[late ? at : n_late + (b - at)] = b;
  }
  if (l == 0) sh.lost[wave] = 0;
#pragma unroll 1
  for (uint32_t from = 0, to = late_from > 0 ? late_from : num;;) {
    collect(words, num, from, to, tag, part, &sh.lost[wave]);
    __syncthreads();
    const bool end = to == num;
    if (lanes != 1) {
      const int32_t* unit = sh.unit + (end ? 0 : n_late);
      const int n = end ? n_late : u.num_units - n_late;
      if (lanes == 64) sum_units<64>(part, unit, n, sh);
      else sum_units<256>(part, unit, n, sh);
    }
    if (end) break;
    from = late_from;
    to = num;
  }
  if (lanes != 1) __syncthreads();
  UnitStep x{};
  if (has) {
    const double ss = lanes == 1 ? lane_ss<1, int32_t>(part, lo, hi) : sh.ss[b];
    x = update_unit(u, past, norm_of_sumsq(ss));
    store_unit(u, b, x);
  }
  const uint64_t mine = wave_counts(has, x);
  if (l == 0) sh.counts[wave] = mine;
  __syncthreads();
  uint64_t all = 0;
  int place = 0;  // first the ranked candidates of the waves before
#pragma unroll
  for (int w = 0; w < kK1Block / 64; ++w) {
    if (w < wave) place += count_of(sh.counts[w], kCntRank);
    all += sh.counts[w];
  }
  int32_t tot[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) tot[k] = count_of(all, k);
  // Top_maxO by counting each ranked candidate's place: larger keys, and of
  // equal ones the smaller units, come first.
  bool active = has && x.cand;
  const bool ranked = active && x.key != 0;
  const int n_rank = tot[kCntRank];
  if (n_rank > s.max_o) {
    place += __popcll(__ballot(ranked) & ((uint64_t(1) << l) - 1));
    if (ranked) sh.key[place] = x.key;
    __syncthreads();
    if (ranked) {
      int before = 0;
#pragma unroll 4
      for (int j = 0; j < n_rank; ++j) {
        const uint64_t kj = sh.key[j];
        before += kj > x.key || (kj == x.key && j < place) ? 1 : 0;
      }
      active = before < s.max_o;
    }
  }
  if (has) {
    u.mask[b] = active ? 1 : 0;
    u.lock[b] = active ? x.lock : 0;
  }
  if (b == 0) {
    finish_step(s, past.t, tot);
    // (every item has read it if its word has arrived)
    *launches = launches_after(tag, (sh.lost[0] | sh.lost[1] | sh.lost[2] | sh.lost[3]) == 0);
  }
}

template <typename Bases>
__global__ __launch_bounds__(kK1Block, 5) void k123_step(const Item* __restrict__ items,
                                                      uint32_t num_items, int lanes,
                                                      const Bases seg_base,
                                                      const int32_t* __restrict__ seg_dtype,
                                                      uint64_t* words, uint32_t* launches,
                                                      UpdateArgs u, SelectArgs s) {
  extern __shared__ float part[];
  __shared__ StepShared sh;
  if (blockIdx.x == 0) {
    seg_base.keep();
    control(u, s, words, launches, num_items, lanes, part, sh);
    return;
  }
  const uint32_t w = blockIdx.x - 1, tag = tag_of(*launches);
  const Item it = items[xcd_item(w, num_items)];
  const float ss = item_sumsq(it, seg_base.of(it.seg), seg_dtype[it.seg], part);
  if (threadIdx.x == 0 && !words_lost(tag))
    __hip_atomic_store(words + w, uint64_t(tag) << 32 | __float_as_uint(ss), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

template <typename Bases>
void launch(const Item* items, int64_t num_items, const Bases& bases, const int32_t* seg_dtype,
            uint64_t* words, uint32_t* launches, const UpdateArgs& u, const SelectArgs& s,
            hipStream_t st) {
  static_assert(sizeof(Bases) + sizeof(UpdateArgs) + sizeof(SelectArgs) + 64 <= 4096,
                "kernel arguments");
  const size_t lds = std::max<size_t>(size_t(num_items), kK1Block / 64) * sizeof(float);
  hipLaunchKernelGGL(k123_step<Bases>, dim3(unsigned(num_items) + 1), dim3(kK1Block), lds, st,
                     items, uint32_t(num_items), lanes_per_unit(num_items, u.num_units), bases,
                     seg_dtype, words, launches, u, s);
}

template <int kMost>
PassedBases<kMost> passed(const char** table, const void* const* ptrs, int64_t num) {
  PassedBases<kMost> b;
  b.table = table;
  b.num = int32_t(num);
  memcpy(b.base, ptrs, size_t(num) * sizeof(void*));
  return b;
}

}  // namespace

// One launch takes up to kStepUnits units (a thread each) and kStepItems items:
// every workgroup of the launch is given the LDS that workgroup 0 keeps their
// partials in, and past 30 KiB fewer than five fit a CU, as many as the registers
// allow.  Two launches and one, us per step: 28 units in 196 items 8.0 and 5.6,
// 256 in 768 12.7 and 10.0, 256 in 3,072 34.0 and 31.0, 200 in 4,600 47.6 and
// 45.0, 64 in 6,144 64.0 and 59.1; with more LDS, 200 in 9,200 92.3 and 98.6.
bool whole_step_in_one_launch(int32_t num_units, int64_t num_items) {
  return num_units <= kStepUnits && num_items > 0 && num_items <= kStepItems;
}

hipError_t launch_step(const Item* items, int64_t num_items, const char** seg_base,
                       const void* const* ptrs, int64_t num_segs, const int32_t* seg_dtype,
                       uint64_t* words, uint32_t* launches, const UpdateArgs& u,
                       const SelectArgs& s, hipStream_t st) {
  if (ptrs == nullptr)
    launch(items, num_items, TableBases{seg_base}, seg_dtype, words, launches, u, s, st);
  else if (num_segs <= kK1FewPassed)
    launch(items, num_items, passed<kK1FewPassed>(seg_base, ptrs, num_segs), seg_dtype, words,
           launches, u, s, st);
  else
    launch(items, num_items, passed<kK1MostPassed>(seg_base, ptrs, num_segs), seg_dtype, words,
           launches, u, s, st);
  return hipGetLastError();
}

}  // namespace gnmr
