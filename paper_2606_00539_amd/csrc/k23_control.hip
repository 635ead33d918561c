// K2 and K3 of the GNMR controller pass for CDNA4 (gfx950).
//
//   K2 k2_update   per unit: fixed-order float64 sum of its K1 partials,
//                  n = sqrt, then Alg. 1 (GNMR, Delta-GNMR, running mean,
//                  queue), the risk R of Alg. 2, and membership of the
//                  candidate pool C_t (Alg. 2; Sec. 3.3)
//   K3 k3_select   one workgroup: Top_maxO over C_t by R (ties to the smaller
//                  index), lock update and step counters (Alg. 2; Sec. 3.3,
//                  3.4)
//
// Deterministic: fixed reduction orders, integer atomics (in LDS) only.
#include <math.h>

#include <type_traits>

#include "gnmr_internal.h"
#include "k3_pool.h"
#include "lane_ops.h"
#include "unit_step.h"

namespace gnmr {
namespace {

struct Min {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a < b ? a : b; }
};
struct Max {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; }
};

template <int L>
__device__ __forceinline__ double unit_ss(const int64_t* __restrict__ off,
                                          const float* __restrict__ partial, int b, int lane,
                                          double* red) {
  const double s = lane_ss<L, int64_t>(partial, off[b] + lane, off[b + 1]);
  if constexpr (L == 1) {
    return s;
  } else if constexpr (L == 64) {
    return wave_sum(s);
  } else {
    static_assert(L == 256, "1, 64 or 256 lanes per unit");
    const double w = wave_sum(s);
    if ((lane & 63) == 0) red[lane >> 6] = w;
    __syncthreads();
    return ((red[0] + red[1]) + red[2]) + red[3];
  }
}

template <int L>
__global__ __launch_bounds__(256) void k_unit_sumsq(const int64_t* __restrict__ off,
                                                    const float* __restrict__ partial,
                                                    int num_units, double* __restrict__ out) {
  __shared__ double red[4];
  const int lane = L == 1 ? 0 : int(threadIdx.x % L);
  const int b = blockIdx.x * (256 / L) + threadIdx.x / L;
  if (b >= num_units) return;  // uniform per workgroup when L = 256
  const double s = unit_ss<L>(off, partial, b, lane, red);
  if (lane == 0) out[b] = s;
}

// K2: L lanes per unit sum its partials; lane 0 then runs Alg. 1, the risk of
// Alg. 2, and marks the unit's membership of the candidate pool C_t.  Each
// workgroup leaves its counts in one word and its members of C_t at the start
// of its own part of the pool: no atomics (42,496 units: 4.2 us, 5.7 with one per
// counter and workgroup on 64 sets of counters).  The mask and Lock are written as
// if all of C_t were selected: K3 clears them for the members of C_t that the
// budget leaves out.
template <int L>
__global__ __launch_bounds__(256) void k2_update(UpdateArgs a) {
  constexpr int kUnits = 256 / L;  // per workgroup
  __shared__ double red[4];
  __shared__ uint64_t s_counts[4];
  const int tid = int(threadIdx.x), wave = tid >> 6;
  const int lane = L == 1 ? 0 : tid % L;
  const int b = blockIdx.x * kUnits + tid / L;
  if (L == 256 && b >= a.num_units) return;  // the whole workgroup
  const bool in = b < a.num_units;           // uniform per wavefront when L = 64
  double n = 0.0;
  if (in) {
    if (a.ext_norm != nullptr) {
      n = a.ext_norm[b];
    } else {
      n = norm_of_sumsq(unit_ss<L>(a.unit_item_off, a.partial, b, lane, red));
    }
  }
  const bool has = in && lane == 0;
  UnitStep u{};
  if (has) u = update_unit(a, past_of_unit(a, b), n);
  const uint64_t members = __ballot(has && u.cand);
  uint64_t mine = wave_counts(has, u);
  int at = __popcll(members & ((uint64_t(1) << (tid & 63)) - 1));
  if constexpr (L < 256) {  // (L = 256: the one unit is the first wave's)
    if ((tid & 63) == 0) s_counts[wave] = mine;
    __syncthreads();
    for (int w = 0; w < wave; ++w) at += count_of(s_counts[w], kCntCand);
    mine = ((s_counts[0] + s_counts[1]) + s_counts[2]) + s_counts[3];
  }
  if (tid == 0) a.wg_counts[blockIdx.x] = mine;
  if (has) {
    if (u.cand) {
      a.pool_rank[blockIdx.x * kUnits + at] = rank_of(u.key);
      a.pool_unit[blockIdx.x * kUnits + at] = b;
      a.key_low[b] = uint32_t(u.key);
    }
    a.mask[b] = u.cand ? 1 : 0;
    a.lock[b] = u.cand ? u.lock : 0;
    store_unit(a, b, u);
  }
}

constexpr int kK3Block = 1024;
constexpr int kK3Cap = 16384;  // candidates held in LDS (128 KiB); larger pools are read again
constexpr int kK3Count = 128;  // pools up to this size are ranked by direct counting
constexpr int kK3Waves = kK3Block / 64;
constexpr int kK23Parts = 10240;  // the most partials that k23_small sums (40 KiB in LDS)

// The k-th largest value (Top_maxO's threshold) by a radix select: 11 bits per
// pass, starting at the highest bit in which value - smallest differs, which
// the few binades of R above 1 leave high in the word.  Once the bucket that
// holds the k-th value has at most 64 members, those are gathered and the
// workgroup finishes by counting, for each, the values above it: after one pass
// for typical pools.
constexpr int kDigit = 11;
constexpr int kBins = 1 << kDigit;
static_assert(kBins == 2 * kK3Block, "two bins per thread");

struct SelectShared {
  uint32_t hist[kBins];          // zero between passes
  uint32_t lo[kK3Waves], hi[kK3Waves];
  uint32_t above[kK3Waves];
  uint64_t key[kK3Count];        // the small bucket's values, or the small pool's keys
  int32_t unit[kK3Count];        // and units
  uint32_t T, bin, k, bucket, n, rest, equal;
};

struct Threshold {
  uint32_t T;      // the k-th largest value
  uint32_t rest;   // how many values equal to T are among the k largest
  uint32_t equal;  // values equal to T
};

// Pool::each(f) calls f(rank, unit, valid) for each of this thread's candidates,
// with the whole wavefront; val(rank, unit, v) says whether a candidate takes
// part and sets its value v; n of them do; lo and hi are at most and at least
// this thread's values (~0 and 0 for none).  Called by every thread of the
// workgroup, with k <= n; sh.n is 0 and sh.hist zero on entry and on return.
template <typename Pool, typename Val>
__device__ Threshold kth_largest(const Pool& pool, Val val, uint32_t k, uint32_t n, uint32_t lo,
                                 uint32_t hi, SelectShared& sh) {
  static_assert(kK3Waves == 16, "a row of lanes per wave sums");
  const int tid = int(threadIdx.x), l = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  lo = wave_scan(lo, ~0u, Min{});
  hi = wave_scan(hi, 0u, Max{});
  if (l == 63) {
    sh.lo[wave] = lo;
    sh.hi[wave] = hi;
  }
  __syncthreads();
  lo = lane_of(row_scan(sh.lo[l & 15], ~0u, Min{}), 15);
  hi = lane_of(row_scan(sh.hi[l & 15], 0u, Max{}), 15);
  if (lo == hi) {     // one value, and one bin for all of the atomics
    __syncthreads();  // (sh.lo and sh.hi are read)
    return Threshold{lo, k, n};
  }
  const int bits = 32 - __clz(int(hi - lo));
  int shift = bits > kDigit ? bits - kDigit : 0, width = kDigit;
  uint32_t prefix = 0;  // (value - lo) >> (shift + width) of the bucket
  for (;;) {
    const uint32_t digits = (1u << width) - 1u;
    pool.each([&](uint32_t rank, int32_t unit, bool valid) {
      uint32_t v = 0;
      const bool in = valid && val(rank, unit, v);
      const uint32_t d = (v - lo) >> shift;
      if (in && (d >> width) == prefix) atomicAdd(&sh.hist[d & digits], 1u);
    });
    __syncthreads();
    // The bin of the k-th largest: thread t holds bins 2t and 2t+1; sums over
    // the threads give the members above them, and the one thread whose bins
    // reach k names the bin.
    const uint32_t h0 = sh.hist[2 * tid], h1 = sh.hist[2 * tid + 1], own = h0 + h1;
    sh.hist[2 * tid] = sh.hist[2 * tid + 1] = 0;
    const uint32_t sum = wave_prefix(own);
    if (l == 63) sh.above[wave] = sum;
    __syncthreads();
    const uint32_t waves = row_prefix(sh.above[l & 15]);  // sums of waves 0 .. l
    const uint32_t above = lane_of(waves, 15) - lane_of(waves, wave) + lane_of(sum, 63) - sum;
    if (above < k && above + own >= k) {
      const bool upper = above + h1 >= k;
      sh.bin = uint32_t(2 * tid) + (upper ? 1u : 0u);
      sh.k = k - above - (upper ? 0u : h1);
      sh.bucket = upper ? h1 : h0;
    }
    __syncthreads();
    prefix = (prefix << width) | sh.bin;
    k = sh.k;
    const uint32_t bucket = sh.bucket;
    if (shift == 0) return Threshold{lo + prefix, k, bucket};
    if (bucket <= 64) break;
    width = shift < kDigit ? shift : kDigit;
    shift -= width;
  }
  pool.each([&](uint32_t rank, int32_t unit, bool valid) {
    uint32_t v = 0;
    if (valid && val(rank, unit, v) && ((v - lo) >> shift) == prefix)
      sh.key[atomicAdd(&sh.n, 1u)] = v;
  });
  __syncthreads();
  {
    // 16 threads a member, four comparisons each
    static_assert(kK3Block == 64 * 16, "");
    const uint32_t m = sh.n, i = uint32_t(tid) >> 4;
    const uint32_t mine = i < m ? uint32_t(sh.key[i]) : 0;
    uint32_t both = 0;  // members above (low half), and at or above
#pragma unroll
    for (uint32_t j = uint32_t(tid) & 15u; j < 64; j += 16) {
      const uint32_t vj = uint32_t(sh.key[j]);  // (stale past m)
      both += j < m ? (vj > mine ? 1u : 0u) + (vj >= mine ? 0x10000u : 0u) : 0u;
    }
#pragma unroll
    for (int x = 8; x >= 1; x >>= 1) both += __shfl_xor(both, x, 16);
    const uint32_t above = both & 0xFFFFu, not_below = both >> 16;
    // the k-th largest: fewer than k above it, at least k at or above
    if (i < m && above < k && not_below >= k) {
      sh.T = mine;
      sh.rest = k - above;
      sh.equal = not_below - above;
    }
  }
  __syncthreads();
  if (tid == 0) sh.n = 0;
  __syncthreads();
  return Threshold{sh.T, sh.rest, sh.equal};
}

// Top_maxO over the pool: drop(unit) for every ranked member of C_t that is not
// in A_t.  Kept units (rank 0: warm-up; continuing units under the admitted-only
// budget; the held static set) are active without ranking; the others are
// ranked for the budget.  When at most maxO are ranked they are all active.
// Otherwise pools of up to kK3Count count each candidate's place in the order (R
// descending, index ascending) directly; larger ones take the maxO-th largest
// rank, then, among the units that share it when not all of them may be taken,
// that of the keys' lower halves (key_low(unit)), and then the index of the last
// unit taken.  pool.lo, pool.hi: the smallest and largest of this thread's
// nonzero ranks.  Units are below `places`.
template <typename Pool, typename Low, typename Drop>
__device__ void select_pool(const Pool& pool, int n_cand, int n_rank, int max_o, uint32_t places,
                            Low key_low, SelectShared& sh, Drop drop) {
  if (n_rank <= max_o) return;
  if (max_o == 0) {
    pool.each([&](uint32_t rank, int32_t unit, bool valid) {
      if (valid && rank != 0) drop(unit);
    });
    return;
  }
  if (n_cand <= kK3Count) {
    pool.each([&](uint32_t rank, int32_t unit, bool valid) {
      if (!valid) return;
      const uint32_t i = atomicAdd(&sh.n, 1u);
      sh.key[i] = uint64_t(rank) << 32 | key_low(unit);
      sh.unit[i] = unit;
    });
    __syncthreads();
    const int i = int(threadIdx.x);
    if (i < n_cand) {
      const uint64_t key = sh.key[i];
      const int32_t unit = sh.unit[i];
      // kept units have rank 0, below every ranked key: none before a ranked one
      int before = 0;
#pragma unroll 8
      for (int j = 0; j < n_cand; ++j) {
        const uint64_t kj = sh.key[j];
        before += (kj > key || (kj == key && sh.unit[j] < unit)) ? 1 : 0;
      }
      if ((key >> 32) != 0 && before >= max_o) drop(unit);
    }
    return;
  }
  const Threshold by_rank = kth_largest(
      pool,
      [](uint32_t rank, int32_t, uint32_t& v) {
        v = rank;
        return rank != 0;
      },
      uint32_t(max_o), uint32_t(n_rank), pool.lo, pool.hi, sh);
  const uint32_t T = by_rank.T;
  uint32_t low_cut = 0;          // among rank T: every lower half,
  int32_t unit_cut = INT32_MAX;  // and among rank T and that lower half: every unit
  if (by_rank.rest < by_rank.equal) {
    // Ties are mostly exact (units that overflowed, a gradient never written): one
    // pass then tells that the lower halves are all the same.  All units tied, us a
    // step, with three passes over 32 bits of each half and now: 4,096 units 37.6 and
    // 14.0, 42,496 331 and 164, 300,000 2,390 and 1,230; half of them infinite: 32.3
    // and 21.3, 258 and 197, 1,870 and 1,450.
    uint32_t lo = ~0u, hi = 0;
    pool.each([&](uint32_t rank, int32_t unit, bool valid) {
      if (!valid || rank != T) return;
      const uint32_t low = key_low(unit);
      lo = low < lo ? low : lo;
      hi = low > hi ? low : hi;
    });
    const Threshold by_low = kth_largest(
        pool,
        [&](uint32_t rank, int32_t unit, uint32_t& v) {
          if (rank != T) return false;
          v = key_low(unit);
          return true;
        },
        by_rank.rest, by_rank.equal, lo, hi, sh);
    low_cut = by_low.T;
    if (by_low.rest < by_low.equal)
      unit_cut = int32_t(~kth_largest(
                              pool,
                              [&](uint32_t rank, int32_t unit, uint32_t& v) {
                                v = ~uint32_t(unit);
                                return rank == T && key_low(unit) == low_cut;
                              },
                              by_low.rest, by_low.equal, ~(places - 1u), ~0u, sh)
                              .T);
  }
  const bool all_of_T = by_rank.rest == by_rank.equal;
  pool.each([&](uint32_t rank, int32_t unit, bool valid) {
    if (!valid || rank == 0 || rank > T || (rank == T && all_of_T)) return;
    if (rank == T) {
      const uint32_t low = key_low(unit);
      if (low > low_cut || (low == low_cut && unit <= unit_cut)) return;
    }
    drop(unit);
  });
}

// One candidate per thread.
struct OwnPool {
  uint32_t rank;
  int32_t unit;
  bool valid;
  uint32_t lo, hi;
  template <typename F>
  __device__ __forceinline__ void each(F f) const {
    f(rank, unit, valid);
  }
};

struct LdsPool {
  const uint32_t* rank;
  const int32_t* unit;
  int n;
  uint32_t lo, hi;
  template <typename F>
  __device__ __forceinline__ void each(F f) const {
    for (int base = 0; base < n; base += kK3Block) {
      const int i = base + int(threadIdx.x);
      f(i < n ? rank[i] : 0, i < n ? unit[i] : 0, i < n);
    }
  }
};

// Larger pools: every place of every K2 workgroup, read again for every pass.
struct GlobalPool {
  const uint32_t* pool_rank;
  const int32_t* pool_unit;
  const uint64_t* wg_counts;
  uint32_t places;
  int shift;
  uint32_t lo, hi;
  template <typename F>
  __device__ __forceinline__ void each(F f) const {
    const uint32_t rounds = pool_rounds(places, kK3Block);
    for (uint32_t r = 0; r < rounds; ++r) {
      const uint32_t i = r * kK3Block + threadIdx.x;
      const bool valid = i < places && int32_t(i & ((1u << shift) - 1u)) <
                                           count_of(wg_counts[i >> shift], kCntCand);
      f(valid ? pool_rank[i] : 0, valid ? pool_unit[i] : 0, valid);
    }
  }
};

// Four bytes a lane straight to LDS: lane l's to p[l] (p the same for the wave).
template <typename T>
__device__ __forceinline__ void load_to_lds(const T* from, T* p) {
  __builtin_amdgcn_global_load_lds((const void*)from,
                                   (__attribute__((address_space(3))) void*)p, 4, 0, 0);
}

// Keeps the smallest and largest nonzero rank.
__device__ __forceinline__ void widen_range(uint32_t rank, uint32_t& lo, uint32_t& hi) {
  lo = rank != 0 && rank < lo ? rank : lo;
  hi = rank > hi ? rank : hi;
}

// K3: a single workgroup, over the members of C_t that K2's workgroups left.
// When the budget takes them all it only adds up the counters.  Bound by
// latency: one load for the counts, one batch of loads for the pool (ranks and
// units; nothing is looked up per candidate unless ranks tie at the cut), then LDS
// passes.  The instruction cache starts cold, so loops stay rolled and sums over
// the waves are rows of lanes: unrolled 12 to a thread the same steps took 11 to
// 12 us.  42,496 units with a pool of about 4,000 for maxO = 64: 8.8 us (19.4
// with keys, flags and locks gathered per unit through 64 lists and 8-bit passes
// over 64-bit keys); no ranking: 4.0 us.
__global__ __launch_bounds__(kK3Block) void k3_select(SelectArgs a) {
  __shared__ SelectShared sh;
  __shared__ int32_t s_off[kK3Block + 1];  // first candidate of each thread's workgroups
  __shared__ uint32_t s_wave[6 * kK3Waves];
  __shared__ uint32_t s_rank[kK3Cap];
  __shared__ int32_t s_unit[kK3Cap];
  const int tid = int(threadIdx.x), l = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t t_now = *a.step + 1;
  const uint32_t places = pool_places(a.num_wgs, a.wg_shift);
  sh.hist[2 * tid] = sh.hist[2 * tid + 1] = 0;
  if (tid == 0) sh.n = 0;
  // Thread t counts for K2 workgroups [t * per, (t + 1) * per).
  const int per = (a.num_wgs + kK3Block - 1) / kK3Block;
  uint32_t sum[6] = {};
  for (int w = tid * per; w < (tid + 1) * per && w < a.num_wgs; ++w) {
    const uint64_t v = a.wg_counts[w];
#pragma unroll
    for (int k = 0; k < 6; ++k) sum[k] += uint32_t(count_of(v, k));
  }
  const uint32_t own = sum[kCntCand];
#pragma unroll
  for (int k = 0; k < 6; ++k) sum[k] = wave_prefix(sum[k]);
  if (l == 63)
#pragma unroll
    for (int k = 0; k < 6; ++k) s_wave[k * kK3Waves + wave] = sum[k];
  __syncthreads();
  // a row of 16 lanes per counter: its sums over the waves
  const uint32_t first4 = row_prefix(s_wave[l]), last2 = row_prefix(s_wave[64 + (l & 31)]);
  const int32_t tot[6] = {
      int32_t(lane_of(first4, 15)), int32_t(lane_of(first4, 31)), int32_t(lane_of(first4, 47)),
      int32_t(lane_of(first4, 63)), int32_t(lane_of(last2, 15)),  int32_t(lane_of(last2, 31))};
  const int n_cand = tot[kCntCand];
  if (tot[kCntRank] > a.max_o) {
    auto drop = [&](int32_t unit) {
      a.mask[unit] = 0;
      a.lock[unit] = 0;
    };
    auto key_low = [&](int32_t unit) { return a.key_low[unit]; };
    uint32_t lo = ~0u, hi = 0;
    s_off[tid] = int32_t((wave > 0 ? lane_of(first4, wave - 1) : 0u) + sum[kCntCand] - own);
    if (tid == 0) s_off[kK3Block] = n_cand;
    __syncthreads();
    if (n_cand <= kK3Cap) {
      if (a.wg_shift >= 6 && per == 1) {
        // K2 workgroups of 256 units: a wavefront each, straight to LDS, so that
        // all of the loads are in flight and the loop stays small
        for (int w = wave; w < a.num_wgs; w += kK3Waves) {
          const int off = __builtin_amdgcn_readfirstlane(s_off[w]);
          const int cnt = __builtin_amdgcn_readfirstlane(s_off[w + 1]) - off;
          const int64_t first = int64_t(w) << a.wg_shift;
          for (int j = 0; j < cnt; j += 64) {
            if (j + l < cnt) {
              load_to_lds(a.pool_rank + first + j + l, s_rank + off + j);
              load_to_lds(a.pool_unit + first + j + l, s_unit + off + j);
            }
          }
        }
        __builtin_amdgcn_s_waitcnt(0);
      } else {
        // Smaller workgroups, or more of them than threads: one to 64 threads each,
        // two latencies a round; or, where that is more than twice as many rounds,
        // candidate i to thread i: bisection finds the thread that counted it, that
        // thread's counts the workgroup.  Us a step with threads to the workgroups and
        // to the candidates: 300,000 units, 1,000 and 16,000 candidates 52.7 and 15.5,
        // 74.4 and 43.5; 2,000,000, 4,000 candidates 262 and 61.8; workgroups of four,
        // 10,000 units, 1,251 and 10,000 candidates 22.1 and 17.7, 24.6 and 32.9.
        const int group = a.wg_shift < 6 ? 1 << a.wg_shift : 64;
        if (pool_rounds(uint32_t(a.num_wgs) * uint32_t(group), kK3Block) <=
            2u * pool_rounds(uint32_t(n_cand), kK3Block)) {
          for (int t = tid / group; t * per < a.num_wgs; t += kK3Block / group) {
            int off = s_off[t];
            for (int w = t * per; w < (t + 1) * per && w < a.num_wgs; ++w) {
              const int cnt = count_of(a.wg_counts[w], kCntCand);
              for (int j = tid & (group - 1); j < cnt; j += group) {
                s_rank[off + j] = a.pool_rank[(int64_t(w) << a.wg_shift) + j];
                s_unit[off + j] = a.pool_unit[(int64_t(w) << a.wg_shift) + j];
              }
              off += cnt;
            }
          }
        } else {
          for (int i = tid; i < n_cand; i += kK3Block) {
            int t = 0;
#pragma unroll 1
            for (int half = kK3Block / 2; half > 0; half /= 2)
              t += s_off[t + half] <= i ? half : 0;
            const int first = i - s_off[t];
            int w = t * per, j = first, seen = 0;
#pragma unroll 4
            for (int k = 1; k < per; ++k) {
              // (past the last workgroup all of them are seen: nothing moves any more)
              seen += count_of(a.wg_counts[min(t * per + k, a.num_wgs) - 1], kCntCand);
              if (seen <= first) {
                w = t * per + k;
                j = first - seen;
              }
            }
            s_rank[i] = a.pool_rank[(int64_t(w) << a.wg_shift) + j];
            s_unit[i] = a.pool_unit[(int64_t(w) << a.wg_shift) + j];
          }
        }
      }
      __syncthreads();
      LdsPool pool{s_rank, s_unit, n_cand, 0, 0};
      pool.each([&](uint32_t rank, int32_t, bool) { widen_range(rank, lo, hi); });
      pool.lo = lo;
      pool.hi = hi;
      select_pool(pool, n_cand, tot[kCntRank], a.max_o, places, key_low, sh, drop);
    } else {
      GlobalPool pool{a.pool_rank, a.pool_unit, a.wg_counts, places, a.wg_shift, 0, 0};
      pool.each([&](uint32_t rank, int32_t, bool) { widen_range(rank, lo, hi); });
      pool.lo = lo;
      pool.hi = hi;
      select_pool(pool, n_cand, tot[kCntRank], a.max_o, places, key_low, sh, drop);
    }
  }
  if (tid == 0) finish_step(a, t_now, tot);
}

// K2 and K3 in one workgroup, for small workloads (single_launch_update_select).
// L lanes sum a unit's partials exactly as in k2_update<L>: one thread straight
// from memory, more of them from LDS, where the partials arrive all in flight at
// once.  Then one thread per unit, with its candidate in its own registers.  One
// launch instead of two; the same arithmetic, so the same results.
template <int L>
__global__ __launch_bounds__(kK3Block) void k23_small(UpdateArgs u, SelectArgs s, int num_parts) {
  __shared__ SelectShared sh;
  __shared__ uint64_t s_counts[kK3Waves];
  __shared__ uint8_t s_out[kK3Block];
  __shared__ int32_t s_off[kK3Block + 1];
  __shared__ double s_ss[kK3Block];
  __shared__ double red[kK3Waves];
  __shared__ float s_part[kK23Parts];
  const int b = int(threadIdx.x), l = b & 63, wave = __builtin_amdgcn_readfirstlane(b >> 6);
  const int64_t t_now = *s.step + 1;
  const bool has = b < u.num_units;
  double n = 0.0;
  if (L == 1) {
    if (has)
      n = u.ext_norm != nullptr
              ? u.ext_norm[b]
              : norm_of_sumsq(unit_ss<1>(u.unit_item_off, u.partial, b, 0, nullptr));
    sh.hist[2 * b] = sh.hist[2 * b + 1] = 0;
    if (b == 0) sh.n = 0;
    s_out[b] = 0;
  } else {
    for (int i = 64 * wave; i < num_parts; i += kK3Block)
      if (i + l < num_parts) load_to_lds(u.partial + i + l, s_part + i);
    if (has) s_off[b + 1] = int32_t(u.unit_item_off[b + 1]);
    if (b == 0) s_off[0] = 0;
    sh.hist[2 * b] = sh.hist[2 * b + 1] = 0;
    if (b == 0) sh.n = 0;
    s_out[b] = 0;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    {
      constexpr int kAtOnce = kK3Block / L;
      for (int first = 0; first < u.num_units; first += kAtOnce) {
        const int x = first + b / L;
        const bool in = x < u.num_units;
        const double w = wave_sum(
            in ? lane_ss<L, int32_t>(s_part, s_off[x] + b % L, s_off[x + 1]) : 0.0);
        if constexpr (L == 64) {
          if (in && l == 0) s_ss[x] = w;
        } else {
          if (l == 0) red[wave] = w;
          __syncthreads();
          if (in && b % L == 0)
            s_ss[x] = ((red[wave] + red[wave + 1]) + red[wave + 2]) + red[wave + 3];
          __syncthreads();
        }
      }
      __syncthreads();
      if (has) n = norm_of_sumsq(s_ss[b]);
    }
  }
  UnitStep x{};
  if (has) {
    x = update_unit(u, past_of_unit(u, b), n);
    store_unit(u, b, x);
  }
  const uint64_t mine = wave_counts(has, x);
  if ((b & 63) == 0) s_counts[b >> 6] = mine;
  __syncthreads();
  const uint64_t of_wave = s_counts[l & 15];  // each row of lanes sums over the waves
  int32_t tot[6];
#pragma unroll
  for (int k = 0; k < 6; ++k)
    tot[k] = int32_t(lane_of(row_prefix(uint32_t(count_of(of_wave, k))), 15));
  bool active = has && x.cand;
  uint32_t lo = ~0u, hi = 0;
  const uint32_t rank = rank_of(x.key);  // (0 for other than ranked candidates)
  widen_range(rank, lo, hi);
  // (a thread's own candidate is the only one whose key it is asked for; it
  // is told through LDS that it is out, by whichever thread ranked it)
  select_pool(OwnPool{rank, b, active, lo, hi}, tot[kCntCand], tot[kCntRank], s.max_o, kK3Block,
              [&](int32_t) { return uint32_t(x.key); }, sh, [&](int32_t unit) { s_out[unit] = 1; });
  __syncthreads();
  active = active && s_out[b] == 0;
  if (has) {
    u.mask[b] = active ? 1 : 0;
    u.lock[b] = active ? x.lock : 0;
  }
  if (b == 0) finish_step(s, t_now, tot);
}

}  // namespace

// Lanes per unit for the partial sums: one thread when units have few items,
// a wavefront for moderate counts, a whole workgroup once long strided walks
// would be latency bound.
int lanes_per_unit(int64_t num_items, int32_t num_units) {
  const int64_t per = num_items / (num_units > 0 ? num_units : 1);
  return per < 32 ? 1 : per < 512 ? 64 : 256;
}

template <int L>
static dim3 unit_grid(int32_t num_units) {
  return dim3(unsigned((int64_t(num_units) * L + 255) / 256));
}

hipError_t launch_unit_sumsq(const int64_t* unit_item_off, const float* partial,
                             int64_t num_items, int32_t num_units, double* out, hipStream_t s) {
  switch (lanes_per_unit(num_items, num_units)) {
    case 1:
      hipLaunchKernelGGL(k_unit_sumsq<1>, unit_grid<1>(num_units), dim3(256), 0, s,
                         unit_item_off, partial, num_units, out);
      break;
    case 64:
      hipLaunchKernelGGL(k_unit_sumsq<64>, unit_grid<64>(num_units), dim3(256), 0, s,
                         unit_item_off, partial, num_units, out);
      break;
    default:
      hipLaunchKernelGGL(k_unit_sumsq<256>, unit_grid<256>(num_units), dim3(256), 0, s,
                         unit_item_off, partial, num_units, out);
  }
  return hipGetLastError();
}

hipError_t launch_update(const UpdateArgs& a, int64_t num_items, SelectArgs* sel, hipStream_t s) {
  const int L = a.ext_norm != nullptr ? 1 : lanes_per_unit(num_items, a.num_units);
  const dim3 grid = L == 1    ? unit_grid<1>(a.num_units)
                    : L == 64 ? unit_grid<64>(a.num_units)
                              : unit_grid<256>(a.num_units);
  sel->num_wgs = int32_t(grid.x);
  sel->wg_shift = L == 1 ? 8 : L == 64 ? 2 : 0;
  if (L == 1)
    hipLaunchKernelGGL(k2_update<1>, grid, dim3(256), 0, s, a);
  else if (L == 64)
    hipLaunchKernelGGL(k2_update<64>, grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(k2_update<256>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_select(const SelectArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k3_select, dim3(1), dim3(kK3Block), 0, s, a);
  return hipGetLastError();
}

// Whether one workgroup does the whole step: a unit by one thread, up to one per
// thread and kK23Parts partials read; by a wavefront or a workgroup's worth of
// lanes, while at most two rounds of 16 or 4 units follow each other.  One launch
// against two, back to back (us): 28 units x 2 partials 3.9, 6.9; 1000 x 5 4.9,
// 6.9; 7 x 691 5.1, 7.0; 1 x 256 3.9, 7.0; but 1000 x 31 8.7, 6.8; 84 x 73 7.0,
// 7.0; 32 x 1000 12, 6.8.
bool single_launch_update_select(const UpdateArgs& a, int64_t num_items) {
  if (a.ext_norm != nullptr) return a.num_units <= kK3Block;
  const int L = lanes_per_unit(num_items, a.num_units);
  return num_items <= kK23Parts &&
         a.num_units <= (L == 1 ? kK3Block : L == 64 ? 2 * kK3Waves : 2 * kK3Waves / 4);
}

hipError_t launch_update_select(const UpdateArgs& u, const SelectArgs& s, int64_t num_items,
                                hipStream_t st) {
  const int L = u.ext_norm != nullptr ? 1 : lanes_per_unit(num_items, u.num_units);
  const int n = u.ext_norm != nullptr ? 0 : int(num_items);
  if (L == 1)
    hipLaunchKernelGGL(k23_small<1>, dim3(1), dim3(kK3Block), 0, st, u, s, n);
  else if (L == 64)
    hipLaunchKernelGGL(k23_small<64>, dim3(1), dim3(kK3Block), 0, st, u, s, n);
  else
    hipLaunchKernelGGL(k23_small<256>, dim3(1), dim3(kK3Block), 0, st, u, s, n);
  return hipGetLastError();
}

}  // namespace gnmr
