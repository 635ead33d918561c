// One unit's step of the controller: its norm from the partial sums, Alg. 1, the
// risk and the candidate pool of Alg. 2, and the step's counters.  Shared by the
// kernels that take steps.
#pragma once

#include <math.h>

#include "gnmr_internal.h"
#include "lane_ops.h"

namespace gnmr {
namespace {

// Fixed-order float64 sum of unit b's item partials by L lanes (lane < L):
// each lane keeps four running sums over a stride-L walk, then the lanes are
// combined by a fixed butterfly (L = 64) and a fixed cross-wave order
// (L = 256).  L = 1 is one thread per unit, for units of few items.
template <int L, typename Index>
__device__ __forceinline__ double lane_ss(const float* partial, Index i, Index hi) {
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  for (; i + 3 * L < hi; i += 4 * L) {
    const float a = partial[i], c = partial[i + L], d = partial[i + 2 * L], e = partial[i + 3 * L];
    s0 += double(a);
    s1 += double(c);
    s2 += double(d);
    s3 += double(e);
  }
  for (; i < hi; i += L) s0 += double(partial[i]);
  return (s0 + s1) + (s2 + s3);
}

// n_{b,t} from a unit's float64 sum of squares.  The sums of squares are
// accumulated in fp32, whose range ends at 2^128: a unit whose sum reaches it
// (a gradient norm of 2^64 or more) has no representable fp32 sum, so its
// norm is taken as +inf, a non-finite norm (the outcome when an fp32 square
// or partial overflows, made independent of how the sum is split into items).
// NaN stays NaN.
__device__ __forceinline__ double norm_of_sumsq(double ss) {
  return ss >= 0x1p128 ? double(INFINITY) : sqrt(ss);
}

// Order-preserving key of a candidate: R >= 0 (or +inf), so its IEEE bits
// are monotone in R; +1 keeps 0 free for "not a candidate".
__device__ __forceinline__ uint64_t cand_key(double R) {
  return uint64_t(__double_as_longlong(R)) + 1;
}

// A candidate's place in the ranking to 32 bits: the key's upper half and one
// more, 0 for a unit that is active without ranking (key 0).  Units that are
// equal here are told apart by the key's lower half.
__device__ __forceinline__ uint32_t rank_of(uint64_t key) {
  return key != 0 ? uint32_t(key >> 32) + 1u : 0u;
}

// One unit's step: what is stored for it, and its part in the counters and the
// candidate pool.
struct UnitStep {
  double n, A, G, D, R, gsum;
  uint64_t key;   // candidates: the ranking key, 0 when active without ranking
  int32_t lock;   // Lock after the step if the unit is selected
  int32_t slot;   // ring slot of the new GNMR
  bool cand, tg, td, tr, finite;
};

// What a unit's step takes from the steps before it.
struct UnitPast {
  int64_t t;          // this step
  double A;           // running mean
  double queue_sum;   // of the queue's values, oldest first, once it holds window of them
  double gsum;
  int32_t lock;
  int32_t slot;       // ring slot of the new GNMR
  bool queue_full, rec, active;
};

__device__ __forceinline__ UnitPast past_of_unit(const UpdateArgs& a, int b) {
  const int U = a.num_units;
  // The step counter lives on the device, so that a captured step replays
  // correctly: t = 1 + steps completed, the queue holds min(t - 1, delta)
  // values, and the oldest value sits in the slot the new one replaces.
  UnitPast p{};
  p.t = *a.step + 1;
  // (a 64-bit remainder is some 150 instructions, as many cache lines as all of Alg. 1)
  const uint64_t done = uint64_t(p.t - 1);
  p.slot = done >> 32 == 0 ? int(uint32_t(done) % uint32_t(a.window))
                           : int(done % uint64_t(uint32_t(a.window)));
  p.queue_full = p.t - 1 >= a.window;
  p.A = a.A[b];
  if (p.queue_full) {
    int slot = p.slot;
    for (int j = 0; j < a.window; ++j) {
      p.queue_sum += a.Q[int64_t(slot) * U + b];
      slot = slot + 1 == a.window ? 0 : slot + 1;
    }
  }
  p.rec = a.rec[b] != 0;
  p.lock = a.lock[b];
  p.active = a.mask[b] != 0;
  if (a.static_set) p.gsum = a.gsum[b];
  return p;
}

// Alg. 1 and the risk of Alg. 2 for a unit given its norm n, and the unit's
// membership of the candidate pool C_t.  Reads and stores nothing.
__device__ __forceinline__ UnitStep update_unit(const UpdateArgs& a, const UnitPast& p, double n) {
  const int64_t t = p.t;
  const bool warm = t <= a.warmup;
  const bool finite = isfinite(n);
  const double A_prev = p.A;
  // Alg. 1: GNMR = 1 at t = 1 or while the historical mean is 0.
  double G = 1.0;
  if (finite && t > 1 && A_prev != 0.0) G = n / (A_prev + a.eps);
  // Alg. 1: Delta-GNMR once the queue holds delta values.
  double D = 1.0;
  if (p.queue_full) {
    const double den = p.queue_sum / double(a.window) + a.eps;
    if (finite && den != 0.0) D = G / den;
  }
  // Alg. 1: running mean (and, in store_unit, the queue push: the new value
  // replaces the oldest).
  UnitStep u{};
  u.n = n;
  u.A = finite ? A_prev + (n - A_prev) / double(t) : A_prev;
  u.slot = p.slot;
  u.finite = finite;
  if (!finite) G = D = INFINITY;
  u.G = G;
  u.D = D;

  // Alg. 2: R = max(GNMR / alpha, Delta-GNMR / beta); the pool C_t holds the
  // recoverable units with R > 1 or a lock left from the previous step.
  const double gt = G / a.alpha;
  const double dt = D / a.beta;
  const double R = gt > dt ? gt : dt;
  u.R = R;
  const bool rec = p.rec;
  const bool trig = R > 1.0;
  const int32_t prev_lock = p.lock;
  const bool prev_active = p.active;
  bool cand = rec && (trig || prev_lock > 0);
  bool keep = false;
  double rank_by = R;
  if (a.static_set) {                 // static baseline: profile, rank once, hold
    u.gsum = p.gsum;
    if (t <= a.warmup) {
      u.gsum += finite ? G : 0.0;
      cand = keep = rec;
    } else if (t == a.warmup + 1) {
      cand = rec;
      rank_by = u.gsum / double(a.warmup);   // mean GNMR over steps 1..W
    } else {
      cand = keep = prev_active;
    }
  } else if (warm) {                  // warm-up: C_t = A_t = B_rec
    cand = rec;
    keep = rec;
  } else if (a.admitted && cand) {    // admitted-only budget: A_{t-1} members stay
    keep = prev_active;
  }
  u.key = cand && !keep ? cand_key(rank_by) : 0;
  u.lock = trig ? a.lock_len : (prev_lock > 0 ? prev_lock - 1 : 0);
  u.cand = cand;
  u.tg = rec && gt > 1.0;
  u.td = rec && dt > 1.0;
  u.tr = rec && trig;
  return u;
}

// Everything of the step but the selection's outcome.
__device__ __forceinline__ void store_unit(const UpdateArgs& a, int b, const UnitStep& u) {
  a.A[b] = u.A;
  a.Q[int64_t(u.slot) * a.num_units + b] = u.finite ? u.G : 1.0;
  if (a.static_set) a.gsum[b] = u.gsum;
  a.norm[b] = u.n;
  a.gnmr[b] = u.G;
  a.dgnmr[b] = u.D;
  a.risk[b] = u.R;
}

// The counters' contributions of one wavefront, kCountBits bits each: at most
// 256 units per workgroup, so the sum over a workgroup's waves fits too.
constexpr int kCountBits = 10;
enum : int { kCntCand, kCntRank, kCntTrigG, kCntTrigD, kCntTrigR, kCntNonFinite };

__device__ __forceinline__ int32_t count_of(uint64_t packed, int which) {
  return int32_t(packed >> (which * kCountBits)) & ((1 << kCountBits) - 1);
}

__device__ __forceinline__ uint64_t wave_counts(bool has, const UnitStep& u) {
  auto count = [&](bool x, int which) {
    return uint64_t(__popcll(__ballot(has && x))) << (which * kCountBits);
  };
  return count(u.cand, kCntCand) | count(u.cand && u.key != 0, kCntRank) |
         count(u.tg, kCntTrigG) | count(u.td, kCntTrigD) | count(u.tr, kCntTrigR) |
         count(!u.finite, kCntNonFinite);
}

// The counters of step t, by thread 0.
__device__ __forceinline__ void finish_step(const SelectArgs& a, int64_t t,
                                            const int32_t (&tot)[6]) {
  const int32_t n_cand = tot[kCntCand], n_rank = tot[kCntRank];
  const bool warm = t <= a.warmup;
  gnmr_stats st;
  st.t = t;
  st.n_trig_gnmr = tot[kCntTrigG];
  st.n_trig_dgnmr = tot[kCntTrigD];
  st.n_trig = tot[kCntTrigR];
  st.n_cand = n_cand;
  // the kept units, and as many ranked ones as the budget takes
  st.n_active = n_cand - n_rank + (n_rank < a.max_o ? n_rank : a.max_o);
  st.hit_maxo = (!warm && n_rank > 0 && n_rank >= a.max_o) ? 1 : 0;
  st.n_nonfinite = tot[kCntNonFinite];
  st.reserved = 0;
  *a.stats = st;
  *a.step = t;
}

}  // namespace
}  // namespace gnmr
