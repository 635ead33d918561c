// Internal declarations shared by the runtime and the kernels of libgnmr.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gnmr.h"
#include "k1_geometry.h"

namespace gnmr {

struct UpdateArgs {
  int32_t num_units;
  int32_t window;      // delta
  int32_t admitted;    // budget_mode == GNMR_BUDGET_ADMITTED
  int32_t static_set;  // budget_mode == GNMR_BUDGET_STATIC
  int32_t warmup;      // warmup_steps (W)
  const int64_t* step; // steps completed so far (device); this step is *step + 1
  double eps, alpha, beta;
  const int64_t* unit_item_off;  // [U+1]
  const float* partial;          // [items]
  const double* ext_norm;        // [U] or nullptr
  double* A;                     // [U]
  double* Q;                     // [window][U]
  double* norm;
  double* gnmr;
  double* dgnmr;
  double* risk;
  const uint8_t* rec;            // [U]
  int32_t lock_len;
  int32_t* lock;                 // [U], in: Lock after step t-1; out: after step t if selected
  uint8_t* mask;                 // [U], in: A_{t-1}; out: C_t
  // Members of C_t; K2 workgroup w of n units fills [w * n, ...).
  uint32_t* pool_rank;           // the upper half of its place in the ranking (larger first), 0:
                                 // active without ranking (warm-up; continuing unit under the
                                 // admitted-only budget)
  int32_t* pool_unit;
  uint32_t* key_low;             // [U], the lower half of each candidate's place in the ranking
  uint64_t* wg_counts;           // [workgroups], the packed counts of each workgroup
  double* gsum;                  // [U], sum of GNMR over the static baseline's profiling steps
};

struct SelectArgs {
  int32_t max_o;
  int32_t warmup;              // warmup_steps (W)
  int64_t* step;               // steps completed (device); advanced by one at the end of K3
  const uint32_t* pool_rank;   // from K2
  const int32_t* pool_unit;    // from K2
  const uint32_t* key_low;     // from K2
  const uint64_t* wg_counts;   // from K2
  int32_t num_wgs;             // K2's workgroups,
  int32_t wg_shift;            // of 1 << wg_shift units each (set by launch_update)
  int32_t* lock;               // [U], from K2; cleared outside A_t
  uint8_t* mask;               // [U], C_t from K2; out: A_t
  gnmr_stats* stats;
};

// K4 (actuator): rows by width, each class with its own lanes per row and
// 16-byte vectors per lane (see k4_actuator.hip).
constexpr int kK4Block = 256;
constexpr int kK4Classes = 12;
constexpr int kK4MaxCols = 16384;
int k4_class(int cols);
// Inputs of up to this many bytes are read with ordinary loads.  Between 34 MB
// (4096 x 4096: 12.4 us against 14.6 non-temporal) and 134 MB (16384 x 4096:
// 52.8 against 51.3); input and output together then fit the memory-side cache.
constexpr int64_t kK4CachedBytes = int64_t(64) << 20;
// Rows of up to this many features count as narrow in the limits on rows per
// call: 4 * kK4MaxWorkgroups of them and kK4MaxWorkgroups longer ones.
constexpr int kK4NarrowCols = 4096;
// A launch's grid holds fewer than 2^32 work items: at most this many
// workgroups of kK4Block lanes.
constexpr int64_t kK4MaxWorkgroups = int64_t(UINT32_MAX) / kK4Block;

struct ActSeg {
  const char* in;
  char* out;
  int32_t cols;
  int32_t unit;
};
static_assert(sizeof(ActSeg) == 24, "ActSeg layout");

struct RowItem {
  int32_t seg;
  int32_t row;
};

// K5 (weight-gradient GEMM with the sum of squares in its epilogue):
// 256x256 output tiles, K steps of 64, four waves; tiles walked in groups of
// kWgGroupRows tile rows.
constexpr int kWgBM = 256;
constexpr int kWgBN = 256;
constexpr int kWgBK = 64;
constexpr int kWgThreads = 256;
constexpr int kWgGroupRows = 8;

constexpr int kWgMaxBatch = 32;   // problems per launch (passed by value)

struct WgProblem {
  const uint16_t* dy;  // [K][M]
  const uint16_t* x;   // [K][N]
  uint16_t* dw;        // [M][N]
  float* tile_ss;      // [tiles_m * tiles_n]
  int64_t K;
  int32_t M, N, tiles_m, tiles_n;
  int32_t accumulate;  // 1: add the product to the stored dw
};

template <int kMost>
struct WgBatchOf {
  int32_t num;
  int32_t total_tiles;
  int32_t tile_begin[kMost];  // each problem's first tile in the launch's tile order
  WgProblem p[kMost];
};
typedef WgBatchOf<kWgMaxBatch> WgBatch;

int64_t wgrad_tiles(int32_t M, int32_t N);
hipError_t launch_wgrad(const WgBatch& batch, hipStream_t s);
// Rows [class_off[c], class_off[c + 1]) of `items` are of row class c; `bytes`
// is the bf16 input of all rows.
hipError_t launch_actuate(const RowItem* items, const int64_t* class_off, int64_t bytes,
                          const ActSeg* segs, const uint8_t* mask, int fmt_low, int fmt_rec,
                          hipStream_t s);
// One [rows][sg.cols] matrix, no row table.
hipError_t launch_actuate_matrix(const ActSeg& sg, int64_t rows, const uint8_t* mask,
                                 int fmt_low, int fmt_rec, hipStream_t s);
// K1 over the items; the segments' addresses from the device table seg_base, or,
// when ptrs is not null, from that host array of num_segs <= kK1MostPassed, which
// goes with the launch and is also left in seg_base.
constexpr int kK1FewPassed = 64, kK1MostPassed = 448;
hipError_t launch_sumsq(const Item* items, int64_t num_items, const char** seg_base,
                        const void* const* ptrs, int64_t num_segs, const int32_t* seg_dtype,
                        float* partial, hipStream_t s);
// K1, K2 and K3 as one launch (k123_step.hip).  words: [num_items] and launches: [1],
// zero before the first launch and used by nothing else.
constexpr int64_t kStepItems = 6144;
bool whole_step_in_one_launch(int32_t num_units, int64_t num_items);
// Lanes that sum one unit's partials.
int lanes_per_unit(int64_t num_items, int32_t num_units);
hipError_t launch_step(const Item* items, int64_t num_items, const char** seg_base,
                       const void* const* ptrs, int64_t num_segs, const int32_t* seg_dtype,
                       uint64_t* words, uint32_t* launches, const UpdateArgs& u,
                       const SelectArgs& s, hipStream_t st);
hipError_t launch_unit_sumsq(const int64_t* unit_item_off, const float* partial,
                             int64_t num_items, int32_t num_units, double* out, hipStream_t s);
hipError_t launch_update(const UpdateArgs& a, int64_t num_items, SelectArgs* sel, hipStream_t s);
hipError_t launch_select(const SelectArgs& a, hipStream_t s);
// K2 and K3 as one single-workgroup launch: used when the workload is small (norms
// given, or up to 10,240 partials: at most 1,024 units, 32 where a wavefront sums a
// unit's partials and 8 where a workgroup's worth of lanes does).
bool single_launch_update_select(const UpdateArgs& a, int64_t num_items);
hipError_t launch_update_select(const UpdateArgs& u, const SelectArgs& s, int64_t num_items,
                                hipStream_t st);

}  // namespace gnmr
