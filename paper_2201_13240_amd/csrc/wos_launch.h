// Host-side launchers of the kernels in wos_kernels.hip, wos_grid.hip and wos_walker_*.hip
// (internal interface).
#pragma once
#include <hip/hip_runtime_api.h>

#include <cstddef>
#include <cstdint>

#include "wos_types.h"

namespace wos {

struct WalkerLaunch {
  int fp64;
  int dim;
  int geom;
  unsigned grid;
  unsigned block;
  const DevItem* items;
  int n_items;
  uint32_t n_tiles;   // tiles of all items
  uint32_t n_queues;  // 1 or kTileQueues: queues the tiles are cut into
  uint32_t* tile_counter;   // [kTileQueues * kTileQueueStride], zeroed before the launch
  uint64_t* slots;    // accumulation slots, slot_words(grad dim) words each, zeroed before the launch
  int slot_words;
  const LaunchParams* lp;
  uint64_t max_steps;
  int variant;
  int compensated;
  int fp32_draws;     // FP64 walker with the FP32 walker's uniforms
  int rr;
  double ww_lo;
  double ww_hi;       // 0: no splitting
  void* grad;         // gradient records (T[grid wave][kGradRecords][2 + 3 dim]) or null
  uint64_t* events;   // non-null selects the event-counting build of the walker
};

// Items of a job handed to the device with the launch that prepares it: their table entries,
// the problems in FP64, and the first block that each takes of the launch.
constexpr int kPrepItems = 16;
struct PrepArgs {
  DevItem item[kPrepItems];
  const void* problem64[kPrepItems];
  uint32_t block0[kPrepItems + 1];
  int32_t n;
  DevItem* table;          // entry of the first item, or null: the table is there already
  LaunchParams* lp;
  uint64_t seed;
  uint32_t* counters;
  uint64_t* slots;
  uint64_t slot_words;     // words to clear
};

hipError_t launch_walker(const WalkerLaunch& L, hipStream_t st);
// The walkers of one precision and dimension (wos_walker_{f32,f64}_{2d,3d}.hip).
hipError_t launch_walker_f32_2d(const WalkerLaunch& L, hipStream_t st);
hipError_t launch_walker_f32_3d(const WalkerLaunch& L, hipStream_t st);
hipError_t launch_walker_f64_2d(const WalkerLaunch& L, hipStream_t st);
hipError_t launch_walker_f64_3d(const WalkerLaunch& L, hipStream_t st);
const void* walker_symbol_f32_2d(int geom, int mode);
const void* walker_symbol_f32_3d(int geom, int mode);
const void* walker_symbol_f64_2d(int geom, int mode);
const void* walker_symbol_f64_3d(int geom, int mode);
// Bytes of the scratch array of wos_solve_static, one copy per GPU.
constexpr size_t kStaticScratchBytes = 128ull << 20;
// Device address of `device`'s copy of that array (looked up on the first call for the
// device, with the device current, and kept).
hipError_t static_scratch(int device, void** ptr);
// 0 delta tracking, 1 delta tracking with splitting or gradient records, 2 next flight
int walker_mode(int variant, bool grad, bool split);
const void* walker_symbol(int fp64, int dim, int geom, int mode);
// Per-point sums of the items from their slots, added into the items' outputs (n_blocks: blocks
// of kReducePoints points from block0 on, each item its own; no two items share outputs).
constexpr int kReducePoints = 256;
hipError_t launch_reduce(int grad_dim, const DevItem* items, int n_items, uint64_t block0, uint64_t n_blocks,
                         const uint64_t* slots, int slot_words, hipStream_t st);
// Zeroes n words at p and the tile counters (a kernel, so that it can sit in a captured graph).
hipError_t launch_clear(uint64_t* p, uint64_t n, uint32_t* counters, hipStream_t st);
hipError_t launch_finalize_components(const double* sum, const double* sum_sq, const uint64_t* nw, int64_t n, int dim,
                                      double* mean, double* se, hipStream_t st);
hipError_t launch_set_params(LaunchParams* lp, uint64_t seed, uint64_t walk_offset_add, hipStream_t st);
hipError_t launch_classify(int dim, int geom, const void* P64, const double* pts, int64_t n, int8_t* inside,
                           hipStream_t st);
// Samples sigma' over the interior ones of cell centres first .. first + n - 1 of a grid
// (`inside`: n bytes of scratch).
hipError_t launch_sigma_sample(int dim, int geom, const void* P64, const double* lo, const double* h, int grid,
                               int64_t first, int64_t n, int nblocks, int8_t* inside, double* out, hipStream_t st);
// Candidate grid of a polygon (P64: the problem on the device with its BVH, of so many levels):
// squared centre distances and list starts of the cells, the total of the list lengths
// (total[0]) and the number of truncated lists (total[1]; sums: scan_sum_words(cells) words of
// scratch), then the lists and records.
size_t scan_sum_words(int64_t cells);
hipError_t launch_segment_count(int depth, const void* P64, const GridShape& s, const GridRule& rule, double* best,
                                uint32_t* count, uint32_t* sums, uint32_t* start, uint32_t* total, hipStream_t st);
hipError_t launch_segment_fill(int depth, const void* P64, const GridShape& s, const GridRule& rule, const double* best,
                               const uint32_t* start, const GridOut& out, hipStream_t st);
// The same for a mesh, whose records hold their lists.
hipError_t launch_mesh_cells(int depth, const void* P64, const GridShape& s, const GridRule& rule, double* best,
                             const GridOut& out, uint32_t* total, hipStream_t st);
// The class of every cell of a closed boundary (reach: centre distance up to which a
// primitive may touch the cell; label, roots: one word per cell of scratch).
hipError_t launch_cell_classes(int dim, const void* P64, const GridShape& s, double reach, const double* best,
                               uint32_t* label, uint32_t* roots, uint32_t* n_roots, uint8_t* cls, hipStream_t st);
// Row lists of the cells of an SDF domain (scale: largest coordinate of its box).
hipError_t launch_sdf_cells(int dim, const void* P64, const GridShape& s, double scale, uint64_t* cells, hipStream_t st);
// Prepares a job: classifies the query points (counters[0] of their item counts those outside),
// evaluates gamma at the interior ones in the walker's precision, writes the item table and the
// launch parameters, and clears the accumulation slots and tile counters. Sets block0.
hipError_t launch_prep(int fp64, int dim, int geom, PrepArgs& a, hipStream_t st);
hipError_t launch_coefficients(int fp64, int dim, const void* P, const double* pts, int64_t n, double* out,
                               hipStream_t st);
hipError_t launch_distance(int fp64, int dim, int geom, const void* P, const double* pts, int64_t n, double* d,
                           double* xb, hipStream_t st);
hipError_t launch_ball(int fp64, int dim, const double* s, int64_t n, double* out, hipStream_t st);
hipError_t launch_sample(int fp64, int dim, double s, int64_t n, uint64_t seed, double* t, uint64_t* trials,
                         hipStream_t st);
hipError_t launch_philox(const uint32_t* ctr, uint64_t key, int64_t n, uint32_t* out, hipStream_t st);
hipError_t launch_bessel(int fp64, int which, const double* x, int64_t n, double* out, hipStream_t st);
hipError_t launch_offcentred(int fp64, int dim, int which, double R, double sigma_bar, const double* u,
                             const double* v, int64_t n, double* out, hipStream_t st);
hipError_t launch_finalize(const double* sum, const double* sum_sq, const uint64_t* nw, int64_t n, double* mean,
                           double* se, hipStream_t st);

}  // namespace wos
