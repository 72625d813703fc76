// The gridded form of the patch: host plan and launchers (k_grid.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "psf_kernels.hpp"

namespace psf {

// Grid of one patch, in cells along the row and column axes (powers of two).
// ml = 0: the patch takes the dense contraction.
struct GridPlan {
  int ml = 0, mm = 0;
};

// Cells per axis of a patch of n pixels: the smallest power of two (at least
// 32) that oversamples it by 1.96 or more; 0 if that exceeds kGridMaxAxis.
constexpr int kGridMaxAxis = 2048;
int grid_axis(int n);
// Bytes of one source's grid, half-transformed grid and state, and what
// aligning them takes: the cells are summed by 64-bit atomics, while a
// caller's workspace may begin anywhere.
constexpr size_t kGridAlign = 16;
size_t grid_bytes(const GridPlan& g, int nm);

struct UvGridScale;  // what scales a source's fixed point (k_grid.hip)

// Per-source part of a gridded launch; direction and grid as in SrcPlan.
// Fused launches form the decorrelation factors from the observation; others
// read records and coefficients.
struct UvGridSrc {
  const BinRec* rec;
  const float2* c;
  uint8_t* work;  // cells, half-transformed grid, state (aligned to kGridAlign, within grid_bytes)
  float* P;
  const double* peak;  // not fused: see SrcPlan
  const double* dir;
  UvGridScale* scale;  // filled by launch_grid
  double l0, m0, l_first, m_first, dl, dm;
  int nl, nm;
  int norm;  // fused: divide by 2 sum Re c, summed here
};

constexpr int kGridMaxSpans = 4608;  // spans of bins per source

struct UvGridArgs {
  ObsView o;
  int n_src;
  int ml, mm;  // cells per axis (every source of the launch)
  int fused;
  // filled by launch_grid: spreading workgroups, levels and number of their
  // spans (per source), init blocks; bins of the shortest span where all bins
  // cost the same
  int n_wg, levels, n_span, n_init;
  int64_t unit_bins;
  UvGridSrc src[kMaxBatch];
};

// Clears the grids, finds the scale, spreads the bins, transforms and writes
// the patches of every source of `a`.
hipError_t launch_grid(int prec, UvGridArgs a, hipStream_t stream);

}  // namespace psf
