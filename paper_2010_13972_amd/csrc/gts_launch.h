// Launch plan shared by the planner (gts_kernels.hip) and the translation
// units that instantiate the SHAP kernels (gts_shap_f32.hip and friends).
// Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "gts_internal.h"

namespace gts {

// Longest path (features) with fully unrolled per-path code.  Longer paths
// run the runtime-loop code, in fp64, which keeps its per-path arrays in
// per-lane private memory; only the long-path kernel variants contain it.
constexpr int kMaxUnrolledShap = 12;
constexpr int kMaxUnrolledInter = 8;
// SHAP paths of 13-16 features run unrolled code in a variant of their own, since
// they need more registers.
constexpr int kMaxUnrolledExt = 16;

// Interaction values of paths of up to 16 features run by quadrature where the
// model has longer ones than the unrolled code takes.
constexpr int kMaxUnrolledQuad = 16;
constexpr int64_t kQuadStaticLds = 640;   // that kernel's static LDS, rounded up

// Kernel variant by the model's longest path: every path has at most 8
// features, at most 12, at most 16 (SHAP values only), or any length up to a
// full bin (63).
constexpr int kQShort = 8;
constexpr int kQMid = 12;
constexpr int kQExt = 16;
constexpr int kQLong = 64;

// The shared-tile launch shapes of a kernel variant that the planner gives: rows,
// waves, and whether the tile holds doubles whatever the model's type.
constexpr bool has_shape(bool f64, bool inter, int qmax, int rw, int waves, bool wide) {
  if (inter) return !wide && (waves == 8 || (waves == 16 && rw <= 16));
  const bool longer = qmax > kQShort;
  if (f64) {
    if (wide) return false;
    if (rw > 16) return waves == 8;
    if (waves == 16) return qmax <= kQMid;
    return rw < 16 || (waves == 12 && longer);
  }
  if (rw == 64) return wide && (waves == 8 || (waves == 12 && !longer) || (waves == 16 && qmax <= kQExt));
  if (rw == 32) return wide && (waves == 8 || (waves == 16 && longer && qmax <= kQExt));
  if (rw == 16) return wide && waves == (longer ? 16 : 12);
  if (rw == 8) return !wide || waves == 12 || (waves == 16 && longer);
  return !wide;
}

// Private-tile launches (64-row tiles, one path per wave) of models with at
// most this many features, and bins enough for every wave, keep rank tables of the
// row tile in LDS: per feature, the 64 row keys in ascending order and, for every
// rank, the mask of the rows below it.  They serve the dead-pair test of a whole bin
// at once.
constexpr int kRankMaxM = 16;
// Whether the tables pay.  They cost a workgroup about 0.7 us and 780 B of LDS a
// feature, and serve only models with zero fractions; without them the per-path test
// finds the dead paths.  Measured with and without on 64 to 100 000 rows of models
// with zero covers (20 to 1000 trees of depth 6 to 16), they pay from 2.5 bins a wave on at
// 4 features, 4 at 6, 6.5 at 8, 9.5 at 10, 18 at 12 and 14, 20 at 16: M = 8, 1000 trees, 5.9
// bins a wave 40.5 us with, 38.6 without, 7.1 77.7 and 82.8, 53 297 and 486; M = 16, 10.8
// 124 and 108, 29 231 and 258.
constexpr bool ranks_pay(int M, int64_t bins, int64_t waves) {
  return 10 * bins >= std::max(M * M, 25) * waves;
}
inline size_t rank_table_bytes(int M) {
  return (size_t)M * 65 * (sizeof(uint64_t) + sizeof(int32_t));
}

// The launch shape of a model and row count: rows per tile, waves, private
// tiles, LDS strides and bytes, bin slices, and the kernel variant.
struct Plan {
  int RW = 0;
  int waves = 8;
  bool priv = false;
  int32_t sx = 0, sp = 0, width = 0;
  size_t lds = 0;
  int splits = 1;
  int min_splits = 1;    // slices enough for the occupancy target alone
  int split_step = 1;    // slice counts are multiples of this (XCD balance)
  int64_t tiles = 0;
  int qmax = kQLong;
  size_t rank_off = 0;   // LDS offset of the rank tables (0: none)
  bool quad = false;     // interactions by quadrature (gts_inter_quad.h)
  bool wide_tile = false;   // the tile in double for an fp32 model
};

// A grid of `total` workgroups.  A launch has fewer than 2^32 work-items in each
// dimension, so the workgroups beyond go to further rows of the grid: workgroup b is
// blockIdx.y * gridDim.x + blockIdx.x, and those from total on (the last row's end)
// leave at once.
constexpr int64_t kMaxWorkItems = 0xffffffffll;
inline dim3 grid_of(int64_t total, int threads) {
  const int64_t x = std::max<int64_t>(1, std::min<int64_t>(total, kMaxWorkItems / threads));
  return dim3((unsigned)x, (unsigned)((total + x - 1) / x));
}

// Arguments of one gts_shap / gts_shap_interactions call.
struct KernelArgs {
  const gts_model* m;
  const void* blob;
  const float* X;
  int64_t rows;
  int64_t ld;
  void* phi;
  void* stream;   // hipStream_t
};

// One launcher per (dtype, kind); each lives in its own translation unit so
// the kernel variants compile in parallel.
gts_status launch_shap_f32(const KernelArgs& a, const Plan& p);
gts_status launch_shap_f64(const KernelArgs& a, const Plan& p);
gts_status launch_inter_f32(const KernelArgs& a, const Plan& p);
gts_status launch_inter_f64(const KernelArgs& a, const Plan& p);
gts_status launch_inter_quad_f32(const KernelArgs& a, const Plan& p);
gts_status launch_inter_quad_f64(const KernelArgs& a, const Plan& p);
// LDS of a workgroup of the quadrature kernel.
size_t quad_lds_f32(int M, int rows, int waves, bool wide);
size_t quad_lds_f64(int M, int rows, int waves, bool wide);

}  // namespace gts
