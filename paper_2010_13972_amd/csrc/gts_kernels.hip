// Launch planning and the device entry points of libgts (gts_shap,
// gts_shap_interactions, gts_launch_config).  The kernels themselves are in
// gts_shap_kernel.h, instantiated by gts_shap_f32.hip, gts_shap_f64.hip,
// gts_inter_f32.hip and gts_inter_f64.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <numeric>
#include <vector>

#include "gts_launch.h"
#include "gts_shap_kernel.h"

namespace gts {
namespace {

struct DeviceInfo {
  int cus = 256;
  int lds_per_block = 64 * 1024;
  int lds_per_cu = 160 * 1024;
};

DeviceInfo device_info() {
  static std::mutex mu;
  static std::vector<DeviceInfo> cache;
  static std::vector<char> have;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return DeviceInfo{};
  std::lock_guard<std::mutex> lock(mu);
  if ((int)cache.size() <= dev) {
    cache.resize(dev + 1);
    have.resize(dev + 1, 0);
  }
  if (!have[dev]) {
    DeviceInfo info;
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      info.cus = n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess &&
        n > 0)
      info.lds_per_block = n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) ==
            hipSuccess &&
        n > 0)
      info.lds_per_cu = n;
    info.lds_per_cu = std::max(info.lds_per_cu, info.lds_per_block);
    cache[dev] = info;
    have[dev] = 1;
  }
  return cache[dev];
}

inline int odd_at_least(int n) { return n | 1; }

// Interaction values of paths of 9 to 16 features: the quadrature kernel, on the
// largest tile of 16, 8 or 4 rows in double a workgroup's LDS holds, or, in fp32
// models beyond 78 features, of 8 or 4 rows in float (200 rows of 100 trees of depth
// 14: M = 82, 8 rows in float 1.22 ms, 4 in double, with 8 waves, 1.45); false where
// none fits (beyond M = 118, fp64 81: then the runtime-length code runs, as for longer
// paths).  Slices: at most one round of workgroups.
template <typename T>
bool plan_quad(const gts_model* m, int64_t rows, const DeviceInfo& dev, Plan& plan) {
  const int q = m->max_path_len - 1;
  if (q <= kMaxUnrolledInter || q > kMaxUnrolledQuad) return false;
  const int M = m->num_features, G = m->num_groups;
  auto lds = [&](int rw, int waves, bool wide) {
    return sizeof(T) == 8 ? quad_lds_f64(M, rw, waves, true) : quad_lds_f32(M, rw, waves, wide);
  };
  struct Shape {
    int rw, waves;
    bool wide;   // tile in double (always for fp64 models)
  };
  constexpr Shape f32[] = {{16, 16, true}, {8, 16, true},  {4, 16, true},
                           {8, 12, false}, {4, 16, false}, {4, 8, false}};
  constexpr Shape f64[] = {{16, 8, true}, {8, 8, true}, {4, 8, true}};
  plan.RW = 0;
  for (int i = 0; i < (sizeof(T) == 8 ? 3 : 6) && plan.RW == 0; ++i) {
    const Shape& x = sizeof(T) == 8 ? f64[i] : f32[i];
    if ((int64_t)lds(x.rw, x.waves, x.wide) + kQuadStaticLds > dev.lds_per_block) continue;
    plan.RW = x.rw;
    plan.waves = x.waves;
    plan.wide_tile = x.wide;
  }
  if (plan.RW == 0) return false;
  plan.quad = true;
  plan.priv = false;
  plan.lds = lds(plan.RW, plan.waves, plan.wide_tile);
  plan.sx = odd_at_least(M);
  plan.width = (M + 1) * (M + 1);
  plan.tiles = (rows + plan.RW - 1) / plan.RW;
  const int64_t base = plan.tiles * G;
  // a CU holds one workgroup: 16 waves of 98 to 128 registers, 12 of 168, or 8 of 150
  // and more; a second round of slices adds its tiles for nothing (M = 24, 200 trees,
  // 40 rows: 85 slices 115 us, 170 135, 341 178; fp64, M = 12, 5 rows: 256 slices 62 us,
  // 569 85)
  const int64_t round = dev.cus;
  plan.splits = (int)std::max<int64_t>(
      1, std::min<int64_t>(round / base, std::max<int64_t>(1, m->num_bins / G / plan.waves)));
  plan.min_splits = plan.splits;
  return true;
}

template <typename T, bool INTER>
gts_status plan_launch(const gts_model* m, int64_t rows, const DeviceInfo& dev, Plan& plan) {
  const int M = m->num_features;
  const int G = m->num_groups;
  const int64_t width64 = INTER ? (int64_t)(M + 1) * (M + 1) : (int64_t)(M + 1);
  if (width64 > (1 << 30)) return fail(GTS_EINVAL, "M = %d is too large", M);
  if constexpr (INTER) {
    if (plan_quad<T>(m, rows, dev, plan)) return GTS_OK;
  }
  const int32_t width = (int32_t)width64;
  const int32_t sx = odd_at_least(M);
  // interactions keep the upper triangle of each row's block in LDS
  const int32_t sp = odd_at_least(INTER ? (int32_t)((int64_t)(M + 1) * (M + 2) / 2) : width);
  // Row tile and accumulation.  If 64 rows with a private phi tile for each
  // of 4 waves fit in 64 KB of LDS, use them (no contention, no atomics).
  // Otherwise the waves of a workgroup share one tile.
  const int longest = std::max(0, m->max_path_len - 1);
  auto need = [&](int rw, int waves, bool priv, bool wide) {
    const size_t entry = wide ? sizeof(double) : sizeof(T);
    const size_t tiles = (size_t)rw * ((size_t)sx * sizeof(float) +
                                       (priv ? (size_t)waves : 1) * (size_t)sp * entry);
    const size_t stage = rw == 64 ? sizeof(Stage<T, false>) : sizeof(Stage<T, true>);
    return ((tiles + 15) & ~(size_t)15) + (size_t)waves * stage;
  };
  int RW = 0;
  int waves = 8;
  bool priv = false;
  bool wide = false;
  constexpr int64_t kSmallTile = 64 * 1024;  // leaves room for several workgroups per CU
  constexpr int64_t kHalfCu = 80 * 1024;     // two workgroups per CU
  const int64_t whole = dev.lds_per_block;
  // takes the shape where it fits and none is taken yet
  auto take = [&](int rw, int w, bool in_double, int64_t budget) {
    if (RW != 0 || (int64_t)need(rw, w, false, in_double) > std::min(budget, whole)) return;
    RW = rw;
    waves = w;
    wide = in_double;
  };
  if ((int64_t)need(64, 4, true, false) <= std::min(kSmallTile, whole)) {
    RW = 64;
    waves = 4;
    priv = true;
  } else if (INTER) {
    // Interaction values: 8 waves on the largest tile of 64 KB; else 16 (the
    // kernel's registers allow one workgroup of them per CU) on the largest of 16,
    // 8 or 4 rows a workgroup's LDS holds.
    for (int rw : {64, 32, 16, 8}) take(rw, 8, false, kSmallTile);
    for (int rw : {16, 8, 4}) take(rw, 16, false, whole);
    take(4, 8, false, whole);
  } else {
    // SHAP values: the largest tile of which a CU holds two, in double also for fp32
    // models (native adds).  8 waves, or 12 for short fp32 paths on 64 rows, whose 64
    // registers leave room for 24 waves a CU.  fp64 kernels of short paths have 110, for
    // 16 waves: 8 there (3000 rows of 100 trees, M = 45: 8 waves 111 us, 12 131), and 32
    // rows from 70 KB on (M = 69), for the sake of small batches (M = 75, 60 rows: 21 us
    // against 29 with 64; 5000 rows: 433 against 359).
    constexpr bool kWide = sizeof(T) == 4;
    const bool is_short = longest <= kQShort;
    if (kWide && is_short) take(64, 12, kWide, kHalfCu);
    take(64, 8, kWide, kWide || !is_short ? kHalfCu : 70 * 1024);
    // The doubles' size alone would halve the rows, and with 64 of them lose the
    // one-path form, of fp32 models whose tile in float takes 64 KB: one workgroup of
    // 16 waves keeps them (10 000 rows, 64 rows against 32: M = 95, paths of 8
    // features, 303 us against 342, of 11 1029 against 1161; 32 against 16: M = 180,
    // of 11 1286 against 1729, of 16 1832 against 2395; 16 rows of short paths run
    // 24 waves a CU and win there, 355 against 430; 16 against 8: M = 373, of 16 2619
    // against 2842, of 11 2034 against 1973).  64 and 32 rows not for paths beyond 16
    // features, whose loops are faster on fewer: M = 95, 3000 rows, 64 rows 4.75 ms, 32
    // 3.91 (M = 350, 16 rows 4.7, 8 8.9).
    const bool unrolled = longest <= kMaxUnrolledExt;
    if (kWide && unrolled && (int64_t)need(64, 8, false, false) <= kSmallTile)
      take(64, 16, true, whole);
    take(32, 8, kWide, kHalfCu);
    if (kWide && unrolled && !is_short && (int64_t)need(32, 8, false, false) <= kSmallTile)
      take(32, 16, true, whole);
    // Short fp32 paths: 24 waves a CU on as many rows as two workgroups of 12 hold in
    // double, 16 to M = 287, then 8 to 576 (100 trees of depth 8, 10 000 rows: M = 333,
    // 8 rows 446 us, 16 rows of which a CU holds one workgroup 505; M = 373, 436, 8 rows in
    // float 558; 16 rows in float 441 and 439).
    if (kWide && is_short) take(16, 12, true, kHalfCu);
    if (kWide && is_short) take(8, 12, true, kHalfCu);
    // At equal waves a CU the larger workgroup, here and below: it needs fewer slices, and
    // every slice adds its tile to phi.  Few row tiles gain (fp64, M = 160, paths of 8, 60
    // rows: one of 16 waves 15.4 us, two of 8 18.7), many would be faster with two (fp32,
    // M = 300, of 11, 10 000 rows, 16 rows: 1849 and 1611 us; fp64, M = 300, of 6, 5000
    // rows: 135 and 109), but fp32 sums of 40 slices instead of one would be 1.2 times as
    // far from fp64 values.
    // Longer fp32 paths, whose registers hold a CU to 16 waves: 16 rows of which a CU
    // holds two tiles, else 8, in double (784 features, paths of up to 16, 3000 rows: 0.55
    // against 0.78 ms in float), also of 12 waves (M = 1400: 16 in float at the same time,
    // 1.1 times as far from fp64 values), else in float, before fewer waves (700 rows of 60
    // trees, M = 1800: 16 waves 0.16 ms, 8 0.35), and 4 rows.
    if (kWide && !is_short) {
      if ((int64_t)need(16, 8, false, true) <= kHalfCu ||
          (longest > kQMid && (int64_t)need(16, 8, false, false) <= kSmallTile))
        take(16, 16, true, whole);
      for (int w : {16, 12}) take(8, w, true, whole);
      for (int rw : {8, 4})
        for (int w : {16, 12, 8}) take(rw, w, false, whole);
    }
    // The others: the rows of which a CU holds two tiles, and as many waves a CU as the
    // LDS allows in whole workgroups, up to what the registers of the variant allow: 24
    // (77 of them, fp32, short paths; in float, 10 classes, 784 features: 6.5 ms, in
    // double 7.0), one workgroup (fp64, longer ones: 177 and more for 8 waves, 168 for
    // 12, 128 for 16), else 16.
    if (RW == 0) {
      if (!kWide) take(16, 8, false, kHalfCu);
      take(8, 8, false, kHalfCu);
      take(8, 8, false, whole);
      take(4, 8, false, whole);
      int best = 0;
      for (int w : {16, 12, 8}) {
        // 16 waves leave 128 registers, and fp64 paths of 11 features and more spill
        // there: 3000 rows of 100 trees, 12 waves against 16, of 12 features 1.19 against
        // 1.69 ms (M = 300), of 16 1.98 against 3.20 (M = 635); of 10, 0.75 against 0.68
        if (RW == 0 || (w == 16 && !kWide && longest > 10)) continue;
        const int64_t n = need(RW, w, false, false);
        if (n > whole) continue;
        const int groups = !is_short ? 1 : (kWide ? 24 : 16) / w;
        const int per_cu = w * (int)std::min<int64_t>(groups, dev.lds_per_cu / n);
        if (per_cu > best) {
          best = per_cu;
          waves = w;
        }
      }
    }
  }
  if (RW == 0) return fail(GTS_EINVAL, "M = %d needs more LDS than a workgroup has", M);
  size_t lds = need(RW, waves, priv, wide);
  // rank tables for the bin-wide dead-pair test of one-path-per-wave launches
  size_t rank_off = 0;
  if (RW == 64 && priv && M <= kRankMaxM) {
    rank_off = (lds + 7) & ~(size_t)7;
    lds = rank_off + rank_table_bytes(M);
  }
  // Bin slices per (row tile, group) when there are too few tiles to fill
  // the GPU.  Every slice adds its tile to phi atomically, so a slice costs
  // rows x width atomic adds.  SHAP values (short phi rows): enough
  // workgroups for two rounds of every CU at the occupancy the LDS allows,
  // or more, up to 128 slices, while every wave still gets 8 bins or more
  // (finer slices even out the last rounds); (group, slice) units a multiple
  // of the 8 XCDs.  Interaction values ((M+1)^2 per row): at most one round,
  // since there the adds outweigh the balance.
  const int64_t tiles = (rows + RW - 1) / RW;
  const int64_t base = tiles * G;
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(8, dev.lds_per_cu / (int64_t)lds));
  const int64_t bins_per_group = std::max<int64_t>(1, m->num_bins / G);
  int splits = 1;
  int min_splits = 1;
  int split_step = 1;
  if constexpr (INTER) {
    const int64_t round = per_cu * dev.cus;
    if (2 * base <= round)
      splits = (int)std::max<int64_t>(1, std::min<int64_t>(round / base, bins_per_group));
    min_splits = splits;
  } else {
    const int64_t target = 2 * per_cu * dev.cus;
    if (base < target) {
      int64_t want = (target + base - 1) / base;
      // A slice with little to do spends its time on its tiles: with fewer than
      // 4 bins a wave, one round of workgroups, of at least 4 bins each (100 trees
      // of depth 8 over 54 features: 1 row 128 slices 13.8 us, 1024 34.7; 200 rows
      // 128 18.7, 256 28.2; 1000 rows 32 32.8, 64 37.2), unless a wave then has two, which
      // takes twice as long (13 rows, 6 bins for 4 waves: 1 slice 16.8 us, 6 12.4), as long
      // as that leaves no CU with two workgroups (fp64, 10 000 rows, 5 bins: 1 slice 15.1, 5
      // 19.5).  Of several groups some have more than the mean: for twice as many (9 rows,
      // 10 groups of 21 bins: 8 slices 15.5, 12 11.3).  Fewer bins than waves are best in
      // one slice, which needs no clearing of phi: 9.3 and 12.2.
      if (bins_per_group < 4 * want * waves) {
        int64_t single = 1;
        if (G == 1 || bins_per_group >= waves)
          single = ((G == 1 ? 1 : 2) * bins_per_group + waves - 1) / waves;
        single = std::min(single, dev.cus / base);
        want = std::min(std::max<int64_t>(1, target / 2 / base),
                        std::max<int64_t>({1, single, bins_per_group / 4}));
      }
      const int64_t step = 8 / std::gcd(G, 8);
      if (want > 1) want = (want + step - 1) / step * step;
      const int64_t fine = std::min<int64_t>(128, bins_per_group / (8 * waves)) / step * step;
      min_splits = (int)std::max<int64_t>(1, std::min<int64_t>(want, bins_per_group));
      want = std::max(want, fine);
      splits = (int)std::max<int64_t>(1, std::min<int64_t>(want, bins_per_group));
      split_step = (int)step;
    }
    min_splits = std::min(min_splits, splits);
  }
  if (rank_off != 0 && !ranks_pay(M, bins_per_group, (int64_t)splits * waves)) {
    rank_off = 0;
    lds = need(RW, waves, priv, wide);
  }
  plan.RW = RW;
  plan.waves = waves;
  plan.priv = priv;
  plan.wide_tile = wide;
  plan.sx = sx;
  plan.sp = sp;
  plan.width = width;
  plan.lds = lds;
  plan.rank_off = rank_off;
  plan.splits = splits;
  plan.min_splits = min_splits;
  plan.split_step = split_step;
  plan.tiles = tiles;
  // the kernel variant: the model's longest path, in features
  plan.qmax = longest <= kQShort ? kQShort
              : (!INTER && longest <= kMaxUnrolledShap) ? kQMid
              : (!INTER && longest <= kMaxUnrolledExt) ? kQExt
                                                           : kQLong;
  return GTS_OK;
}

gts_status launch(const gts_model* m, const void* blob, const float* X, int64_t rows,
                  int64_t ld, void* phi, void* stream, bool inter) {
  Plan plan;
  const DeviceInfo dev = device_info();
  gts_status st;
  if (m->dtype == GTS_F64)
    st = inter ? plan_launch<double, true>(m, rows, dev, plan)
               : plan_launch<double, false>(m, rows, dev, plan);
  else
    st = inter ? plan_launch<float, true>(m, rows, dev, plan)
               : plan_launch<float, false>(m, rows, dev, plan);
  if (st != GTS_OK) return st;
  const KernelArgs a{m, blob, X, rows, ld, phi, stream};
  if (plan.quad)
    return m->dtype == GTS_F64 ? launch_inter_quad_f64(a, plan) : launch_inter_quad_f32(a, plan);
  if (m->dtype == GTS_F64) return inter ? launch_inter_f64(a, plan) : launch_shap_f64(a, plan);
  return inter ? launch_inter_f32(a, plan) : launch_shap_f32(a, plan);
}

gts_status entry(const gts_model* model, const void* d_model, const float* d_X, int64_t rows,
                 int64_t ld_x, void* d_phi, void* stream, bool inter) {
  clear_error();
  gts_status st = check_model(model);
  if (st != GTS_OK) return st;
  if (rows < 0) return fail(GTS_EINVAL, "rows must be >= 0");
  if (rows == 0) return GTS_OK;
  if (d_model == nullptr || d_X == nullptr || d_phi == nullptr)
    return fail(GTS_EINVAL, "device pointers must not be NULL");
  if (ld_x < model->num_features) return fail(GTS_EINVAL, "ld_x < num_features");
  return launch(model, d_model, d_X, rows, ld_x, d_phi, stream, inter);
}

}  // namespace
}  // namespace gts

extern "C" gts_status gts_launch_config(const gts_model* model, int64_t rows,
                                        int32_t interactions, gts_launch* out) {
  using namespace gts;
  clear_error();
  if (out == nullptr) return fail(GTS_EINVAL, "out must not be NULL");
  gts_status st = check_model(model);
  if (st != GTS_OK) return st;
  if (rows < 0) return fail(GTS_EINVAL, "rows must be >= 0");
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return fail(GTS_EDEVICE, "no HIP device");
  Plan plan;
  const DeviceInfo info = device_info();
  const int64_t r = rows > 0 ? rows : 1;
  if (model->dtype == GTS_F64)
    st = interactions ? plan_launch<double, true>(model, r, info, plan)
                      : plan_launch<double, false>(model, r, info, plan);
  else
    st = interactions ? plan_launch<float, true>(model, r, info, plan)
                      : plan_launch<float, false>(model, r, info, plan);
  if (st != GTS_OK) return st;
  out->rows_per_tile = plan.RW;
  out->waves = plan.waves;
  out->private_tiles = plan.priv ? 1 : 0;
  out->slices = plan.splits;
  out->workgroups = rows > 0 ? plan.tiles * model->num_groups * plan.splits : 0;
  out->lds_bytes = (int64_t)plan.lds;
  return GTS_OK;
}

extern "C" gts_status gts_shap(const gts_model* model, const void* d_model, const float* d_X,
                               int64_t rows, int64_t ld_x, void* d_phi, void* stream) {
  return gts::entry(model, d_model, d_X, rows, ld_x, d_phi, stream, false);
}

extern "C" gts_status gts_shap_interactions(const gts_model* model, const void* d_model,
                                            const float* d_X, int64_t rows, int64_t ld_x,
                                            void* d_phi, void* stream) {
  return gts::entry(model, d_model, d_X, rows, ld_x, d_phi, stream, true);
}
