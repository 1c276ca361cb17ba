// SHAP interaction values of models whose longest path holds 9 to 16 features,
// for gfx950 (CDNA4, wave64); included by the translation units that
// instantiate the kernel (gts_inter_quad_f32.hip, gts_inter_quad_f64.hip).
//
// The Shapley weights are Beta integrals: with a_k(t) = z_k (1 - t) + o_k t, the
// value of a path's element i (Eq. 2) and the interaction of i and j (Eq. 4-5) are
//   phi_i    = v   integral over [0, 1] of (o_i - z_i) prod_{k != i} a_k
//   Delta_ij = v/2 integral over [0, 1] of (o_i - z_i)(o_j - z_j) prod_{k != i,j} a_k
// polynomials of degree q - 1 and q - 2, which N = 4 (q <= 8) or 8 (q <= 16)
// Gauss-Legendre nodes integrate exactly.  At a node no factor is negative and
// every a_k of a contributing path is positive, so with P = weight v prod a_k and
// rho_k = (o_k - z_k) / a_k
//   phi_i = sum_n P rho_i,   Delta_ij = 1/2 sum_n P rho_i rho_j,
//   phi_ii = phi_i - sum_{j != i} Delta_ij = sum_n P rho_i (1 - (R - rho_i) / 2),
// R = sum_k rho_k: one multiply-add per pair and node.  (The packed-path kernel
// of gts_shap_kernel.h unwinds the path polynomial for every pair, with runtime
// loops over arrays in private memory beyond 8 features: 10.9 ms for 200 rows of
// 100 trees of depth 16 over 54 features, fp32, against 0.29 ms here.  Up to 8
// features its unrolled code is the faster one: 0.29 against 1.0 ms for 1000 rows
// of 100 trees of depth 8 over 54 features.)
//
// Lanes.  A wave takes one path for RW rows; LPR neighbouring lanes share a row
// and hold NPL = N / LPR nodes each.  The LPR lanes' partial sums of LPR entries
// are exchanged by DPP so that every lane ends with one whole entry, and all 64
// lanes add to the tile at once.  VALU issue bounds it (about 80 % of the SIMD
// cycles at the size above), the pairs' multiply-adds and exchanges most of it.
//
// Tile.  A is the type of the tile's entries.  gfx950 adds doubles in LDS
// natively (ds_add_f64, about 8 cycles per wave instruction and CU, no result to
// wait for), floats only by compare-and-swap at a useful rate (14 cycles and a
// round trip of 200; ds_add_f32: 192 cycles).  So an fp32 model's tile is in
// double where 16 rows of it fit in LDS (M <= 38 or so); 8 rows in double
// instead of 16 in float lose more than the adds gain (0.33 against 0.29 ms at
// M = 54).
#pragma once

#include "gts_shap_kernel.h"

namespace gts {
namespace {

constexpr int kQuadMaxQ = 16;
constexpr int kQuadItems = kQuadMaxQ * (kQuadMaxQ + 1) / 2;   // entries of one path

// Gauss-Legendre nodes and weights on [0, 1] for N = 4 and 8.
__device__ const double kNodeT[2][8] = {
    {0.069431844202973712388, 0.33000947820757186760, 0.66999052179242813240,
     0.93056815579702628761},
    {0.019855071751231884158, 0.10166676129318663020, 0.23723379504183550709,
     0.40828267875217509753, 0.59171732124782490247, 0.76276620495816449291,
     0.89833323870681336980, 0.98014492824876811584}};
__device__ const double kNodeW[2][8] = {
    {0.17392742256872692869, 0.32607257743127307131, 0.32607257743127307131,
     0.17392742256872692869},
    {0.050614268145188129576, 0.11119051722668723527, 0.15685332293894364367,
     0.18134189168918099148, 0.18134189168918099148, 0.15685332293894364367,
     0.11119051722668723527, 0.050614268145188129576}};

// Per wave in LDS: the bin, and the tile entry of every pair of its current path.
template <typename T>
struct QuadStage {
  Stage<T, false> bin;
  int entry[kQuadItems];
};

__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// The value of the lane that DPP pattern C names.
template <int C>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), C, 0xf, 0xf, true));
}
template <int C>
__device__ __forceinline__ double dpp(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)b, C, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(b >> 32), C, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over the LPR lanes of a row of the LPR values v[0..LPR): lane g of the row
// gets the sum of v[g].  Neighbours swap the halves they do not keep.
template <int LPR, typename T>
__device__ __forceinline__ T scatter_sum(const T (&v)[LPR], int g) {
  static_assert(LPR == 4 || LPR == 8, "a row has four or eight lanes");
  T x[LPR / 2];
#pragma unroll
  for (int i = 0; i < LPR / 2; ++i) {
    const T mine = (g & 1) ? v[2 * i + 1] : v[2 * i];
    const T other = (g & 1) ? v[2 * i] : v[2 * i + 1];
    x[i] = mine + dpp<0xB1>(other);   // quad_perm 1,0,3,2
  }
  T y[LPR / 4];
#pragma unroll
  for (int i = 0; i < LPR / 4; ++i) {
    const T mine = (g & 2) ? x[2 * i + 1] : x[2 * i];
    const T other = (g & 2) ? x[2 * i] : x[2 * i + 1];
    y[i] = mine + dpp<0x4E>(other);   // quad_perm 2,3,0,1
  }
  if constexpr (LPR == 4) {
    return y[0];
  } else {
    const T mine = (g & 4) ? y[1] : y[0];
    const T other = (g & 4) ? y[0] : y[1];
    // row_shl / row_shr by 4: the lane four up or four down in its row of 16
    const T up = dpp<0x104>(other), down = dpp<0x114>(other);
    return mine + ((g & 4) ? down : up);
  }
}

template <typename T, int NPL>
struct Nodes {
  bool row;   // the lane has a row
  T t[NPL], c[NPL], k[NPL], w[NPL];   // node, 1 - node, its reciprocal, weight
};

// One path (root in slot s, q features, padded to Q) for the wave's rows.
template <typename T, typename A, int Q, int NPL, int LPR, int STRIDE>
__device__ __forceinline__ void quad_path(QuadStage<T>* st, int s, int q, const Nodes<T, NPL>& nd,
                                          const int* __restrict__ xrow, A* __restrict__ tile,
                                          const unsigned short* __restrict__ pairs, int lane,
                                          int W) {
  const int g = lane % LPR;
  T P[NPL], R[NPL], rho[Q][NPL];
  const T v = st->bin.w(s);
#pragma unroll
  for (int n = 0; n < NPL; ++n) {
    P[n] = nd.w[n] * v;
    R[n] = T(0);
  }
  bool live = nd.row;
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    // past the path's end: z = 1 and present, a factor of 1 with rho = 0
    const bool real = k < q;
    const int e = s + (real ? 1 + k : 0);
    const int4 head = st->bin.head[e];
    const T z = real ? st->bin.z(e) : T(1);
    const bool o = !real || in_range(xrow[real ? head.x : 0], head.y, (unsigned)head.z);
    live &= o | (z != T(0));   // else a zero factor: the path leaves nothing here
    const T d = T(1) - z;
#pragma unroll
    for (int n = 0; n < NPL; ++n) {
      const T hi = fma(z, nd.c[n], nd.t[n]);
      const T a = o ? hi : z * nd.c[n];
      T r = d * recip(hi);
      keep(r);
      r = o ? r : -nd.k[n];
      P[n] *= a;
      R[n] += r;
      rho[k][n] = r;
    }
  }
  if (__ballot(live) == 0) return;

  // the tile entries of the path's pairs, item j (j + 1) / 2 + i for i <= j
  const int items = q * (q + 1) / 2;
  for (int m = lane; m < items; m += 64) {
    const int ij = pairs[m];
    const int fi = st->bin.head[s + 1 + (ij & 0xff)].x;
    const int fj = st->bin.head[s + 1 + (ij >> 8)].x;
    st->entry[m] = tri_at(fi, fj, W) * STRIDE;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  constexpr int kItems = Q * (Q + 1) / 2;
  constexpr int kGroups = (kItems + LPR - 1) / LPR;
  constexpr int kBatch = 6;   // adds in flight
  T part[LPR];
  A* p[kBatch];
  A val[kBatch];
  bool on[kBatch];
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    T u[NPL];
#pragma unroll
    for (int n = 0; n < NPL; ++n) u[n] = T(0.5) * P[n] * rho[j][n];
#pragma unroll
    for (int i = 0; i <= j; ++i) {
      const int m = j * (j + 1) / 2 + i;
      T x = T(0);
#pragma unroll
      for (int n = 0; n < NPL; ++n)
        x = fma(u[n], i < j ? rho[i][n] : T(2) - (R[n] - rho[j][n]), x);
      part[m % LPR] = x;
      if (m == kItems - 1) {
#pragma unroll
        for (int l = m % LPR + 1; l < LPR; ++l) part[l] = T(0);
      }
      if (m % LPR == LPR - 1 || m == kItems - 1) {
        const int grp = m / LPR;
        const int b = grp % kBatch;
        const int mine = grp * LPR + g;
        val[b] = (A)scatter_sum<LPR>(part, g);
        on[b] = live & (mine < items);
        p[b] = tile + (on[b] ? st->entry[mine] : 0);
        if (b == kBatch - 1 || grp == kGroups - 1) {
          if (grp == kGroups - 1) {
#pragma unroll
            for (int l = b + 1; l < kBatch; ++l) {
              p[l] = tile;
              val[l] = A(0);
              on[l] = false;
            }
          }
          if constexpr (sizeof(A) == 8) {
            // native, without a result to wait for
#pragma unroll
            for (int l = 0; l < kBatch; ++l)
              if (on[l])
                __hip_atomic_fetch_add(p[l], val[l], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
          } else {
            tile_add<kBatched>(p, val, on);
          }
        }
      }
    }
  }
  // the next path overwrites the entries
  __builtin_amdgcn_wave_barrier();
}

// One workgroup: rows [tile RW, tile RW + RW) of output group g, every splits-th
// bin of the group from bin s on, as shap_kernel.  The tile holds the upper
// triangle of every row's block, entry by entry (rows of one entry are
// neighbours, STRIDE = RW + 1 apart), so the lanes of one add fall on different
// banks and so do the lanes of the final write.
template <typename T, typename A, int RW, int LPR, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void inter_quad_kernel(DevModel<T> d,
                                                               const float* __restrict__ X,
                                                               T* __restrict__ phi, Launch L) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ unsigned short pairs[kQuadItems];
  constexpr int kThreads = 64 * WAVES;
  constexpr int STRIDE = RW + 1;
  const int M = d.M, G = d.G, W = M + 1;
  const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (b >= (int64_t)L.tiles * G * L.splits) return;   // the whole workgroup, before any barrier
  const int64_t tile = b % L.tiles;
  const int u = (int)(b / L.tiles);
  const int g = u / L.splits;
  const int s = u - g * L.splits;
  const int64_t r0 = tile * RW;
  const int gb0 = d.group_bins[g], gb1 = d.group_bins[g + 1];
  const int tile_elems = W * (W + 1) / 2 * STRIDE;
  A* ps = reinterpret_cast<A*>(smem);
  int* xs = reinterpret_cast<int*>(smem + (((size_t)tile_elems * sizeof(A) + 15) & ~(size_t)15));
  QuadStage<T>* stages = reinterpret_cast<QuadStage<T>*>(
      reinterpret_cast<unsigned char*>(xs) + (((size_t)RW * L.sx * sizeof(int) + 15) & ~(size_t)15));
  for (int i = threadIdx.x; i < RW * M; i += kThreads) {
    const int r = i / M, c = i - r * M;
    const int64_t row = r0 + r;
    xs[r * L.sx + c] = fkey(row < L.rows ? X[row * L.ld + c] : 0.0f);
  }
  for (int i = threadIdx.x; i < tile_elems; i += kThreads) ps[i] = A(0);
  for (int i = threadIdx.x; i < kQuadItems; i += kThreads) {
    int j = 0;
    while ((j + 1) * (j + 2) / 2 <= i) ++j;
    pairs[i] = (unsigned short)((i - j * (j + 1) / 2) | j << 8);
  }
  __syncthreads();

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  // a tile of 4 rows leaves the upper half of the wave without rows
  const int r = (lane / LPR) % RW;
  const bool mine = lane / LPR < RW && r0 + r < L.rows;
  Nodes<T, 8 / LPR> n8;
  n8.row = mine;
  Nodes<T, (LPR == 4 ? 1 : 8 / LPR)> n4;   // LPR == 8 runs all lengths on 8 nodes
#pragma unroll
  for (int n = 0; n < 8 / LPR; ++n) {
    const double t = kNodeT[1][(lane % LPR) * (8 / LPR) + n];
    n8.t[n] = (T)t;
    n8.c[n] = (T)(1.0 - t);
    n8.k[n] = (T)(1.0 / (1.0 - t));
    n8.w[n] = (T)kNodeW[1][(lane % LPR) * (8 / LPR) + n];
  }
  if constexpr (LPR == 4) {
    const double t = kNodeT[0][lane % LPR];
    n4.t[0] = (T)t;
    n4.c[0] = (T)(1.0 - t);
    n4.k[0] = (T)(1.0 / (1.0 - t));
    n4.w[0] = (T)kNodeW[0][lane % LPR];
    n4.row = mine;
  } else {
    n4 = n8;
  }
  QuadStage<T>* st = stages + wave;
  const int* xrow = xs + r * L.sx;
  A* tp = ps + r;
  for (int bi = gb0 + s + wave * L.splits; bi < gb1; bi += WAVES * L.splits) {
    const Bin<T> bin = load_bin(d, bi, lane);
    const BinIndex ix = index_bin(bin, lane);
    stage_bin(&st->bin, bin, lane, ix);
    for (uint64_t rest = ix.roots; rest != 0; rest &= rest - 1ull) {
      const int rl = __builtin_ctzll(rest);
      const int q = __builtin_amdgcn_readlane(ix.info, rl) & 0xff;
#define GTS_QUAD(n, nd)                                                                     \
  case n: quad_path<T, A, n, (int)(sizeof(nd.t) / sizeof(T)), LPR, STRIDE>(st, rl, q, nd, xrow, tp,    \
                                                                 pairs, lane, W);            \
    break;
      switch (q <= 2 ? q : (q + 1) & ~1) {
        GTS_QUAD(1, n4) GTS_QUAD(2, n4) GTS_QUAD(4, n4) GTS_QUAD(6, n4) GTS_QUAD(8, n4)
        GTS_QUAD(10, n8) GTS_QUAD(12, n8) GTS_QUAD(14, n8) GTS_QUAD(16, n8)
        default: break;
      }
#undef GTS_QUAD
    }
    // the next bin overwrites the stage
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();

  const T bias = s == 0 ? d.bias[g] : T(0);
  const int WW = W * W;
  for (int i = threadIdx.x; i < RW * WW; i += kThreads) {
    const int rr = i / WW, c = i - rr * WW;
    const int64_t row = r0 + rr;
    if (row >= L.rows) break;
    const int a = c / W;
    T val = (T)ps[tri_at(a, c - a * W, W) * STRIDE + rr];
    if (c == WW - 1) val += bias;
    T* out = phi + (row * G + g) * (int64_t)WW + c;
    if (L.accumulate) unsafeAtomicAdd(out, val);
    else *out = val;
  }
}

template <typename T>
size_t quad_lds(int M, int rows, int waves, bool wide) {
  const size_t tri = (size_t)(M + 1) * (M + 2) / 2;
  const size_t tile = (tri * (rows + 1) * (wide ? sizeof(double) : sizeof(T)) + 15) & ~(size_t)15;
  const size_t x = ((size_t)rows * (M | 1) * sizeof(int) + 15) & ~(size_t)15;
  return tile + x + (size_t)waves * sizeof(QuadStage<T>);
}

template <typename T, typename A, int RW, int LPR, int WAVES>
gts_status launch_quad(const KernelArgs& a, const Plan& p) {
  const gts_model* m = a.m;
  hipStream_t stream = static_cast<hipStream_t>(a.stream);
  DevModel<T> d = dev_model<T>(m, a.blob);
  Launch L{};
  L.rows = a.rows;
  L.ld = a.ld;
  L.tiles = (int32_t)p.tiles;
  L.splits = p.splits;
  L.sx = p.sx;
  L.accumulate = p.splits > 1 ? 1 : 0;
  const int64_t grid = p.tiles * m->num_groups * p.splits;
  if (grid > 0x7fffffffLL) return fail(GTS_EINVAL, "problem too large for one launch");
  auto kern = inter_quad_kernel<T, A, RW, LPR, WAVES>;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds) != hipSuccess) {
    (void)hipGetLastError();
    return fail(GTS_EDEVICE, "cannot set the LDS size of the kernel to %zu bytes", p.lds);
  }
  const int64_t total = a.rows * (int64_t)m->num_groups * p.width;
  if (L.accumulate) {
    const int64_t blocks = std::min<int64_t>((total + 255) / 256, 65536);
    hipLaunchKernelGGL(fill_zero<T>, dim3((unsigned)blocks), dim3(256), 0, stream,
                       static_cast<T*>(a.phi), total);
  }
  hipLaunchKernelGGL(kern, grid_of(grid, 64 * WAVES), dim3(64 * WAVES), p.lds, stream, d, a.X,
                     static_cast<T*>(a.phi), L);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail(GTS_EDEVICE, "kernel launch failed: %s", hipGetErrorString(err));
  return GTS_OK;
}

template <typename T>
gts_status launch_quad_shape(const KernelArgs& a, const Plan& p) {
  if constexpr (sizeof(T) == 4) {
    if (p.wide_tile) return launch_quad<T, double, 16, 4, 16>(a, p);
    if (p.RW == 16) return launch_quad<T, float, 16, 4, 16>(a, p);
    if (p.RW == 8) return launch_quad<T, float, 8, 8, 16>(a, p);
    return launch_quad<T, float, 4, 8, 8>(a, p);
  } else {
    if (p.RW == 16) return launch_quad<T, double, 16, 4, 8>(a, p);
    if (p.RW == 8) return launch_quad<T, double, 8, 8, 8>(a, p);
    return launch_quad<T, double, 4, 8, 8>(a, p);
  }
}

}  // namespace
}  // namespace gts
