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
// loops over arrays in private memory beyond 8 features: 10.8 ms for 200 rows of
// 100 trees of depth 16 over 54 features, fp32, against 0.31 ms here.  Up to 8
// features its unrolled code is the faster one: 0.29 against 1.0 ms for 1000 rows
// of 100 trees of depth 8 over 54 features.)
//
// Lanes.  A wave takes one path for RW rows; LPR neighbouring lanes share a row
// and hold NPL = N / LPR nodes each.  The LPR lanes' partial sums of LPR entries
// are exchanged by DPP so that every lane ends with one whole entry, and all 64
// lanes add to the tile at once.
//
// Tile and arithmetic.  A is the type of the tile's entries, C of the arithmetic.
// The runtime-length code takes these paths in fp64 and adds to a tile of the
// model's type; no launch here is further from fp64 values than it.
//   C float, A double (fp32 models): the tile's sums are all but exact, which leaves
//     the paths' own arithmetic.  Node pairs that fp32 holds (kPairC), a reciprocal
//     with its remainder and a diagonal that holds phi_i until the tile is written,
//     when the row's Delta_ij are taken from it, keep that small: 100 trees of depth
//     14, 200 rows, distance from fp64 0.86e-7 at M = 40 (runtime-length code 1.59e-7),
//     0.55e-7 at M = 54 (1.12e-7), 1.0e-7 at M = 77 (2.5e-7).  With rounded nodes and
//     phi_ii formed path by path it was 1.13e-7 at M = 40, and with a float tile
//     1.21e-7 at M = 54 and 2.75e-7 at M = 77, at 0.96 and 0.88 of the time.
//   C double, A float (fp32 models of M >= 79, where 4 rows in double do not fit):
//     phi_ii path by path, each entry rounded once per path, as the runtime-length
//     code does.
//   C and A double (fp64 models): phi_ii path by path too (from the tile 1.41e-15
//     instead of 1.28e-15 from fp64 values, M = 29).
// gfx950 adds doubles in LDS natively (ds_add_f64, about 8 cycles per wave
// instruction and CU, no result to wait for), floats only by compare-and-swap at a
// useful rate (14 cycles and a round trip of 200; ds_add_f32: 192 cycles).
#pragma once

#include "gts_shap_kernel.h"

namespace gts {
namespace {

constexpr int kQuadMaxQ = 16;
constexpr int kQuadItems = kQuadMaxQ * (kQuadMaxQ + 1) / 2;   // entries of one path

// Node pairs of fp32 arithmetic, for N = 4 (set 0) and N = 8 (set 1) nodes.  A path's
// polynomial is homogeneous in (c, t) = (1 - t, t), so any pair with the node's ratio
// serves: a factor z c + o t is then the node's times S = c + t.  Rounded nodes would
// move the products of all paths alike, by up to 16 errors of 3e-8; of the 2^23 floats
// c from 1 - t up to its double, these are the ones for which t, 1 / c and 2 / S are all
// within 2.5e-10 of a float.
__device__ constexpr float kPairC[2][8] = {
    {0x1.45f48p+0f, 0x1.7ca0ep-1f, 0x1.9dbfaep-2f, 0x1.74e742p-4f},
    {0x1.07f282p+0f, 0x1.0eb69p+0f, 0x1.9675cp-1f, 0x1.4e90fap-1f, 0x1.9d6df6p-1f,
     0x1.0d549ap-2f, 0x1.60516p-3f, 0x1.a20c36p-6f}};
__device__ constexpr float kPairT[2][8] = {
    {0x1.851fccp-4f, 0x1.76f6a6p-2f, 0x1.a3ffeap-1f, 0x1.385e12p+0f},
    {0x1.5632dep-6f, 0x1.ea327cp-4f, 0x1.f9aa3cp-3f, 0x1.cdb2eep-2f, 0x1.2b969ap+0f,
     0x1.b0fb88p-1f, 0x1.852338p+0f, 0x1.4273a4p+0f}};

// Their weights over S^(Q - 2), the scale of P rho_i rho_j: [LPR == 8][(Q + 1) / 2][node],
// Q = 1, 2, 4, ... 16 (four lanes a row run Q <= 8 on four nodes).
struct PairWeights {
  float w[2][9][8] = {};
  constexpr PairWeights() {
    for (int l = 0; l < 2; ++l)
      for (int h = 0; h < 9; ++h) {
        const int set = l == 0 && h <= 4 ? 0 : 1;
        const int Q = h == 0 ? 1 : 2 * h;
        for (int n = 0; n < (set ? 8 : 4); ++n) {
          const double S = (double)kPairC[set][n] + (double)kPairT[set][n];
          double x = kGaussWeight[set ? 7 : 3][n] * (Q == 1 ? S : 1.0);
          for (int i = 2; i < Q; ++i) x /= S;
          w[l][h][n] = (float)x;
        }
      }
  }
};
__device__ constexpr PairWeights kPairWeights;

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

// A lane's nodes: factors are z c + o t, k = 1 / c, two = 2 / S, w = the weight (of fp32
// arithmetic it depends on the path's length: kPairWeights).
template <typename C, int NPL>
struct Nodes {
  bool row;   // the lane has a row
  C t[NPL], c[NPL], k[NPL], two[NPL], w[NPL];
};

template <typename C, int NPL>
__device__ __forceinline__ void set_node(Nodes<C, NPL>& nd, int i, int set, int n) {
  if constexpr (sizeof(C) == 4) {
    nd.c[i] = kPairC[set][n];
    nd.t[i] = kPairT[set][n];
    nd.k[i] = (C)(1.0 / (double)nd.c[i]);
    nd.two[i] = (C)(2.0 / ((double)nd.c[i] + (double)nd.t[i]));
    nd.w[i] = C(0);
  } else {
    const double t = kGaussNode[set ? 7 : 3][n];
    nd.t[i] = t;
    nd.c[i] = 1.0 - t;
    nd.k[i] = 1.0 / (1.0 - t);
    nd.two[i] = 2.0;
    nd.w[i] = kGaussWeight[set ? 7 : 3][n];
  }
}

// One path (root in slot s, q features, padded to Q) for the wave's rows.
template <typename T, typename C, typename A, int Q, int NPL, int LPR, int STRIDE>
__device__ __forceinline__ void quad_path(QuadStage<T>* st, int s, int q, const Nodes<C, NPL>& nd,
                                          const float* __restrict__ weights,
                                          const int* __restrict__ xrow, A* __restrict__ tile,
                                          const unsigned short* __restrict__ pairs, int lane,
                                          int W) {
  constexpr bool kLater = sizeof(C) == 4;   // phi_ii is formed when the tile is written
  const int g = lane % LPR;
  C P[NPL], R[NPL], rho[Q][NPL];
  const C v = (C)st->bin.w(s);
#pragma unroll
  for (int n = 0; n < NPL; ++n) {
    if constexpr (sizeof(C) == 4) P[n] = weights[g * NPL + n] * v;
    else P[n] = nd.w[n] * v;
    R[n] = C(0);
  }
  bool live = nd.row;
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    // past the path's end: z = 1 and present, a factor of S with rho = 0
    const bool real = k < q;
    const int e = s + (real ? 1 + k : 0);
    const int4 head = st->bin.head[e];
    const C z = real ? (C)st->bin.z(e) : C(1);
    const bool o = !real || in_range(xrow[real ? head.x : 0], head.y, (unsigned)head.z);
    live &= o | (z != C(0));   // else a zero factor: the path leaves nothing here
    const C d = C(1) - z;
#pragma unroll
    for (int n = 0; n < NPL; ++n) {
      const C hi = fma(z, nd.c[n], nd.t[n]);
      const C a = o ? hi : z * nd.c[n];
      const C y = recip(hi);
      C r = d * y;
      // v_rcp_f32 leaves out up to one last bit: the remainder's share back
      if constexpr (sizeof(C) == 4) r = fma(fma(-hi, r, d), y, r);
      keep(r);
      r = o ? r : -nd.k[n];
      P[n] *= a;
      if constexpr (!kLater) R[n] += r;
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
  C part[LPR];
  A* p[kBatch];
  A val[kBatch];
  bool on[kBatch];
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    C u[NPL];
#pragma unroll
    for (int n = 0; n < NPL; ++n) u[n] = C(0.5) * P[n] * rho[j][n];
#pragma unroll
    for (int i = 0; i <= j; ++i) {
      const int m = j * (j + 1) / 2 + i;
      C x = C(0);
#pragma unroll
      for (int n = 0; n < NPL; ++n)
        x = fma(u[n],
                i < j    ? rho[i][n]
                : kLater ? nd.two[n]
                         : nd.two[n] - (R[n] - rho[j][n]),
                x);
      part[m % LPR] = x;
      if (m == kItems - 1) {
#pragma unroll
        for (int l = m % LPR + 1; l < LPR; ++l) part[l] = C(0);
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
          tile_add<kBatched>(p, val, on);
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
template <typename T, typename C, typename A, int RW, int LPR, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void inter_quad_kernel(DevModel<T> d,
                                                               const float* __restrict__ X,
                                                               T* __restrict__ phi, Launch L) {
  extern __shared__ __align__(16) unsigned char smem[];
  static_assert(sizeof(C) == 8 || sizeof(A) == 8, "fp32 arithmetic needs a tile in double");
  __shared__ unsigned short pairs[kQuadItems];
  __shared__ float weights[sizeof(C) == 4 ? 9 * 8 : 1];
  constexpr int kThreads = 64 * WAVES;
  constexpr int STRIDE = RW + 1;
  const int M = d.M, G = d.G, W = M + 1;
  const unsigned b = blockIdx.y * L.grid_x + blockIdx.x;
  if (b >= L.groups) return;   // the whole workgroup, before any barrier
  const int64_t tile = b % (unsigned)L.tiles;
  const int u = (int)(b / (unsigned)L.tiles);
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
  if constexpr (sizeof(C) == 4)
    if (threadIdx.x < 9 * 8)
      weights[threadIdx.x] = kPairWeights.w[LPR == 8][threadIdx.x / 8][threadIdx.x % 8];
  __syncthreads();

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  // a tile of 4 rows leaves the upper half of the wave without rows
  const int r = (lane / LPR) % RW;
  const bool mine = lane / LPR < RW && r0 + r < L.rows;
  Nodes<C, 8 / LPR> n8;
  n8.row = mine;
  Nodes<C, (LPR == 4 ? 1 : 8 / LPR)> n4;   // LPR == 8 runs all lengths on 8 nodes
#pragma unroll
  for (int n = 0; n < 8 / LPR; ++n) set_node(n8, n, 1, (lane % LPR) * (8 / LPR) + n);
  if constexpr (LPR == 4) {
    set_node(n4, 0, 0, lane % LPR);
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
    stage_bin<false>(&st->bin, bin, lane, ix);
    for (uint64_t rest = ix.roots; rest != 0; rest &= rest - 1ull) {
      const int rl = __builtin_ctzll(rest);
      const int q = __builtin_amdgcn_readlane(ix.info, rl) & 0xff;
#define GTS_QUAD(n, nd)                                                                      \
  case n:                                                                                    \
    quad_path<T, C, A, n, (int)(sizeof(nd.t) / sizeof(C)), LPR, STRIDE>(                     \
        st, rl, q, nd, weights + (sizeof(C) == 4 ? (n / 2) * 8 : 0), xrow, tp, pairs, lane,  \
        W);                                                                                  \
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

  if constexpr (sizeof(C) == 4) {
    // phi_ii = phi_i - sum of Delta_ij: rows of one entry are neighbours, and the
    // entries (j, f), j < f, lie W - 1 - j apart, then (f, j) one after the other
    for (int i = threadIdx.x; i < RW * M; i += kThreads) {
      const int f = i / RW, rr = i - f * RW;
      A* const row = ps + rr;
      A sum = row[(tri_row(f, W) + f) * STRIDE];
      int at = f;
      for (int j = 0; j < f; ++j) {
        sum -= row[at * STRIDE];
        at += W - 1 - j;
      }
      for (int j = f + 1; j < M; ++j) sum -= row[++at * STRIDE];
      row[(tri_row(f, W) + f) * STRIDE] = sum;
    }
    __syncthreads();
  }

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

template <typename T, typename C, typename A, int RW, int LPR, int WAVES>
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
  auto kern = inter_quad_kernel<T, C, A, RW, LPR, WAVES>;
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
  const dim3 dims = grid_of(grid, 64 * WAVES);
  L.grid_x = dims.x;
  L.groups = (uint32_t)grid;
  hipLaunchKernelGGL(kern, dims, dim3(64 * WAVES), p.lds, stream, d, a.X,
                     static_cast<T*>(a.phi), L);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail(GTS_EDEVICE, "kernel launch failed: %s", hipGetErrorString(err));
  return GTS_OK;
}

template <typename T>
gts_status launch_quad_shape(const KernelArgs& a, const Plan& p) {
  if constexpr (sizeof(T) == 4) {
    if (p.wide_tile) {
      if (p.RW == 16) return launch_quad<T, float, double, 16, 4, 16>(a, p);
      if (p.RW == 8) return launch_quad<T, float, double, 8, 8, 16>(a, p);
      return launch_quad<T, float, double, 4, 8, 16>(a, p);
    }
    if (p.RW == 8) return launch_quad<T, double, float, 8, 8, 12>(a, p);
    if (p.waves == 16) return launch_quad<T, double, float, 4, 8, 16>(a, p);
    return launch_quad<T, double, float, 4, 8, 8>(a, p);
  } else {
    if (p.RW == 16) return launch_quad<T, double, double, 16, 4, 8>(a, p);
    if (p.RW == 8) return launch_quad<T, double, double, 8, 8, 8>(a, p);
    return launch_quad<T, double, double, 4, 8, 8>(a, p);
  }
}

}  // namespace
}  // namespace gts
