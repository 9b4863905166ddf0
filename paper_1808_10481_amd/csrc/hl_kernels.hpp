// hl_kernels.hpp - Hermite-leapfrog half-step kernels for gfx950.
//
// One work-item per output node.  For the pressure half-step at primal node
// j the cell's corners are the dual nodes q = j - 1 + e, e in {0,1}^d; for the
// velocity half-step at dual node q they are the primal nodes j = q + e
// (Sec. 2, eqs. (pGrid), (dGrid); Sec. 5).  The interpolant of the corner
// data (Sec. 2, eq. (interp)) is built one dimension at a time (Sec. 5): the
// x pass runs explicitly with compile-time coefficients; the remaining
// dimensions' interpolation and the Cauchy-Kowalevsky weights (Sec. 2,
// eq. (final1); Sec. 3.1.2, eqs. (pdup), (vdup)) are applied together through
// a runtime merged table (hl_layout.hpp) acting on sums and differences of
// corners, so the (2m+2)^d interpolant never exists as a whole.
//
// Storage (hl_storage.hpp) is a template policy S: S::C is the arithmetic
// type, S::load / S::update / S::planes / S::bload the only memory accesses
// to the state.  Planes are coefficient-major: plane index
// comp * (m+1)^d + c, c = a_1 + (m+1)(a_2 + (m+1) a_3), node
// n = i_1 + E_1 (i_2 + E_2 i_3) in an array of extents E.
//
// Boundaries.  Periodic: both grids have K nodes per dimension, corner
// indices wrap.  Reflecting walls: the primal grid has K+1 nodes (the end
// nodes on the walls), the dual grid K nodes stored inside a (K+2)-node array
// whose outer shell holds ghost nodes (filled by ghost_fill before every
// pressure half-step); no index wraps.  A Grid describes one half-step: the
// nodes it updates (K, stored at index j + ooff of the output array) and the
// corner array (corner lo of node j at j + soff, hi at lo + 1, wrapped into
// [0, sext) for periodic grids).
//
// Launch: tiles of TileShape nodes, one workgroup per tile.  Workgroup i runs
// on XCD i mod 8 and takes tile number t = (i mod 8) * per_xcd + i / 8, so
// each XCD sweeps one contiguous band of tile numbers.  Tile numbers run x
// fastest, then y inside a group of `ygroup` tile rows, then z, then the
// groups; in 3D a small group keeps the z-neighbour planes of the tiles in
// flight inside the XCD's L2 (a whole z-plane of corner data does not fit).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "hl_layout.hpp"
#include "hl_storage.hpp"

// Scheduling barrier mask inside the merged-table loop: instruction classes
// allowed to move across (0 = none; 0x2 VALU, 0x4 SALU, 0x20 VMEM reads).
// Scalar table loads never cross, which bounds the table's live range in
// SGPRs; measured on the 2D m=3 workload, 0 is fastest (letting vector loads
// cross raised register pressure and cost 5-8%).
#ifndef HL_SCHED_MASK
#define HL_SCHED_MASK 0
#endif
// Buffer-instruction cache policy of streamed outputs (Grid::stream): the
// non-temporal bit.
constexpr int kStreamAux = 2;

// Minimum waves per SIMD requested from the register allocator (0 = none).
#ifndef HL_WAVES_PER_EU
#define HL_WAVES_PER_EU 0
#endif
// 3D tile extent in x and y (x * y = 256 work-items).
#ifndef HL_TILE3_X
#define HL_TILE3_X 64
#endif

namespace hl {

constexpr int kXcds = 8;

// Constant-address-space view of a table: uniform reads become scalar loads
// (a pointer read from memory, or made opaque, is otherwise generic).
template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ ConstPtr<T> const_ptr(const T* p) {
  return (ConstPtr<T>)(uintptr_t)p;
}

struct Grid {
  int32_t K[3];       // nodes updated per dimension (1 for unused dimensions)
  int32_t nt[3];      // tiles per dimension
  int32_t tiles;      // nt[0] * nt[1] * nt[2]
  int32_t per_xcd;    // ceil(tiles / kXcds)
  int32_t ygroup;     // tile rows per group in the tile numbering, 1..nt[1]
  int32_t ystaged;    // the same for the staged 3D half-steps (layered())
  int32_t ooff;       // output node j is stored at index j + ooff (0, or 1 in a ghost-padded array)
  int32_t oext[3];    // output array extents
  int32_t soff;       // lower corner of node j at index j + soff (-1 or 0)
  int32_t sext[3];    // corner (source) array extents
  int32_t tx, ty;     // tile extents in x and y = the workgroup shape (tx * ty <= 256)
  // Outputs are read and written with the non-temporal policy.  Each output
  // word is touched once per half-step, so streaming it leaves the caches to
  // the corner words.  It pays only where every access covers whole 128-byte
  // lines (a line shared by two accesses is otherwise fetched twice) and the
  // state does not fit the 256 MB last-level cache, where cached outputs
  // are still found by the next half-step (make_grid).  Measured, velocity
  // half-step, streamed / cached: 3D m = 2 FP64 256^3 5.04 / 5.33 ms, 64^3
  // 98 / 83 us; FP32 161x150x143 1006 / 684 us.
  int32_t stream;
  int32_t open;  // corners outside the source array are zero (no wrap; walled adjoint)
  int64_t onodes;     // output array nodes (plane size)
  int64_t snodes;     // source array nodes (plane size)
};

template <int D>
struct TileShape {
  static constexpr int X = D == 1 ? 256 : D == 2 ? 64 : HL_TILE3_X;
  static constexpr int Y = 256 / X;
  static constexpr int Z = 1;
};

// out[b] = sum_l pass_coef<M,FLIP>(b, l) * (b + l + FLIP even ? R_l + L_l : R_l - L_l)
template <int M, int FLIP, typename T>
__device__ __forceinline__ void pass1d(const T* L, const T* R, T* out) {
  constexpr int MP = M + 1, N2 = 2 * M + 2;
  T sg[MP], df[MP];
#pragma unroll
  for (int l = 0; l < MP; ++l) {
    sg[l] = R[l] + L[l];
    df[l] = R[l] - L[l];
  }
#pragma unroll
  for (int b = 0; b < N2; ++b) {
    T acc = T(0);
#pragma unroll
    for (int l = 0; l < MP; ++l) {
      const double c = pass_coef<M, FLIP>(b, l);
      if (c != 0.0) acc = fma(T(c), ((b + l + FLIP) & 1) ? df[l] : sg[l], acc);
    }
    out[b] = acc;
  }
}

// Tile coordinates of tile number t.
template <int D>
__device__ __forceinline__ void tile_coords(const Grid& g, int t, int32_t* c) {
  c[0] = t % g.nt[0];
  c[1] = c[2] = 0;
  if constexpr (D > 1) {
    const int r = t / g.nt[0];
    const int grp_rows = g.ygroup * g.nt[2];  // tile rows (y, z) per group
    const int grp = r / grp_rows;
    const int rem = r - grp * grp_rows;
    const int gy = min(g.ygroup, g.nt[1] - grp * g.ygroup);  // rows of y in this (possibly ragged) group
    c[1] = grp * g.ygroup + rem % gy;
    c[2] = rem / gy;
  }
}

// Node of this work-item in workgroup `blk` of the grid's launch; false when
// outside the grid.
template <int D>
__device__ __forceinline__ bool node_of_block(const Grid& g, int blk, int32_t* j) {
  const int i = blk;
  const int t = (i % kXcds) * g.per_xcd + i / kXcds;
  if (t >= g.tiles) return false;
  int32_t c[3];
  tile_coords<D>(g, t, c);
  j[0] = c[0] * g.tx + threadIdx.x;
  j[1] = c[1] * g.ty + threadIdx.y;
  j[2] = c[2];
  return j[0] < g.K[0] && j[1] < g.K[1] && j[2] < g.K[2];
}

template <int D>
__device__ __forceinline__ uint32_t node_index(int32_t x, int32_t y, int32_t z, const int32_t* E) {
  uint32_t n = (uint32_t)x;
  if (D > 1) n += (uint32_t)E[0] * (uint32_t)y;
  if (D > 2) n += (uint32_t)E[0] * (uint32_t)E[1] * (uint32_t)z;
  return n;
}

// Index of this work-item's output node in the output array.
template <int D>
__device__ __forceinline__ uint32_t out_index(const Grid& g, const int32_t* j) {
  return node_index<D>(j[0] + g.ooff, j[1] + g.ooff, j[2] + g.ooff, g.oext);
}

// Node indices of the 2^d cell corners e (bit k of e: upper side in
// dimension k): lo = j + soff and hi = lo + 1, wrapped into the source array.
template <int D>
__device__ __forceinline__ void corner_nodes(const Grid& g, const int32_t* j, uint32_t* cn) {
  int32_t lo[3], hi[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (k < D) {
      lo[k] = j[k] + g.soff;
      hi[k] = lo[k] + 1;
      if (lo[k] < 0) lo[k] += g.sext[k];
      if (hi[k] == g.sext[k]) hi[k] = 0;
    } else {
      lo[k] = hi[k] = 0;
    }
  }
#pragma unroll
  for (int e = 0; e < (1 << D); ++e)
    cn[e] = node_index<D>((e & 1) ? hi[0] : lo[0], (e & 2) ? hi[1] : lo[1], (e & 4) ? hi[2] : lo[2], g.sext);
}

// Entry of plane pl at node n0 of a half-step's output.  3D kernels address
// their planes through buffer descriptors (scalar plane base, 32-bit per-lane
// offset), the others through plain pointers.
template <int D, class S, bool NT>
__device__ __forceinline__ typename S::C load_output(const typename S::View& v, int pl, uint32_t n0) {
  if constexpr (D == 3)
    return S::template bload<NT ? kStreamAux : 0>(S::planes(v, pl), n0);
  else if constexpr (NT)
    return S::load_nt(v, pl, n0);
  else
    return S::load(v, pl, n0);
}
template <int D, class S, bool NT>
__device__ __forceinline__ void store_output(const typename S::View& v, int pl, uint32_t n0, typename S::C x) {
  if constexpr (D == 3)
    S::template bstore<NT ? kStreamAux : 0>(S::planes(v, pl), n0, x);
  else if constexpr (NT)
    S::store_nt(v, pl, n0, x);
  else
    S::store(v, pl, n0, x);
}

// entry <- f(i, entry) for the N output planes plane(0) .. plane(N - 1) at node
// n0.  The planes may alias as far as the compiler knows, so that written
// entry by entry each load waits for the store before it: one memory latency
// per plane.  The loads are therefore issued in batches of B, the next batch
// before the stores of the current one (B = 9 in 3D; 3 in 2D, where more of
// them cost resident wavefronts).  Velocity half-step: 3D m = 2 FP64 256^3
// 6.14 -> 5.06 ms, 2D m = 3 FP32_COMP 1024^2 129 -> 95 us, FP64 512^2 35.5 ->
// 28.9 us.
template <int D, class S, int N, bool NT, class P, class F>
__device__ __forceinline__ void update_outputs_as(const typename S::View& v, uint32_t n0, P plane, F f) {
  using T = typename S::C;
  constexpr int B = D == 3 ? 9 : 3;
  T x[2][B];
#pragma unroll
  for (int i = 0; i < B; ++i)
    if (i < N) x[0][i] = load_output<D, S, NT>(v, plane(i), n0);
#pragma unroll
  for (int c = 0; c * B < N; ++c) {
    int zero = 0;  // 3D: opaque, so that plane bases are formed here and not all held from the start
    if constexpr (D == 3 && N > B) asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
#pragma unroll
    for (int i = 0; i < B; ++i)
      if ((c + 1) * B + i < N) x[(c + 1) & 1][i] = load_output<D, S, NT>(v, plane((c + 1) * B + i) + zero, n0);
#pragma unroll
    for (int i = 0; i < B; ++i)
      if (c * B + i < N) store_output<D, S, NT>(v, plane(c * B + i) + zero, n0, f(c * B + i, x[c & 1][i]));
  }
}

// Whether a 1D or 2D half-step's streamed outputs are updated one by one: the
// work-item's own wait for each store then spaces the streams.  One by one /
// batched: 2D pressure m = 3 1024^2 FP64 114 / 131 us (cached outputs, 512^2,
// 31.6 / 25.9); velocity m = 1 4096x2048 FP64 200 / 264 us, FP32_COMP 160 / 207
// us, m = 2 2048x1500 FP64 191 / 224 us, but m = 3 1024^2 FP32_COMP 129 / 95 us;
// 1D m = 1 2^24 nodes FP64 114 / 139 us, m = 5 406 / 447 us.
template <int D, int M, bool VEL>
constexpr bool kOneByOne = D == 1 || (D == 2 && (!VEL || M <= 2));

// Which accesses a kernel's output update holds: both and the choice (kEither),
// or one of them (1D and 2D half-steps, chosen by the launch).  The choice stands
// between the outputs' loads and all before it, which half-steps of few data
// feel (velocity 2D m = 1 4096x2048 FP64 222 us with it, 200 without).
enum OutputMode { kEither, kCached, kStreamed };

template <int D, class S, int N, bool ONE = false, int MODE = kEither, class P, class F>
__device__ __forceinline__ void update_outputs(const Grid& g, const typename S::View& v, uint32_t n0, P plane, F f) {
  if constexpr (MODE == kEither) {
    if (g.stream)
      update_outputs<D, S, N, ONE, kStreamed>(g, v, n0, plane, f);
    else
      update_outputs<D, S, N, ONE, kCached>(g, v, n0, plane, f);
  } else if constexpr (MODE == kStreamed && ONE) {
#pragma unroll
    for (int i = 0; i < N; ++i) S::store_nt(v, plane(i), n0, f(i, S::load_nt(v, plane(i), n0)));
  } else {
    update_outputs_as<D, S, N, MODE == kStreamed>(v, n0, plane, f);
  }
}

// p -= acc at node n0.
template <int D, int M, class S, int MODE = kEither>
__device__ __forceinline__ void finish_pressure(const Grid& g, const typename S::View& p, uint32_t n0,
                                                const typename S::C* acc) {
  using T = typename S::C;
  update_outputs<D, S, Dims<D, M>::NC, kOneByOne<D, M, false>, MODE>(g, p, n0, [](int s) { return s; },
                                                                     [&](int s, T x) { return x - acc[s]; });
}

// u_i[s] -= wscale * (s_i + 1) / h_i * Q[s + e_i]   (Q on the set G)
template <int D, int M, class S, int MODE = kEither>
__device__ __forceinline__ void finish_velocity(const Grid& g, const typename S::View& u, uint32_t n0,
                                                const typename S::C* Q, typename S::C wscale, const typename S::C* ih) {
  using T = typename S::C;
  constexpr int MP = M + 1, NC = Dims<D, M>::NC;
  T f[D];
#pragma unroll
  for (int i = 0; i < D; ++i) f[i] = wscale * ih[i];
  update_outputs<D, S, D * NC, kOneByOne<D, M, true>, MODE>(g, u, n0, [](int t) { return t; }, [&](int t, T x) {
    const int i = t / NC, s = t % NC;
    const T a = -(T)(digit(s, MP, i) + 1) * f[i];
    return fma(a, Q[kGIndex<D, M>.g[i][s]], x);
  });
}

// ---------------------------------------------------------------------------
// 1D and 2D kernels: the merged table covers the last dimension.
// ---------------------------------------------------------------------------

// Slice of the interpolant for last-dimension corner eL and last-dimension
// datum l: Y[b], b in {0..2m+1}^{d-1}, from the 2^{d-1} corners with that eL.
// FLIP0 = 1 makes the x pass the derivative pass (units of 1/h_x).  comp:
// field component; cn[e]: corner node indices.
template <int D, int M, int FLIP0, class S>
__device__ __forceinline__ void slice(const typename S::View& f, int comp, const uint32_t* cn, int eL, int l,
                                      typename S::C* Y) {
  using T = typename S::C;
  constexpr int MP = M + 1, NC = Dims<D, M>::NC;
  static_assert(D == 1 || D == 2, "3D uses the x-line kernels");
  if constexpr (D == 1) {
    Y[0] = S::load(f, comp * NC + l, cn[eL]);
  } else {
    T Lv[MP], Rv[MP];
#pragma unroll
    for (int a0 = 0; a0 < MP; ++a0) {
      const int pl = comp * NC + a0 + MP * l;
      Lv[a0] = S::load(f, pl, cn[0 + 2 * eL]);
      Rv[a0] = S::load(f, pl, cn[1 + 2 * eL]);
    }
    pass1d<M, FLIP0>(Lv, Rv, Y);
  }
}

// acc[o] += sum_b Mt[t] * (sigma or delta)[b] over the structurally nonzero
// (o, b) of one merged table row-block (datum l); the walk comes from the
// compile-time MergeSpec, so every index is a constant after unrolling.
template <int D, int M, bool VEL, int FLIPL, typename T, typename TP>
__device__ __forceinline__ void merge(TP Mt, int l, const T* Sg, const T* Df, T* acc) {
  using Sp = MergeSpec<D, M, VEL, FLIPL>;
  // Scalar table loads are consumed in chunks: without the barriers the
  // scheduler hoists every s_load of the table to the top of the kernel and
  // runs out of SGPRs (spilling them through VGPR lanes).
  constexpr int kChunk = sizeof(T) == 8 ? 16 : 32;
#pragma unroll
  for (int t = 0; t < Sp::NNZ; ++t) {
    if (t % kChunk == 0) __builtin_amdgcn_sched_barrier(HL_SCHED_MASK);
    const int o = kMerge<D, M, VEL, FLIPL>.o[t];
    const int b = kMerge<D, M, VEL, FLIPL>.b[t];
    const bool dl = kMerge<D, M, VEL, FLIPL>.base_delta[o] != ((l & 1) != 0);
    acc[o] = fma(Mt[t], dl ? Df[b] : Sg[b], acc[o]);
  }
}

// Sigma/delta of the two last-dimension slices, then the merged table.
template <int D, int M, bool VEL, int FLIP0, int FLIPL, class S, typename TP>
__device__ __forceinline__ void slice_pair_merge(const typename S::View& f, int comp, const uint32_t* cn, int l, TP Mt,
                                                 typename S::C* acc) {
  using T = typename S::C;
  constexpr int NB = Dims<D, M>::NB;
  T YL[NB], YR[NB], Sg[NB], Df[NB];
  slice<D, M, FLIP0, S>(f, comp, cn, 0, l, YL);
  slice<D, M, FLIP0, S>(f, comp, cn, 1, l, YR);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    Sg[b] = YR[b] + YL[b];
    Df[b] = YR[b] - YL[b];
  }
  merge<D, M, VEL, FLIPL>(Mt, l, Sg, Df, acc);
}

// Pressure increment at a primal node from its dual corners (1D and 2D).
// tab: packed merged tables (hl_layout.hpp TableLayout), in S::C.
template <int D, int M, class S, typename TP>
__device__ __forceinline__ void p_half_acc(const typename S::View& u, TP tab, const uint32_t* cn,
                                           typename S::C* acc) {
  using T = typename S::C;
  using TL = TableLayout<D, M>;
  constexpr int MP = M + 1, NC = Dims<D, M>::NC;
  constexpr int NNZ = merged_nnz<D, M>(false);
#pragma unroll
  for (int s = 0; s < NC; ++s) acc[s] = T(0);
#pragma unroll
  for (int l = 0; l < MP; ++l) {
    // x-component (2D): derivative pass in x, interpolation in the merged table
    if constexpr (D > 1) slice_pair_merge<D, M, false, 1, 0, S>(u, 0, cn, l, tab + TL::P_A_OFF + l * NNZ, acc);
    // last component: interpolation pass in x, derivative in the merged table
    slice_pair_merge<D, M, false, 0, 1, S>(u, D - 1, cn, l, tab + TL::P_B_OFF + l * NNZ, acc);
  }
}

// Pressure half-step at every primal node (1D and 2D).
template <int D, int M, class S, int MODE, typename TP>
__device__ __forceinline__ void p_half_body(typename S::View p, typename S::View u,
                                            TP tab,
                                            Grid g, int blk) {
  int32_t j[3];
  if (!node_of_block<D>(g, blk, j)) return;
  uint32_t cn[1 << D];
  corner_nodes<D>(g, j, cn);  // dual q = j - 1 + e
  typename S::C acc[Dims<D, M>::NC];
  p_half_acc<D, M, S>(u, tab, cn, acc);
  finish_pressure<D, M, S, MODE>(g, p, out_index<D>(g, j), acc);
}

template <int D, int M, class S, int MODE>
__global__ void __launch_bounds__(256, HL_WAVES_PER_EU) p_half_kernel(typename S::View p, typename S::View u,
                                                                       const typename S::C* __restrict__ tab,
                                                                       Grid g) {
  p_half_body<D, M, S, MODE, const typename S::C* __restrict__>(p, u, tab, g, blockIdx.x);
}

// Q on the set G at a dual node from its primal corners (1D and 2D).
template <int D, int M, class S, typename TP>
__device__ __forceinline__ void u_half_Q(const typename S::View& p, TP tab, const uint32_t* cn, typename S::C* Q) {
  using T = typename S::C;
  using TL = TableLayout<D, M>;
  constexpr int NNZ = merged_nnz<D, M>(true);
#pragma unroll
  for (int o = 0; o < GSet<D, M>::NG; ++o) Q[o] = T(0);
#pragma unroll
  for (int l = 0; l <= M; ++l) slice_pair_merge<D, M, true, 0, 0, S>(p, 0, cn, l, tab + TL::U_OFF + l * NNZ, Q);
}

// Velocity half-step at every dual node (1D and 2D), weights scaled by wscale.
template <int D, int M, class S, int MODE, typename TP>
__device__ __forceinline__ void u_half_body(typename S::View u, typename S::View p,
                                            TP tab,
                                            Grid g, typename S::C wscale,
                                            typename S::C ih0, typename S::C ih1,
                                            typename S::C ih2, int blk) {
  using T = typename S::C;
  int32_t j[3];
  if (!node_of_block<D>(g, blk, j)) return;
  uint32_t cn[1 << D];
  corner_nodes<D>(g, j, cn);  // primal j = q + e
  T Q[GSet<D, M>::NG];
  u_half_Q<D, M, S>(p, tab, cn, Q);
  const T ih[3] = {ih0, ih1, ih2};
  finish_velocity<D, M, S, MODE>(g, u, out_index<D>(g, j), Q, wscale, ih);
}

template <int D, int M, class S, int MODE>
__global__ void __launch_bounds__(256, HL_WAVES_PER_EU) u_half_kernel(typename S::View u, typename S::View p,
                                                                       const typename S::C* __restrict__ tab,
                                                                       Grid g, typename S::C wscale,
                                                                       typename S::C ih0, typename S::C ih1,
                                                                       typename S::C ih2) {
  u_half_body<D, M, S, MODE, const typename S::C* __restrict__>(u, p, tab, g, wscale, ih0, ih1, ih2, blockIdx.x);
}

// ---------------------------------------------------------------------------
// 1D: several steps per launch.  A 1D half-step is a few multiply-adds per
// node, so stepping by two launches is launch latency (1.8 us each, whatever
// the grid below about 10^5 nodes).  Here a workgroup holds a stretch of nodes
// of both fields in LDS and runs all of a launch's steps on it: the whole grid
// in one workgroup (whole), or B owned nodes plus a halo of `steps` nodes on
// either side, of which each step makes one more node per side invalid (the
// pressure half-step reads the dual node to the left, the velocity half-step
// the primal node to the right).  Halo nodes are computed by the same
// arithmetic from the same data as their owner computes them, so every result
// equals stepping launch by launch bit for bit (FP64 and FP32 words; an
// FP32_COMP value may have two hi + lo encodings, and LDS would not keep which).
// With a halo, neighbours still read the
// old state while a workgroup writes, so the result goes to other buffers than
// the source.  200 cells, m = 1, FP64, 400 steps: 3.7 -> 0.55 us per step.
// ---------------------------------------------------------------------------
constexpr int kSteps1Whole = 768;  // one workgroup up to this many nodes
constexpr int kSteps1Own = 256;    // nodes owned by a workgroup otherwise ..
constexpr int kSteps1Halo = 32;    // .. and the most steps of such a launch
struct Steps1 {
  int32_t K;      // cells
  int32_t walls;  // reflecting walls: primal 0 .. K, dual 0 .. K - 1 at index q + 1 of a padded array
  int32_t whole;  // the grid in one workgroup
  int32_t own, halo, n;  // owned nodes, halo, local nodes (own + 2 halo)
  int32_t steps;
  int32_t last;   // the launch that leaves the final state: ghosts as the last step's refresh left them
};

template <int M, class S>
__global__ void __launch_bounds__(1024) steps_1d(typename S::View ps, typename S::View us, typename S::View pd,
                                                 typename S::View ud, const typename S::C* __restrict__ tab, Steps1 a,
                                                 typename S::C ih0) {
  using T = typename S::C;
  using TL = TableLayout<1, M>;
  constexpr int MP = M + 1, NG = GSet<1, M>::NG;
  extern __shared__ __align__(16) char steps1_lds[];
  T* P = reinterpret_cast<T*>(steps1_lds);  // [c][local node]
  T* U = P + MP * a.n;
  const int np = a.walls ? a.K + 1 : a.K, off = a.walls ? 1 : 0;  // primal nodes; dual node q at index q + off
  const int first = (int)blockIdx.x * a.own;                      // first owned node
  // global node of local node i on the primal / dual grid, -1 where there is none
  auto node = [&](int i, int count) -> int {
    int g = first - a.halo + i;
    if (!a.walls) {
      g %= a.K;
      return g < 0 ? g + a.K : g;
    }
    return g >= 0 && g < count ? g : -1;
  };
  for (int i = threadIdx.x; i < a.n; i += blockDim.x) {
    const int j = node(i, np), q = node(i, a.K);
#pragma unroll
    for (int c = 0; c < MP; ++c) {
      P[c * a.n + i] = j < 0 ? T(0) : S::load(ps, c, (uint32_t)j);
      U[c * a.n + i] = q < 0 ? T(0) : S::load(us, c, (uint32_t)(q + off));
    }
  }
  __syncthreads();
  // a dual node beyond a wall is the mirror of the node inside (normal
  // component even: (-1)^c)
  auto mirrored = [](int c, T x) { return (c & 1) ? -x : x; };
  for (int t = 0; t < a.steps; ++t) {
    if (a.walls && a.last && t + 1 == a.steps) {  // the ghosts of the last refresh
      for (int i = threadIdx.x; i < a.n; i += blockDim.x) {
        const int q = first - a.halo + i;
        if (i < a.halo || i >= a.halo + a.own) continue;
#pragma unroll
        for (int c = 0; c < MP; ++c) {
          if (q == 0) S::store(ud, c, 0u, mirrored(c, U[c * a.n + i]));
          if (q == a.K - 1) S::store(ud, c, (uint32_t)(a.K + 1), mirrored(c, U[c * a.n + i]));
        }
      }
    }
    for (int i = threadIdx.x; i < a.n; i += blockDim.x) {
      const int g = first - a.halo + i;
      int lo = i - 1, hi = i;
      bool mlo = false, mhi = false;
      if (a.walls) {
        if (g == 0) lo = i, mlo = true;         // ghost dual -1 mirrors dual 0
        if (g == a.K) hi = i - 1, mhi = true;   // ghost dual K mirrors dual K - 1
      } else if (a.whole && i == 0) {
        lo = a.n - 1;
      }
      lo = max(lo, 0);
      hi = max(hi, 0);
      T acc[MP];
#pragma unroll
      for (int s = 0; s < MP; ++s) acc[s] = T(0);
#pragma unroll
      for (int l = 0; l < MP; ++l) {
        const T ul = U[l * a.n + lo], ur = U[l * a.n + hi];
        const T YL = mlo ? mirrored(l, ul) : ul, YR = mhi ? mirrored(l, ur) : ur;
        const T Sg[1] = {YR + YL}, Df[1] = {YR - YL};
        merge<1, M, false, 1>(tab + TL::P_B_OFF + l * merged_nnz<1, M>(false), l, Sg, Df, acc);
      }
#pragma unroll
      for (int s = 0; s < MP; ++s) P[s * a.n + i] = P[s * a.n + i] - acc[s];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < a.n; i += blockDim.x) {
      const int hi = i + 1 < a.n ? i + 1 : (a.whole && !a.walls ? 0 : i);
      T Q[NG];
#pragma unroll
      for (int o = 0; o < NG; ++o) Q[o] = T(0);
#pragma unroll
      for (int l = 0; l < MP; ++l) {
        const T YL = P[l * a.n + i], YR = P[l * a.n + hi];
        const T Sg[1] = {YR + YL}, Df[1] = {YR - YL};
        merge<1, M, true, 0>(tab + TL::U_OFF + l * merged_nnz<1, M>(true), l, Sg, Df, Q);
      }
      const T f = T(1) * ih0;
#pragma unroll
      for (int s = 0; s < MP; ++s) {
        const T w = -(T)(s + 1) * f;
        U[s * a.n + i] = fma(w, Q[kGIndex<1, M>.g[0][s]], U[s * a.n + i]);
      }
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < a.own; i += blockDim.x) {
    const int g = first + i, k = a.halo + i;
#pragma unroll
    for (int c = 0; c < MP; ++c) {
      if (g < np) S::store(pd, c, (uint32_t)g, P[c * a.n + k]);
      if (g < a.K) S::store(ud, c, (uint32_t)(g + off), U[c * a.n + k]);
    }
  }
}

// ---------------------------------------------------------------------------
// 3D kernels.  Interpolation in x, y and z, the Cauchy-Kowalevsky weights and
// the divergence are all in one runtime table (hl_layout.hpp TableLayout<3, M>):
// per datum (one coefficient plane of one source field) a node's 8 corner
// values are combined into sigma / delta in x, y and z, and every output takes
// the one combination whose parity in each dimension is that of
// o_k + a_k (+ 1 in the divergence dimension), times its table entry.
//
// What bounds these kernels is HBM, and how many distinct lines they keep in
// flight: per datum a node needs 8 corner words of which 7 are shared with its
// neighbours.  So a workgroup stages each datum's tile of source words (its
// nodes' corners: (tx + 1) x (ty + 1) x 2) through LDS: every word is loaded
// once per workgroup instead of up to 8 times.  The data go in groups of
// kStageGroup: a group's words are loaded into registers (NE per work-item and
// datum) while the previous group is computed, then written to one of two LDS
// buffers, so that one barrier per group separates the writes of a group from
// the reads of the group two before.  256^3, m = 2, pressure / velocity half-
// step, every work-item loading its own corners -> staged: FP64 7.5 / 6.7 ->
// 4.3 / 5.1 ms (the pressure half-step then reads and writes 21.7 GB at 5.0
// TB/s, a device copy's rate), FP32 2.9 / 3.1 -> 2.3 / 2.6 ms, FP32_COMP
// 5.1 / 6.8 -> 3.6 / 4.0 ms (a staged word is widened once, not once per
// corner).  A loop over the lines of data in place of the unrolled code (the
// sigma / delta choice made by signs) is 5 times smaller but runs 4.5 / 2.5 /
// 4.0 ms.
//
// Coefficient planes are read through buffer descriptors, one per plane, with
// a 32-bit per-lane offset: the kernels touch 4 (m+1)^3 planes, too many for
// a 64-bit scalar base each.
// ---------------------------------------------------------------------------
constexpr int kStageGroup = 3;

// Wavefront classes of a workgroup: the outputs are split over NS = 1 or 2
// classes of wavefronts by the parity of their x index, all reading the same
// staged words.  A class forms only the sigma or the delta in x that its
// outputs take, so no arithmetic is repeated.  Split where the accumulators
// of all outputs would leave too few resident wavefronts.
template <int M, class S>
constexpr int kPSplit = M >= 3 ? 2 : 1;
template <int M, class S>
constexpr int kUSplit = M >= 2 ? 2 : 1;
// Node layers in z of a workgroup's tile: TZ layers stage TZ + 1 planes, so
// two layers fetch 1.5 planes per layer instead of 2 (FP64 256^3 pressure
// half-step: 19.8 -> 18.1 GB read, 4.73 -> 4.43 ms).  Its workgroups are
// twice as large: only where at least kLayeredTiles of them remain (two per
// CU); 40^3 FP32 runs 39 us with one layer, 51 us with two.
template <int M, class S>
constexpr int kPLayers = M >= 3 ? 1 : 2;
constexpr int kLayeredTiles = 512;

// Work-items of one class: the tile rounded up to whole wavefronts.
__host__ __device__ constexpr int class_items(int tx, int ty, int tz) { return (tx * ty * tz + 63) / 64 * 64; }
// Staged words of a tile, and whether NE words per work-item cover them.
__host__ __device__ constexpr int stage_words(int tx, int ty, int tz) { return (tz + 1) * (tx + 1) * (ty + 1); }
__host__ __device__ constexpr bool stage_fits(int tx, int ty, int tz, int ns, int ne) {
  return stage_words(tx, ty, tz) <= ne * ns * class_items(tx, ty, tz);
}
// Words per work-item and datum for the default 64 x 4 tile, and for any tile
// hl_set_tile takes.
constexpr int stage_few(int ns, int tz) {
  int ne = 1;
  while (!stage_fits(64, 4, tz, ns, ne)) ++ne;
  return ne;
}
constexpr int stage_any(int ns, int tz) {
  int ne = 1;
  for (int tx = 32; tx <= 256; tx += 32)
    for (int ty = 1; tx * ty <= 256; ++ty)
      while (tx * ty >= 64 && !stage_fits(tx, ty, tz, ns, ne)) ++ne;
  return ne;
}
// One half-step's workgroup shape: NS classes, TZ layers, NE staged words per
// work-item and datum; CAP LDS words per buffer (NE words of the most
// work-items a workgroup has).
// ANY: tiles that need fewer than NE words skip the rest.
template <int NS_, int TZ_, int NE_, bool ANY_>
struct StageShape {
  static constexpr bool ANY = ANY_, DIRECT = false;
  static constexpr int NS = NS_, TZ = TZ_, NE = NE_, CAP = NE_ * NS_ * 256 * TZ_, LDS = 2 * kStageGroup * CAP;
};
// Every work-item loads its own corners (the tile's work-items as they are):
// m = 0, whose three data (pressure; one for the velocity) are not worth the
// staging's barriers and address arithmetic, and FP32 batches (kBatchForm).  m = 0, staged / direct: step of
// 192^3 FP32 130 / 70 us, FP32_COMP 178 / 102 us, FP64 162 / 137 us; transposed
// step of 161x150x143 FP32_COMP 372 / 125 us.
struct DirectShape {
  static constexpr bool DIRECT = true;
  static constexpr int NS = 1, TZ = 1, LDS = 1;
};
// The default tile with its layers, with one layer, any tile, and no staging.
enum StageForm { kLayered, kOneLayer, kAnyTile, kDirect };
template <int NS, int TZ, int FORM>
struct ShapeOf {
  using type = StageShape<NS, FORM == kLayered ? TZ : 1,
                          FORM == kAnyTile ? stage_any(NS, 1) : stage_few(NS, FORM == kLayered ? TZ : 1),
                          FORM == kAnyTile>;
};
template <int NS, int TZ>
struct ShapeOf<NS, TZ, kDirect> {
  using type = DirectShape;
};
template <int M>
constexpr int form3(int form) {
  return M == 0 ? (int)kDirect : form;
}
template <int M, class S, int FORM>
using PShape = typename ShapeOf<kPSplit<M, S>, kPLayers<M, S>, form3<M>(FORM)>::type;
template <int M, class S, int FORM>
using UShape = typename ShapeOf<kUSplit<M, S>, 1, form3<M>(FORM)>::type;
// Whether a shape takes tiles of tx x ty nodes.
template <class SH>
__host__ constexpr bool takes_tile(int tx, int ty) {
  if constexpr (SH::DIRECT)
    return true;
  else
    return stage_fits(tx, ty, SH::TZ, SH::NS, SH::NE);
}

// One workgroup's tile: this work-item's node and the source nodes of the
// words it stages.
template <class SH>
struct Stage3 {
  static constexpr int NE = SH::NE;
  int32_t j[3];        // this work-item's output node
  bool active;         // inside the grid (all work-items stage and meet the barriers)
  int cls;             // class of this wavefront, 0 .. NS - 1
  int item, items;     // this work-item's first staged word, and the stride to its next
  int total;           // staged words
  int base, sx, sxy;   // LDS index of corner 0 and the strides in y and z
  uint32_t src[NE];    // source node of each staged word

  // false: this workgroup has no tile (uniform)
  __device__ __forceinline__ bool init(const Grid& g, int blk) {
    const int t = (blk % kXcds) * g.per_xcd + blk / kXcds;
    if (t >= g.tiles) return false;
    int32_t o[3];
    tile_coords<3>(g, t, o);
    const int per = class_items(g.tx, g.ty, SH::TZ);
    item = threadIdx.x;
    items = SH::NS * per;
    cls = __builtin_amdgcn_readfirstlane(item / per);
    const int l = item - cls * per;
    const int ix = l % g.tx, iyz = l / g.tx;
    const int iy = SH::TZ == 1 ? iyz : iyz % g.ty, iz = SH::TZ == 1 ? 0 : iyz / g.ty;
    o[0] *= g.tx;
    o[1] *= g.ty;
    o[2] *= SH::TZ;
    j[0] = o[0] + ix;
    j[1] = o[1] + iy;
    j[2] = o[2] + iz;
    active = iy < g.ty && iz < SH::TZ && j[0] < g.K[0] && j[1] < g.K[1] && j[2] < g.K[2];
    sx = g.tx + 1;
    sxy = sx * (g.ty + 1);
    total = (SH::TZ + 1) * sxy;
    base = ix + sx * min(iy, g.ty - 1) + sxy * min(iz, SH::TZ - 1);
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int e = min(item + k * items, total - 1);
      const int c[3] = {e % sx, (e / sx) % (g.ty + 1), e / sxy};
      int32_t n[3];
      bool outside = false;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        // the corners of the grid's nodes wrap at most once; words of nodes
        // outside the grid are clamped into the array and never used
        int32_t i = o[q] + g.soff + c[q];
        outside = outside || i < 0 || i >= g.sext[q];
        if (i < 0) i += g.sext[q];
        if (i >= g.sext[q]) i -= g.sext[q];
        n[q] = min(i, g.sext[q] - 1);
      }
      // past the plane: the buffer descriptor answers with zero
      src[k] = g.open && outside ? (uint32_t)g.snodes : node_index<3>(n[0], n[1], n[2], g.sext);
    }
    return true;
  }
  // Output node; outside the grid the first index past the plane, whose
  // loads the buffer descriptor answers with zero and whose stores it drops.
  __device__ __forceinline__ uint32_t out(const Grid& g) const {
    return active ? out_index<3>(g, j) : (uint32_t)g.onodes;
  }
};

// One work-item's node when it loads its own corners.
struct Direct3 {
  int32_t j[3];
  uint32_t cn[8];
  static constexpr bool active = true;
  static constexpr int cls = 0;
  // false: no node (per work-item)
  __device__ __forceinline__ bool init(const Grid& g, int blk) {
    if (!node_of_block<3>(g, blk, j)) return false;
    corner_nodes<3>(g, j, cn);
    return true;
  }
  // For an open grid: corners outside the source array are zero.
  __device__ __forceinline__ void open_corners(const Grid& g) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int32_t c = j[k] + g.soff + ((e >> k) & 1);
        if (c < 0 || c >= g.sext[k]) cn[e] = (uint32_t)g.snodes;  // past the plane: the descriptor answers with zero
      }
  }
  __device__ __forceinline__ uint32_t out(const Grid& g) const { return out_index<3>(g, j); }
};
template <class SH>
struct SourceOf {
  using type = Stage3<SH>;
};
template <>
struct SourceOf<DirectShape> {
  using type = Direct3;
};
template <class SH>
using Source3 = typename SourceOf<SH>::type;

// Issue the loads of plane pl's staged words.
template <class S, class SH>
__device__ __forceinline__ void stage_load(const typename S::View& f, int pl, const Stage3<SH>& st,
                                           typename S::Raw* r) {
  int zero;  // opaque: the plane base is formed here, not hoisted to the kernel start
  asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
  const typename S::Planes pr = S::planes(f, pl + zero);
#pragma unroll
  for (int k = 0; k < SH::NE; ++k)
    if (!SH::ANY || k * st.items < st.total) r[k] = S::raw_load(pr, st.src[k]);
}

template <class S, class SH>
__device__ __forceinline__ void stage_store(typename S::C* buf, const Stage3<SH>& st, const typename S::Raw* r) {
#pragma unroll
  for (int k = 0; k < SH::NE; ++k)
    if (!SH::ANY || k * st.items < st.total) buf[st.item + k * st.items] = S::value(r[k]);
}

// Corner combinations of the staged datum in X[k_x + 2 k_y + 4 k_z] (0 = sigma,
// 1 = delta); only those with k_x = KX when KX >= 0.
template <int KX, typename T>
__device__ __forceinline__ void butterfly3(const T* c, int sx, int sxy, T* X) {
  T x[8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const T* row = c + (q & 1) * sx + (q >> 1) * sxy;
    const T lo = row[0], hi = row[1];
    if (KX != 1) x[2 * q] = hi + lo;
    if (KX != 0) x[2 * q + 1] = hi - lo;
  }
#pragma unroll
  for (int kx = 0; kx < 2; ++kx) {
    if (KX >= 0 && kx != KX) continue;
    T y[4];  // [k_y + 2 e_z]
#pragma unroll
    for (int ez = 0; ez < 2; ++ez) {
      const T lo = x[kx + 4 * ez], hi = x[kx + 2 + 4 * ez];
      y[2 * ez] = hi + lo;
      y[1 + 2 * ez] = hi - lo;
    }
#pragma unroll
    for (int ky = 0; ky < 2; ++ky) {
      X[kx + 2 * ky] = y[ky + 2] + y[ky];
      X[kx + 2 * ky + 4] = y[ky + 2] - y[ky];
    }
  }
}

// Keeps an accumulator's arithmetic where it is written (no instruction):
// otherwise the compiler moves every datum's products past the last barrier,
// to where the sums are used, and holds all table entries in registers.
template <typename T>
__device__ __forceinline__ void pin(T& x) {
  asm volatile("" : "+v"(x));
}
// .. of a 3D half-step's accumulators (at m = 0 there is nothing to keep apart)
template <int M, typename T>
__device__ __forceinline__ void pin_acc(T& x) {
  if constexpr (M > 0) pin(x);
}

// A sum that carries its rounding errors along; the terms of one work-item are
// added plainly (exact products there changed no digit of the result).
struct ExactSum {
  double hi = 0.0, lo = 0.0;
  __device__ __forceinline__ void add(double x, double xlo) {
    const double t = hi + x, b = t - hi;
    lo += ((hi - (t - b)) + (x - b)) + xlo;
    hi = t;
  }
  __device__ __forceinline__ void add_product(double a, double b) {
    hi = fma(a, b, hi);
  }
};

// The data loop of one wavefront class: per datum q = 0 .. NQ - 1 (plane q of
// f) its staged corners' combinations X are handed to apply.  F::kx(q) is the
// combination in x that the class's outputs take (NS = 2).
template <class S, class SH, int Q, class F>
__device__ __forceinline__ void stage_datum(const Stage3<SH>& st, const typename S::C* buf, F& apply) {
  // keep the scalar table loads of one datum together (SGPR pressure)
  __builtin_amdgcn_sched_barrier(0);
  typename S::C X[8];
  butterfly3<SH::NS == 2 ? F::kx(Q) : -1>(buf + (Q % kStageGroup) * SH::CAP + st.base, st.sx, st.sxy, X);
  apply.template operator()<Q>(X);
}

template <int NQ, class S, class SH, int GR, class F, int... I>
__device__ __forceinline__ void stage_group(const typename S::View& f, const Stage3<SH>& st, typename S::C* lds,
                                            typename S::Raw (*r)[SH::NE], F& apply, std::integer_sequence<int, I...>) {
  constexpr int G = kStageGroup;
  __builtin_amdgcn_sched_barrier(0);
  typename S::C* buf = lds + (GR & 1) * G * SH::CAP;
#pragma unroll
  for (int i = 0; i < (int)sizeof...(I); ++i) stage_store<S, SH>(buf + i * SH::CAP, st, r[i]);
#pragma unroll
  for (int i = 0; i < G; ++i)
    if ((GR + 1) * G + i < NQ) stage_load<S, SH>(f, (GR + 1) * G + i, st, r[i]);
  __syncthreads();
  (stage_datum<S, SH, GR * G + I>(st, buf, apply), ...);
}

template <int NQ, class S, class SH, class F, int... GR>
__device__ __forceinline__ void stage_loop(const typename S::View& f, const Stage3<SH>& st, typename S::C* lds, F& apply,
                                           std::integer_sequence<int, GR...>) {
  constexpr int G = kStageGroup;
  typename S::Raw r[G][SH::NE];
#pragma unroll
  for (int i = 0; i < G && i < NQ; ++i) stage_load<S, SH>(f, i, st, r[i]);
  (stage_group<NQ, S, SH, GR>(f, st, lds, r, apply,
                              std::make_integer_sequence<int, ((GR + 1) * G <= NQ ? G : NQ - GR * G)>{}),
   ...);
}
template <int NQ>
using StageGroups = std::make_integer_sequence<int, (NQ + kStageGroup - 1) / kStageGroup>;

// The data loop of a work-item that loads its own corners, W - 1 data ahead.
template <class S>
__device__ __forceinline__ void direct_load(const typename S::View& f, int pl, const uint32_t* cn, typename S::C* v) {
  int zero;  // opaque: the plane base is formed here, not hoisted to the kernel start
  asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
  const typename S::Planes pr = S::planes(f, pl + zero);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = S::bload(pr, cn[e]);
}
template <int NQ, class S, int W, int Q, class F>
__device__ __forceinline__ void direct_datum(const typename S::View& f, const uint32_t* cn, typename S::C (*v)[8],
                                             F& apply) {
  // keep the scalar table loads of one datum together (SGPR pressure)
  if constexpr (NQ > 3) __builtin_amdgcn_sched_barrier(0);
  if constexpr (Q + W - 1 < NQ) direct_load<S>(f, Q + W - 1, cn, v[(Q + W - 1) % W]);
  typename S::C X[8];
  butterfly3<-1>(v[Q % W], 2, 4, X);
  apply.template operator()<Q>(X);
}
template <int NQ, class S, class F, int... Q>
__device__ __forceinline__ void direct_loop(const typename S::View& f, const uint32_t* cn, F& apply,
                                            std::integer_sequence<int, Q...>) {
  constexpr int W = NQ <= 3 ? NQ : 1;  // all of m = 0's data at once
  typename S::C v[W][8];
#pragma unroll
  for (int q = 0; q + 1 < W; ++q) direct_load<S>(f, q, cn, v[q]);
  (direct_datum<NQ, S, W, Q>(f, cn, v, apply), ...);
}

// The combinations of data 0 .. NQ - 1 of a node, handed to apply.
template <int NQ, class S, class SH, class F>
__device__ __forceinline__ void data_loop(const typename S::View& f, const Source3<SH>& st, typename S::C* lds,
                                          F& apply) {
  if constexpr (SH::DIRECT)
    direct_loop<NQ, S>(f, st.cn, apply, std::make_integer_sequence<int, NQ>{});
  else
    stage_loop<NQ, S, SH>(f, st, lds, apply, StageGroups<NQ>{});
}

template <int N>
struct IndexList {
  int n;
  short v[N];
};

// Pressure half-step, 3D.  Table F[i][a][rank(o)]: component i, datum a, output
// o.  Per node and datum at m = 2: 24 add/sub and 27 multiply-adds.
template <int M, class S, int CLS, int NS, typename TP>
struct PApply3 {
  using T = typename S::C;
  static constexpr int MP = M + 1, NC = Dims<3, M>::NC;
  TP tab;
  T acc[NC];
  static constexpr int kx(int q) { return (CLS + q % NC % MP + (q / NC == 0)) & 1; }
  static constexpr bool mine(int o) { return NS == 1 || ((o % MP) & 1) == CLS; }
  // the planes this class writes
  static constexpr IndexList<NC> outputs() {
    IndexList<NC> l{};
    for (int o = 0; o < NC; ++o)
      if (mine(o)) l.v[l.n++] = (short)o;
    return l;
  }
  static constexpr IndexList<NC> kOut = outputs();
  template <int Q>
  __device__ __forceinline__ void operator()(const T* X) {
    constexpr int i = Q / NC, a = Q % NC, ax = a % MP, ay = (a / MP) % MP, az = a / (MP * MP);
#pragma unroll
    for (int o = 0; o < NC; ++o) {
      if (!mine(o)) continue;
      const int ox = o % MP, oy = (o / MP) % MP, oz = o / (MP * MP);
      const int k = ((ox + ax + (i == 0)) & 1) + 2 * ((oy + ay + (i == 1)) & 1) + 4 * ((oz + az + (i == 2)) & 1);
      acc[o] = fma(tab[TableLayout<3, M>::F_OFF + Q * NC + kPRank<M>.r[o]], X[k], acc[o]);
    }
#pragma unroll
    for (int o = 0; o < NC; ++o)
      if (mine(o)) pin_acc<M>(acc[o]);
  }
};

// DOT: p is not updated; returns this work-item's part of -<p, increment>.
template <int M, class S, class SH, int CLS, bool DOT, typename TP>
__device__ __forceinline__ ExactSum p_half_3d_class(const typename S::View& p, const typename S::View& u, TP tab,
                                                    const Grid& g, const Source3<SH>& st, typename S::C* lds) {
  using T = typename S::C;
  constexpr int NC = Dims<3, M>::NC;
  using A = PApply3<M, S, CLS, SH::NS, TP>;
  A f;
  f.tab = tab;
#pragma unroll
  for (int s = 0; s < NC; ++s) f.acc[s] = T(0);
  data_loop<3 * NC, S, SH>(u, st, lds, f);
  const uint32_t n0 = st.out(g);
  if constexpr (DOT) {
    ExactSum d;
    if (st.active) {
#pragma unroll
      for (int k = 0; k < A::kOut.n; ++k)
        d.add_product((double)f.acc[A::kOut.v[k]], (double)load_output<3, S, false>(p, A::kOut.v[k], n0));
    }
    return d;
  } else {
    update_outputs<3, S, A::kOut.n>(g, p, n0, [](int k) { return A::kOut.v[k]; },
                                    [&](int k, T x) { return x - f.acc[A::kOut.v[k]]; });
    return {};
  }
}

template <int M, class S, class SH, typename TP, bool DOT = false>
__device__ __forceinline__ ExactSum p_half_3d_body(typename S::View p, typename S::View u, TP tab, Grid g, int blk) {
  __shared__ typename S::C lds[SH::LDS];
  Source3<SH> st;
  if (!st.init(g, blk)) return {};  // dual q = j - 1 + e
  if (SH::NS == 1 || st.cls == 0)
    return p_half_3d_class<M, S, SH, 0, DOT>(p, u, tab, g, st, lds);
  else if constexpr (SH::NS > 1)
    return p_half_3d_class<M, S, SH, 1, DOT>(p, u, tab, g, st, lds);
  return {};
}

template <int M, class S, int FORM>
__global__ void __launch_bounds__((256 * PShape<M, S, FORM>::NS * PShape<M, S, FORM>::TZ), HL_WAVES_PER_EU)
    p_half_3d(typename S::View p, typename S::View u, const typename S::C* __restrict__ tab, Grid g) {
  p_half_3d_body<M, S, PShape<M, S, FORM>, const typename S::C* __restrict__>(p, u, tab, g, blockIdx.x);
}

// Velocity half-step, 3D.  Table Fu[a][rank(o)]: datum a, member o of G.  Per
// node and datum at m = 2: 24 add/sub and 53 multiply-adds, split
// over two wavefront classes by the parity of the member's x index (29 and 24
// members): 12 add/sub each.
template <int M, class S, int CLS, int NS, typename TP>
struct UApply3 {
  using T = typename S::C;
  static constexpr int MP = M + 1, NG = GSet<3, M>::NG;
  TP tab;
  T Q[NG];
  static constexpr int kx(int a) { return (CLS + a % MP) & 1; }
  static constexpr bool mine(int o) { return NS == 1 || (kGSet<3, M>.dig[o][0] & 1) == CLS; }
  // the planes i NC + s this class writes: those whose member is its own
  static constexpr int NC = Dims<3, M>::NC;
  static constexpr IndexList<3 * NC> outputs() {
    IndexList<3 * NC> l{};
    for (int t = 0; t < 3 * NC; ++t)
      if (mine(kGIndex<3, M>.g[t / NC][t % NC])) l.v[l.n++] = (short)t;
    return l;
  }
  static constexpr IndexList<3 * NC> kOut = outputs();
  template <int A>
  __device__ __forceinline__ void operator()(const T* X) {
    constexpr int ax = A % MP, ay = (A / MP) % MP, az = A / (MP * MP);
#pragma unroll
    for (int o = 0; o < NG; ++o) {
      if (NS == 1 && o == NG / 2) __builtin_amdgcn_sched_barrier(0);  // two halves of the datum's table loads
      if (!mine(o)) continue;
      const int k = ((kGSet<3, M>.dig[o][0] + ax) & 1) + 2 * ((kGSet<3, M>.dig[o][1] + ay) & 1) +
                    4 * ((kGSet<3, M>.dig[o][2] + az) & 1);
      Q[o] = fma(tab[TableLayout<3, M>::FU_OFF + A * NG + kURank<M>.r[o]], X[k], Q[o]);
    }
#pragma unroll
    for (int o = 0; o < NG; ++o)
      if (mine(o)) pin_acc<M>(Q[o]);
  }
};

template <int M, class S, class SH, int CLS, bool DOT, typename TP>
__device__ __forceinline__ ExactSum u_half_3d_class(const typename S::View& u, const typename S::View& p, TP tab,
                                                const Grid& g, typename S::C wscale, const typename S::C* ih,
                                                const Source3<SH>& st, typename S::C* lds) {
  using T = typename S::C;
  constexpr int NC = Dims<3, M>::NC, MP = M + 1, NG = GSet<3, M>::NG;
  using A = UApply3<M, S, CLS, SH::NS, TP>;
  A f;
  f.tab = tab;
#pragma unroll
  for (int o = 0; o < NG; ++o) f.Q[o] = T(0);
  data_loop<NC, S, SH>(p, st, lds, f);
  const uint32_t n0 = st.out(g);
  // u_i[s] -= wscale * (s_i + 1) / h_i * Q[s + e_i]
  const T w[3] = {wscale * ih[0], wscale * ih[1], wscale * ih[2]};
  if constexpr (DOT) {
    ExactSum d;
    if (st.active) {
#pragma unroll
      for (int k = 0; k < A::kOut.n; ++k) {
        const int i = A::kOut.v[k] / NC, s = A::kOut.v[k] % NC;
        const T a = (T)(digit(s, MP, i) + 1) * w[i];
        d.add_product((double)(a * f.Q[kGIndex<3, M>.g[i][s]]), (double)load_output<3, S, false>(u, A::kOut.v[k], n0));
      }
    }
    return d;
  } else {
    update_outputs<3, S, A::kOut.n>(g, u, n0, [](int k) { return A::kOut.v[k]; }, [&](int k, T x) {
      const int i = A::kOut.v[k] / NC, s = A::kOut.v[k] % NC;
      const T a = -(T)(digit(s, MP, i) + 1) * w[i];
      return fma(a, f.Q[kGIndex<3, M>.g[i][s]], x);
    });
    return {};
  }
}

template <int M, class S, class SH, typename TP, bool DOT = false>
__device__ __forceinline__ ExactSum u_half_3d_body(typename S::View u, typename S::View p, TP tab, Grid g,
                                               typename S::C wscale, typename S::C ih0, typename S::C ih1,
                                               typename S::C ih2, int blk) {
  using T = typename S::C;
  __shared__ T lds[SH::LDS];
  Source3<SH> st;
  if (!st.init(g, blk)) return {};  // primal j = q + e
  const T ih[3] = {ih0, ih1, ih2};
  if (SH::NS == 1 || st.cls == 0)
    return u_half_3d_class<M, S, SH, 0, DOT>(u, p, tab, g, wscale, ih, st, lds);
  else if constexpr (SH::NS > 1)
    return u_half_3d_class<M, S, SH, 1, DOT>(u, p, tab, g, wscale, ih, st, lds);
  return {};
}

template <int M, class S, int FORM>
__global__ void __launch_bounds__((256 * UShape<M, S, FORM>::NS), HL_WAVES_PER_EU)
    u_half_3d(typename S::View u, typename S::View p, const typename S::C* __restrict__ tab, Grid g,
              typename S::C wscale, typename S::C ih0, typename S::C ih1, typename S::C ih2) {
  u_half_3d_body<M, S, UShape<M, S, FORM>, const typename S::C* __restrict__>(u, p, tab, g, wscale, ih0, ih1, ih2,
                                                                             blockIdx.x);
}

// ---------------------------------------------------------------------------
// Ghost dual nodes for reflecting walls (Sec. 5, "Imposing reflective boundary
// conditions"): p = 0 on the walls makes p odd across each wall, so by
// u_t = -grad p the normal velocity component is even and the tangential ones
// odd.  The velocity array is padded by one node per side (extents E_k =
// K_k + 2); each shell node is the mirror of the interior node reached by
// reflecting every ghost index across its wall (0 <- 1, E-1 <- E-2).  A scaled
// coefficient mirrored in dimension k gets (-1)^{a_k}, and -1 more for a
// tangential component (i != k).  Edge and corner ghosts are mirrors in
// several dimensions at once.
//
// Launch: grid (ceil(max face nodes / 256), D, plane groups), block 256.  A
// work-item takes kGhostPlanes planes of one shell node, their loads before
// their stores: with every plane in turn (each load waiting for the store
// before it) the shell of a 1001 x 777 box, m = 3 FP32, took 13.7 us, now 5.1.
// Face k (grid y) holds the shell nodes whose first ghost index is in dimension k: index k in
// {0, E_k - 1}, indices j < k interior, indices j > k anything; every shell
// node is written by exactly one work-item.
// ---------------------------------------------------------------------------
constexpr int kGhostPlanes = 4;
template <int D, int M, class S>
__global__ void __launch_bounds__(256) ghost_fill(typename S::View u, int32_t E0, int32_t E1, int32_t E2) {
  using T = typename S::C;
  constexpr int MP = M + 1, NC = Dims<D, M>::NC;
  const int32_t E[3] = {E0, E1, E2};
  const int k = blockIdx.y;
  int64_t cnt = 2;
  for (int j = 0; j < D; ++j)
    if (j != k) cnt *= (j < k) ? (E[j] - 2) : E[j];
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= cnt) return;
  int32_t idx[3] = {0, 0, 0};
  int64_t r = t / 2;
  for (int j = 0; j < D; ++j) {
    if (j == k) {
      idx[j] = (t % 2) ? E[j] - 1 : 0;
    } else if (j < k) {
      idx[j] = 1 + (int32_t)(r % (E[j] - 2));
      r /= (E[j] - 2);
    } else {
      idx[j] = (int32_t)(r % E[j]);
      r /= E[j];
    }
  }
  int32_t src[3] = {0, 0, 0};
  bool mir[3] = {false, false, false};
  for (int j = 0; j < D; ++j) {
    mir[j] = idx[j] == 0 || idx[j] == E[j] - 1;
    src[j] = idx[j] == 0 ? 1 : (idx[j] == E[j] - 1 ? E[j] - 2 : idx[j]);
  }
  const uint32_t n_dst = node_index<D>(idx[0], idx[1], idx[2], E);
  const uint32_t n_src = node_index<D>(src[0], src[1], src[2], E);
  const int pl0 = blockIdx.z * kGhostPlanes;
  T v[kGhostPlanes];
#pragma unroll
  for (int q = 0; q < kGhostPlanes; ++q) v[q] = S::load(u, min(pl0 + q, D * NC - 1), n_src);
#pragma unroll
  for (int q = 0; q < kGhostPlanes; ++q) {
    const int pl = pl0 + q;
    if (pl >= D * NC) break;
    const int i = pl / NC, c = pl % NC;
    bool neg = false;
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (mir[j]) neg ^= ((digit(c, MP, j) & 1) != 0) != (i != j);
    S::store(u, pl, n_dst, neg ? -v[q] : v[q]);
  }
}

}  // namespace hl
