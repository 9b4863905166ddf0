// hl_kernels_ext.hpp - kernels beyond the constant-coefficient step: the
// discrete adjoint (periodic and walled), the variable-coefficient half-steps
// and their adjoint, the batched-shot launches and their sources.  They reuse
// the half-step bodies and helpers of hl_kernels.hpp.
#pragma once

#include "hl_kernels.hpp"

namespace hl {

// ---------------------------------------------------------------------------
// Discrete adjoint.  A step maps (P, U) to P' = P - A U, U' = U - B P'; its
// transpose is Pb <- Pb - B^T Ub, then Ub <- Ub - A^T Pb: the transposed
// half-steps in reverse order.  On the periodic grid each transposed half-step
// is again a gather with the forward stencil: B^T Ub at primal node j reads
// the dual nodes q = j - 1 + e' (the pressure half-step's corners) and A^T Pb
// at dual node q reads the primal nodes j = q + e' (the velocity half-step's),
// so no atomics are needed.  The operator of corner e' is that of the all-
// upper corner up to sign: -1 for a lower corner in a dimension k in which
// r_k + c_k + [k = i] is odd (output coefficient r, input coefficient c,
// velocity component i on either side), because every interpolant coefficient
// that links them has the parity of that component's derivative.  So, as in
// the forward half-steps, an output takes one sigma / delta combination of the
// 2^D corners of each datum times one table entry (1D: both corners, each times
// the entry with its sign): 2^D times fewer multiply-adds than a dense block per
// corner (2D m = 2 512^2 FP64 16 + 17 us; 34 + 37 us with dense blocks; 3D m = 2
// 17496 multiply-adds per node and half-step against 2187).
//   PTYPE = true:  out = Pb (1 component), in = Ub (D components)
//   PTYPE = false: out = Ub (D components), in = Pb (1 component)
// Table: entry (t, o), datum t = (input component, c), output o = (output
// component, r), built on the host from the same interpolation and weight
// operators as the forward tables; in 3D the outputs of a row are stored even
// r_x + [i = 0] first (pressure: the forward table's order, so that Pb runs
// the pressure half-step's own kernel on it).
// With reflecting walls the step is P' = P - A G U, U' = U - B P', G the ghost
// refresh; Ub -= G^T A^T Pb goes through a zeroed scratch array shaped like
// the padded velocity: A^T Pb on every slot (an open grid: primal corners past
// a wall contribute nothing), then the fold G^T (ghost_fold).  B writes no
// ghost, so the ghost slots of Ub are held at zero.
// ---------------------------------------------------------------------------
// OPEN: an open grid (a kernel of its own, so that the others hold no code for it).
template <int D, int M, class S, bool PTYPE, bool OPEN>
__global__ void __launch_bounds__(256) adjoint_half(typename S::View out, typename S::View in,
                                                    const typename S::C* __restrict__ tab, Grid g) {
  static_assert(D <= 2, "3D uses the staged kernels");
  using T = typename S::C;
  constexpr int MP = M + 1, NC = Dims<D, M>::NC, NI = PTYPE ? D : 1, NO = PTYPE ? NC : D * NC, NE = 1 << D;
  int32_t j[3];
  if (!node_of_block<D>(g, blockIdx.x, j)) return;
  uint32_t cn[NE];
  corner_nodes<D>(g, j, cn);
  bool in_grid[NE];
  if constexpr (OPEN) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      in_grid[e] = true;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const int c = j[k] + g.soff + ((e >> k) & 1);
        in_grid[e] = in_grid[e] && c >= 0 && c < g.sext[k];
      }
      if (!in_grid[e]) cn[e] = 0;
    }
  }
  auto corner = [&](int t, int e) {
    const T x = S::load(in, t, cn[e]);
    if constexpr (OPEN) return in_grid[e] ? x : T(0);
    return x;
  };
  const auto update = [&](const T* acc) {
    update_outputs<D, S, NO>(g, out, out_index<D>(g, j), [](int o) { return o; }, [&](int o, T x) { return x - acc[o]; });
  };
  T acc[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o) acc[o] = T(0);
  if constexpr (D == 1) {
    // Two corners: sums and differences save little and round more than each
    // corner's own products (one half-step FP32 m = 1: 1.2 times as far off
    // FP64), and all data are few enough to be loaded at once.
    T v[NE][NC];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int t = 0; t < NC; ++t) v[e][t] = corner(t, e);
#pragma unroll
    for (int e = 0; e < NE; ++e)  // corner by corner: their sums cancel for large m
#pragma unroll
      for (int t = 0; t < NC; ++t) {
        // keep the scalar table loads of one datum together (SGPR pressure)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          const T w = tab[t * NO + o];
          acc[o] = fma(e == 0 && ((o + t + 1) & 1) ? -w : w, v[e][t], acc[o]);
        }
      }
    return update(acc);
  }
  T vn[NE];  // the next datum's corners, loaded one datum ahead
#pragma unroll
  for (int e = 0; e < NE; ++e) vn[e] = corner(0, e);
#pragma unroll
  for (int t = 0; t < NI * NC; ++t) {
    // keep the scalar table loads of one datum together (SGPR pressure)
    __builtin_amdgcn_sched_barrier(0);
    T X[NE], v[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) v[e] = vn[e];
    if (t + 1 < NI * NC) {
#pragma unroll
      for (int e = 0; e < NE; ++e) vn[e] = corner(t + 1, e);
    }
#pragma unroll
    for (int q = 0; q < NE / 2; ++q) {
      X[2 * q] = v[2 * q + 1] + v[2 * q];
      X[2 * q + 1] = v[2 * q + 1] - v[2 * q];
    }
    if constexpr (D == 2) {
#pragma unroll
      for (int kx = 0; kx < 2; ++kx) {
        const T lo = X[kx], hi = X[kx + 2];
        X[kx] = hi + lo;
        X[kx + 2] = hi - lo;
      }
    }
    const int c = t % NC;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      const int r = o % NC, i = PTYPE ? t / NC : o / NC;
      int k = 0;
#pragma unroll
      for (int d = 0; d < D; ++d) k += ((digit(r, MP, d) + digit(c, MP, d) + (d == i)) & 1) << d;
      acc[o] = fma(tab[t * NO + o], X[k], acc[o]);
    }
  }
  update(acc);
}

// Ub -= A^T Pb in 3D: the velocity half-step's staging and wavefront classes
// with 3 (m+1)^3 outputs, a class taking one parity of r_x + [i = 0].
template <int M>
struct ARank {
  short r[3 * Dims<3, M>::NC];
  static constexpr int par(int o) { return (o % (M + 1) + (o / Dims<3, M>::NC == 0)) & 1; }
  constexpr ARank() : r() {
    int n = 0;
    for (int p = 0; p < 2; ++p)
      for (int o = 0; o < 3 * Dims<3, M>::NC; ++o)
        if (par(o) == p) r[o] = (short)n++;
  }
};
template <int M>
inline constexpr ARank<M> kARank{};

template <int M, class S, int CLS, int NS, typename TP>
struct AApply3 {
  using T = typename S::C;
  static constexpr int MP = M + 1, NC = Dims<3, M>::NC, NO = 3 * NC;
  TP tab;
  T acc[NO];
  static constexpr int kx(int a) { return (CLS + a % MP) & 1; }
  static constexpr bool mine(int o) { return NS == 1 || ARank<M>::par(o) == CLS; }
  static constexpr IndexList<NO> outputs() {
    IndexList<NO> l{};
    for (int o = 0; o < NO; ++o)
      if (mine(o)) l.v[l.n++] = (short)o;
    return l;
  }
  static constexpr IndexList<NO> kOut = outputs();
  template <int A>
  __device__ __forceinline__ void operator()(const T* X) {
    constexpr int ax = A % MP, ay = (A / MP) % MP, az = A / (MP * MP);
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      if (!mine(o)) continue;
      const int i = o / NC, r = o % NC;
      const int k = ((r % MP + ax + (i == 0)) & 1) + 2 * (((r / MP) % MP + ay + (i == 1)) & 1) +
                    4 * ((r / (MP * MP) + az + (i == 2)) & 1);
      acc[o] = fma(tab[A * NO + kARank<M>.r[o]], X[k], acc[o]);
    }
#pragma unroll
    for (int o = 0; o < NO; ++o)
      if (mine(o)) pin_acc<M>(acc[o]);
  }
};

template <int M, class S, class SH, int CLS, typename TP>
__device__ __forceinline__ void adjoint_u_3d_class(const typename S::View& out, const typename S::View& in, TP tab,
                                                   const Grid& g, const Source3<SH>& st, typename S::C* lds) {
  using T = typename S::C;
  using A = AApply3<M, S, CLS, SH::NS, TP>;
  A f;
  f.tab = tab;
#pragma unroll
  for (int o = 0; o < A::NO; ++o) f.acc[o] = T(0);
  data_loop<A::NC, S, SH>(in, st, lds, f);
  update_outputs<3, S, A::kOut.n>(g, out, st.out(g), [](int k) { return A::kOut.v[k]; },
                                  [&](int k, T x) { return x - f.acc[A::kOut.v[k]]; });
}

template <int M, class S>
__global__ void __launch_bounds__((256 * UShape<M, S, kAnyTile>::NS)) adjoint_u_3d(
    typename S::View out, typename S::View in, const typename S::C* __restrict__ tab, Grid g) {
  using SH = UShape<M, S, kAnyTile>;
  __shared__ typename S::C lds[SH::LDS];
  Source3<SH> st;
  if (!st.init(g, blockIdx.x)) return;
  if constexpr (SH::DIRECT)
    if (g.open) st.open_corners(g);
  if (SH::NS == 1 || st.cls == 0)
    adjoint_u_3d_class<M, S, SH, 0>(out, in, tab, g, st, lds);
  else if constexpr (SH::NS > 1)
    adjoint_u_3d_class<M, S, SH, 1>(out, in, tab, g, st, lds);
}

// ---------------------------------------------------------------------------
// Inner products of a field with a half-step's increment, without forming the
// increment: part[workgroup] -= <pb, A U> (pressure tables) or <ub, B P>.
// The kappa gradient takes them with the kappa-derivative tables once per step;
// a workgroup adds to its own entry, so the sum over steps has a fixed order.
// The terms of smooth fields may all but cancel over the grid (orthogonal modes:
// a sum of 1e-13 from terms of 1e4 in all), so the sums over work-items,
// workgroups and steps carry their rounding errors along (hi, lo).
// Against storing the increment and a dot product over the whole arrays,
// 2D m = 2 512^2 FP64: 15 + 13 us instead of 17 + 28 + 17 + 19 us and two clears.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void add_block_sum(ExactSum d, double* part) {
  __shared__ double red[2][16];
  const int tid = threadIdx.x + blockDim.x * threadIdx.y, n = blockDim.x * blockDim.y;
  const int lane = tid & 63, lanes = min(64, n - (tid & ~63));
  for (int k = 32; k > 0; k >>= 1) {
    const double x = __shfl_down(d.hi, k), xl = __shfl_down(d.lo, k);
    if (lane + k < lanes) d.add(x, xl);
  }
  if (lane == 0) {
    red[0][tid >> 6] = d.hi;
    red[1][tid >> 6] = d.lo;
  }
  __syncthreads();
  if (tid == 0) {
    ExactSum s{part[2 * blockIdx.x], part[2 * blockIdx.x + 1]};
    for (int w = 0; w < (n + 63) / 64; ++w) s.add(-red[0][w], -red[1][w]);
    part[2 * blockIdx.x] = s.hi;
    part[2 * blockIdx.x + 1] = s.lo;
  }
}

template <int D, int M, class S>
__global__ void __launch_bounds__(256) p_dot(typename S::View pb, typename S::View u,
                                             const typename S::C* __restrict__ tab, Grid g, double* part) {
  static_assert(D <= 2, "3D uses the staged kernels");
  using T = typename S::C;
  int32_t j[3];
  ExactSum d;
  if (node_of_block<D>(g, blockIdx.x, j)) {
    uint32_t cn[1 << D];
    corner_nodes<D>(g, j, cn);
    T acc[Dims<D, M>::NC];
    p_half_acc<D, M, S>(u, tab, cn, acc);
    const uint32_t n0 = out_index<D>(g, j);
#pragma unroll
    for (int s = 0; s < Dims<D, M>::NC; ++s) d.add_product((double)acc[s], (double)S::load(pb, s, n0));
  }
  add_block_sum(d, part);
}

template <int D, int M, class S>
__global__ void __launch_bounds__(256) u_dot(typename S::View ub, typename S::View p,
                                             const typename S::C* __restrict__ tab, Grid g, typename S::C ih0,
                                             typename S::C ih1, double* part) {
  static_assert(D <= 2, "3D uses the staged kernels");
  using T = typename S::C;
  constexpr int MP = M + 1, NC = Dims<D, M>::NC;
  int32_t j[3];
  ExactSum d;
  if (node_of_block<D>(g, blockIdx.x, j)) {
    uint32_t cn[1 << D];
    corner_nodes<D>(g, j, cn);
    T Q[GSet<D, M>::NG];
    u_half_Q<D, M, S>(p, tab, cn, Q);
    const uint32_t n0 = out_index<D>(g, j);
    const T ih[2] = {ih0, ih1};
#pragma unroll
    for (int t = 0; t < D * NC; ++t) {
      const int i = t / NC, s = t % NC;
      const T a = (T)(digit(s, MP, i) + 1) * ih[i];
      d.add_product((double)(a * Q[kGIndex<D, M>.g[i][s]]), (double)S::load(ub, t, n0));
    }
  }
  add_block_sum(d, part);
}

template <int M, class S>
__global__ void __launch_bounds__((256 * PShape<M, S, kAnyTile>::NS)) p_dot_3d(typename S::View pb,
                                                                               typename S::View u,
                                                                               const typename S::C* __restrict__ tab,
                                                                               Grid g, double* part) {
  add_block_sum(p_half_3d_body<M, S, PShape<M, S, kAnyTile>, const typename S::C* __restrict__, true>(pb, u, tab, g,
                                                                                                      blockIdx.x),
                part);
}

template <int M, class S>
__global__ void __launch_bounds__((256 * UShape<M, S, kAnyTile>::NS)) u_dot_3d(
    typename S::View ub, typename S::View p, const typename S::C* __restrict__ tab, Grid g, typename S::C ih0,
    typename S::C ih1, typename S::C ih2, double* part) {
  add_block_sum(u_half_3d_body<M, S, UShape<M, S, kAnyTile>, const typename S::C* __restrict__, true>(
                    ub, p, tab, g, typename S::C(1), ih0, ih1, ih2, blockIdx.x),
                part);
}

// G^T: ub[q] += scr[q] + sum over the ghost slots mirroring q of the signed
// ghost value, and every scratch slot read is cleared (each ghost mirrors
// exactly one interior node, so each slot is read once).  One work-item per
// interior dual node and kGhostPlanes planes (grid y), their loads before
// their stores; E the padded extents.
template <int D, int M, class S>
__global__ void __launch_bounds__(256) ghost_fold(typename S::View ub, typename S::View scr, int32_t E0, int32_t E1,
                                                  int32_t E2) {
  using T = typename S::C;
  constexpr int MP = M + 1, NC = Dims<D, M>::NC;
  const int32_t E[3] = {E0, E1, E2};
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int32_t q[3] = {1, 1, 1};  // padded index of the interior node
  int64_t total = 1;
  for (int k = 0; k < D; ++k) total *= E[k] - 2;
  if (t >= total) return;
  for (int k = 0; k < D; ++k) {
    q[k] = 1 + (int32_t)(t % (E[k] - 2));
    t /= (E[k] - 2);
  }
  // dimensions where q touches a wall and the ghost index across it
  int32_t gidx[3] = {0, 0, 0};
  bool at[3] = {false, false, false};
  for (int k = 0; k < D; ++k) {
    if (q[k] == 1) {
      at[k] = true;
      gidx[k] = 0;
    } else if (q[k] == E[k] - 2) {
      at[k] = true;
      gidx[k] = E[k] - 1;
    }
  }
  const uint32_t n_q = node_index<D>(q[0], q[1], q[2], E);
  const int pl0 = blockIdx.y * kGhostPlanes;
  bool wall = false;
  for (int k = 0; k < D; ++k) wall = wall || at[k];
  T v[kGhostPlanes], x[kGhostPlanes];
#pragma unroll
  for (int p = 0; p < kGhostPlanes; ++p) {
    const int pl = min(pl0 + p, D * NC - 1);
    v[p] = S::load(scr, pl, n_q);
    x[p] = S::load(ub, pl, n_q);
  }
#pragma unroll
  for (int p = 0; p < kGhostPlanes; ++p) {
    const int pl = pl0 + p;
    if (pl >= D * NC) break;
    S::store(scr, pl, n_q, T(0));
    if (wall) {
      // every nonempty subset R of the wall dimensions: the ghost reflected in R
      const int i = pl / NC, c = pl % NC;
#pragma unroll
      for (int R = 1; R < (1 << D); ++R) {
        bool ok = true, neg = false;
        int32_t gq[3] = {q[0], q[1], q[2]};
#pragma unroll
        for (int k = 0; k < D; ++k)
          if ((R >> k) & 1) {
            ok = ok && at[k];
            gq[k] = gidx[k];
            neg ^= ((digit(c, MP, k) & 1) != 0) != (i != k);
          }
        if (!ok) continue;
        const uint32_t n_g = node_index<D>(gq[0], gq[1], gq[2], E);
        const T w = S::load(scr, pl, n_g);
        S::store(scr, pl, n_g, T(0));
        v[p] += neg ? -w : w;
      }
    }
    S::store(ub, pl, n_q, x[p] + v[p]);
  }
}

// Zero the ghost shell of a padded velocity array (E the padded extents).
template <int D, int M, class S>
__global__ void __launch_bounds__(256) ghost_zero(typename S::View u, int32_t E0, int32_t E1, int32_t E2) {
  using T = typename S::C;
  constexpr int NC = Dims<D, M>::NC;
  const int32_t E[3] = {E0, E1, E2};
  int64_t total = 1;
  for (int k = 0; k < D; ++k) total *= E[k];
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  int32_t idx[3] = {0, 0, 0};
  bool shell = false;
  for (int k = 0; k < D; ++k) {
    idx[k] = (int32_t)(t % E[k]);
    t /= E[k];
    shell = shell || idx[k] == 0 || idx[k] == E[k] - 1;
  }
  if (!shell) return;
  const uint32_t n = node_index<D>(idx[0], idx[1], idx[2], E);
  for (int pl = 0; pl < D * NC; ++pl) S::store(u, pl, n, T(0));
}

// ---------------------------------------------------------------------------
// Variable coefficient kappa(x) (Sec. 4, "Smoothly varying wave speed"):
// kappa is given per node as a Taylor polynomial of degree 2m+1 per variable
// (scaled like the data), about the primal nodes for the pressure half-step
// and the dual nodes for the velocity half-step.  From p_t = -kappa div u and
// u_t = -grad p the odd time derivatives are
//   d_t^{2k+1} p = -(kappa Lap)^k (kappa div u),   d_t^{2k+1} u = -grad (kappa Lap)^k p,
// evaluated on the cell polynomials with every product truncated to degree
// 2m+1 per variable, k = 0..kmax, kmax = d m (the last k at which Lap^k of a
// polynomial of degree 2m+1 in each variable can be nonzero, i.e. where the
// constant-coefficient series ends; with variable kappa the series would go
// on, and this length is a reading for d >= 2):
//   P <- P - sum_k w_k r_k,   r_0 = T[kappa div c],  r_k = T[kappa Lap r_{k-1}]
//   U_i <- U_i - sum_k w_k D_i g_k,   g_0 = c,  g_k = T[kappa Lap g_{k-1}].
// No operator can be merged into a constant table here (kappa differs per
// cell), so the kernels build the full (2m+2)^d interpolant in registers, one
// work-item per node (d = 1, d = 2, and d = 3 with m <= 1); 3D m >= 2 uses
// one wavefront per node (below).
// ---------------------------------------------------------------------------
template <int D, int M>
struct VK {
  static constexpr int N2 = 2 * M + 2, MP = M + 1;
  static constexpr int NP = ipow(N2, D);            // cell polynomial coefficients
  static constexpr int KMAX = D * M;
};

// w_k / w_{k-1} for k = 1..kVarMaxK (kmax = d m <= 10 for every built (d, m):
// 2D m = 5 reaches 10).
constexpr int kVarMaxK = 10;

// The series is accumulated as t_k = w_k r_k with t_k = (w_k / w_{k-1})
// T[kappa Lap t_{k-1}]: the ratio (dt/2)^2 / (2k (2k+1)) cancels the 1/h^2 of
// each Laplacian, so every term stays O(1) (r_k alone grows like h^{-2k} and
// overflows FP32 for large m).
template <typename T>
struct VarArgs {
  T w0;        // w_0 = dt
  T ratio[kVarMaxK + 1];  // w_k / w_{k-1} = (dt/2)^2 / (2k (2k+1)), k = 1..kmax
  T ih[3];     // 1 / h_k
};

// Coefficients a half-step's result depends on.  t_k = T[kappa Lap t_{k-1}]
// feeds the result directly on the output set (pressure: {0..m}^D; velocity,
// VEL: s + e_i with s in {0..m}^D) and through the remaining J = kmax - k
// Laplacians, each of which reads two orders up in one variable; a product's
// coefficient b reads its operands at all orders <= b.  So t_k and the operand
// Lap t_{k-1} are formed only on the coefficients b of need(b) <= J, need(b)
// the least number of Laplacians from b down into the output set; every kept
// coefficient is the same sum in the same order.  Multiply-adds of the products
// of one half-step against full products: 2D m = 3 6120 of 9072 (pressure),
// 3D m = 2 37044 of 64827.
template <int D, int M, bool VEL>
struct Need {
  static constexpr int N2 = 2 * M + 2, NP = ipow(N2, D);
  static constexpr int over(int b, int top) { return b > top ? (b - top + 1) / 2 : 0; }
  // per-variable orders (b_x, b_y, b_z), 0 beyond D
  static constexpr int of(int bx, int by, int bz) {
    const int dg[3] = {bx, by, bz};
    int best = 99;
    for (int i = 0; i < (VEL ? D : 1); ++i) {
      int n = 0;
      for (int k = 0; k < D; ++k) n += over(dg[k], VEL && k == i ? M + 1 : M);
      best = n < best ? n : best;
    }
    return best;
  }
  static constexpr int at(int b) { return of(b % N2, D > 1 ? (b / N2) % N2 : 0, D > 2 ? b / (N2 * N2) : 0); }
  static constexpr int top() {
    int t = 0;
    for (int b = 0; b < NP; ++b) t = at(b) > t ? at(b) : t;
    return t;
  }
  signed char n[NP];
  constexpr Need() : n() {
    for (int b = 0; b < NP; ++b) n[b] = (signed char)at(b);
  }
};
template <int D, int M, bool VEL>
inline constexpr Need<D, M, VEL> kNeed{};
// Products from J = kNeedTop on are full.
template <int D, int M, bool VEL>
constexpr int kNeedTop = Need<D, M, VEL>::top();

// The truncated products of the adjoint kernels load their kappa terms in
// groups of kKappaGroup, each group issued while the previous one is applied.
// The plane base of every load is formed from an opaque scalar zero taken
// once per group: otherwise the compiler keeps one 64-bit address per kappa
// plane for the whole kernel (2 VGPRs per term: 128 at 2D m = 3), and with
// the scheduling barrier after each group it cannot hoist every load of a
// product to its start either.
constexpr int kKappaGroup = 4;

// out_b += kappa_A f_{b-A} (TR = false: T[kappa f]) or out_b += kappa_A f_{A+b}
// (TR = true: T^T[kappa] f), for one term A.
// Only coefficients of need <= J (J >= kNeedTop: all).
template <int D, int M, bool VEL, int J, bool TR, int A, typename T>
__device__ __forceinline__ void kterm_apply(T ka, const T* f, T* out) {
  constexpr int N2 = 2 * M + 2, AX = A % N2, AY = (A / N2) % N2, AZ = A / (N2 * N2);
  constexpr int NY = D > 1 ? N2 : 1, NZ = D > 2 ? N2 : 1;
#pragma unroll
  for (int bz = 0; bz + AZ < NZ; ++bz)
#pragma unroll
    for (int by = 0; by + AY < NY; ++by)
#pragma unroll
      for (int bx = 0; bx + AX < N2; ++bx) {
        const int lo = bx + N2 * (by + N2 * bz), hi = (bx + AX) + N2 * ((by + AY) + N2 * (bz + AZ));
        if (kNeed<D, M, VEL>.n[hi] > J) continue;
        if constexpr (TR)
          out[lo] = fma(ka, f[hi], out[lo]);
        else
          out[hi] = fma(ka, f[lo], out[hi]);
      }
}

template <int D, int M, bool VEL, int J, bool TR, int BASE, typename T, int... I>
__device__ __forceinline__ void kgroup_apply(const T* kc, const T* f, T* out, std::integer_sequence<int, I...>) {
  (kterm_apply<D, M, VEL, J, TR, BASE + I>(kc[I], f, out), ...);
}

// kb[i] = kappa_{BASE + i} for the terms BASE + i < NP of need <= J.
template <class S, int D, int M, bool VEL, int J, int BASE, int NP>
__device__ __forceinline__ void kgroup_load(const typename S::View& kv, uint32_t n0, typename S::C* kb) {
  int zero;
  asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
#pragma unroll
  for (int i = 0; i < kKappaGroup; ++i)
    if (BASE + i < NP && kNeed<D, M, VEL>.n[BASE + i < NP ? BASE + i : 0] <= J)
      kb[i] = S::load(kv, BASE + i + zero, n0);
}

template <int D, int M, bool VEL, int J, bool TR, class S, int GRP>
__device__ __forceinline__ void kgroup_step(const typename S::View& kv, uint32_t n0, const typename S::C* f,
                                            typename S::C* out, typename S::C (*kb)[kKappaGroup]) {
  constexpr int G = kKappaGroup, NP = VK<D, M>::NP, NG = (NP + G - 1) / G;
  constexpr int CNT = NP - GRP * G < G ? NP - GRP * G : G;
  if constexpr (GRP + 1 < NG) kgroup_load<S, D, M, VEL, J, (GRP + 1) * G, NP>(kv, n0, kb[(GRP + 1) & 1]);
  kgroup_apply<D, M, VEL, J, TR, GRP * G>(kb[GRP & 1], f, out, std::make_integer_sequence<int, CNT>{});
  __builtin_amdgcn_sched_barrier(0);
}

template <int D, int M, bool VEL, int J, bool TR, class S, int... GRP>
__device__ __forceinline__ void kgroup_steps(const typename S::View& kv, uint32_t n0, const typename S::C* f,
                                             typename S::C* out, std::integer_sequence<int, GRP...>) {
  typename S::C kb[2][kKappaGroup];
  kgroup_load<S, D, M, VEL, J, 0, VK<D, M>::NP>(kv, n0, kb[0]);
  (kgroup_step<D, M, VEL, J, TR, S, GRP>(kv, n0, f, out, kb), ...);
}

// out = T[kappa f] (TR = false) or T^T[kappa] f (TR = true) on the coefficients
// of need <= J, kappa_a read from plane a of the kappa array at node n0.  The
// same terms in the same order as tprod.  (TR: f is zero off that set, and so
// is the result.)
template <int D, int M, bool VEL, int J, bool TR, class S>
__device__ __forceinline__ void tprod_grouped(const typename S::View& kv, uint32_t n0, const typename S::C* f,
                                              typename S::C* out) {
  using T = typename S::C;
  constexpr int NP = VK<D, M>::NP, NG = (NP + kKappaGroup - 1) / kKappaGroup;
#pragma unroll
  for (int b = 0; b < NP; ++b) out[b] = T(0);
  kgroup_steps<D, M, VEL, J, TR, S>(kv, n0, f, out, std::make_integer_sequence<int, NG>{});
}

// The forward variable-kappa half-steps take the grouped kappa loads from
// m = 4 on, where the per-term loads' addresses spill (2D m = 4 FP64: 788 ->
// 124 bytes of scratch per lane, m = 5 FP32: 507 -> 359 VGPRs); below, the
// per-term loads measured faster (2D m = 3 1024^2 FP32 0.86 against 0.91 ms).
template <int D, int M, bool VEL, int J, class S>
__device__ __forceinline__ void tprod_fwd(const typename S::View& kv, uint32_t n0, const typename S::C* f,
                                          typename S::C* out) {
  if constexpr (M >= 4)
    tprod_grouped<D, M, VEL, J, false, S>(kv, n0, f, out);
  else
    tprod<D, M, VEL, J, S>(kv, n0, f, out);
}

// Full interpolant c[b_x + N2 (b_y + N2 b_z)] of one component from its 2^D
// corner blocks.
template <int D, int M, class S>
__device__ __forceinline__ void interp_full(const typename S::View& f, int comp, const uint32_t* cn,
                                            typename S::C* c) {
  using T = typename S::C;
  constexpr int MP = M + 1, N2 = 2 * M + 2, NC = Dims<D, M>::NC;
  if constexpr (D == 3) {
    // x pass on the 8 corners' x-lines per (a_y, a_z), then y, then z
    T Xc[2][2][MP][MP][N2];  // [e_y][e_z][a_y][a_z][b_x]
#pragma unroll
    for (int ez = 0; ez < 2; ++ez)
#pragma unroll
      for (int ey = 0; ey < 2; ++ey)
#pragma unroll
        for (int az = 0; az < MP; ++az)
#pragma unroll
          for (int ay = 0; ay < MP; ++ay) {
            T L[MP], R[MP];
#pragma unroll
            for (int ax = 0; ax < MP; ++ax) {
              const int pl = comp * NC + ax + MP * (ay + MP * az);
              L[ax] = S::load(f, pl, cn[0 + 2 * ey + 4 * ez]);
              R[ax] = S::load(f, pl, cn[1 + 2 * ey + 4 * ez]);
            }
            pass1d<M, 0>(L, R, Xc[ey][ez][ay][az]);
          }
    T Yc[2][MP][N2][N2];  // [e_z][a_z][b_x][b_y]
#pragma unroll
    for (int ez = 0; ez < 2; ++ez)
#pragma unroll
      for (int az = 0; az < MP; ++az)
#pragma unroll
        for (int bx = 0; bx < N2; ++bx) {
          T L[MP], R[MP];
#pragma unroll
          for (int ay = 0; ay < MP; ++ay) {
            L[ay] = Xc[0][ez][ay][az][bx];
            R[ay] = Xc[1][ez][ay][az][bx];
          }
          pass1d<M, 0>(L, R, Yc[ez][az][bx]);
        }
#pragma unroll
    for (int by = 0; by < N2; ++by)
#pragma unroll
      for (int bx = 0; bx < N2; ++bx) {
        T L[MP], R[MP], out[N2];
#pragma unroll
        for (int az = 0; az < MP; ++az) {
          L[az] = Yc[0][az][bx][by];
          R[az] = Yc[1][az][bx][by];
        }
        pass1d<M, 0>(L, R, out);
#pragma unroll
        for (int bz = 0; bz < N2; ++bz) c[bx + N2 * (by + N2 * bz)] = out[bz];
      }
  } else if constexpr (D == 1) {
    T L[MP], R[MP];
#pragma unroll
    for (int a = 0; a < MP; ++a) {
      L[a] = S::load(f, comp * NC + a, cn[0]);
      R[a] = S::load(f, comp * NC + a, cn[1]);
    }
    pass1d<M, 0>(L, R, c);
  } else {
    T Yl[MP][N2], Yh[MP][N2];  // x pass at the lower / upper y corners, per a_y
#pragma unroll
    for (int ay = 0; ay < MP; ++ay) {
      T L[MP], R[MP];
#pragma unroll
      for (int ax = 0; ax < MP; ++ax) {
        L[ax] = S::load(f, comp * NC + ax + MP * ay, cn[0]);
        R[ax] = S::load(f, comp * NC + ax + MP * ay, cn[1]);
      }
      pass1d<M, 0>(L, R, Yl[ay]);
#pragma unroll
      for (int ax = 0; ax < MP; ++ax) {
        L[ax] = S::load(f, comp * NC + ax + MP * ay, cn[2]);
        R[ax] = S::load(f, comp * NC + ax + MP * ay, cn[3]);
      }
      pass1d<M, 0>(L, R, Yh[ay]);
    }
#pragma unroll
    for (int bx = 0; bx < N2; ++bx) {
      T L[MP], R[MP], out[N2];
#pragma unroll
      for (int ay = 0; ay < MP; ++ay) {
        L[ay] = Yl[ay][bx];
        R[ay] = Yh[ay][bx];
      }
      pass1d<M, 0>(L, R, out);
#pragma unroll
      for (int by = 0; by < N2; ++by) c[bx + N2 * by] = out[by];
    }
  }
}

// out += kappa_A f shifted by A (one term of the truncated product; A is a
// template argument so that every register index is a compile-time constant:
// as one 64 x 64 loop nest the compiler stopped unrolling and indexed f
// through scratch memory).
template <int D, int M, bool VEL, int J, int A, class S>
__device__ __forceinline__ void tprod_term(const typename S::View& kv, uint32_t n0, const typename S::C* f,
                                           typename S::C* out) {
  constexpr int N2 = 2 * M + 2, AX = A % N2, AY = (A / N2) % N2, AZ = A / (N2 * N2);
  constexpr int NY = D > 1 ? N2 : 1, NZ = D > 2 ? N2 : 1;
  if constexpr (kNeed<D, M, VEL>.n[A] > J) return;
  const typename S::C ka = S::load(kv, A, n0);
#pragma unroll
  for (int bz = AZ; bz < NZ; ++bz)
#pragma unroll
    for (int by = AY; by < NY; ++by)
#pragma unroll
      for (int bx = AX; bx < N2; ++bx) {
        const int o = bx + N2 * (by + N2 * bz);
        if (kNeed<D, M, VEL>.n[o] > J) continue;
        out[o] = fma(ka, f[(bx - AX) + N2 * ((by - AY) + N2 * (bz - AZ))], out[o]);
      }
}

template <int D, int M, bool VEL, int J, class S, int... A>
__device__ __forceinline__ void tprod_terms(const typename S::View& kv, uint32_t n0, const typename S::C* f,
                                            typename S::C* out, std::integer_sequence<int, A...>) {
  (tprod_term<D, M, VEL, J, A, S>(kv, n0, f, out), ...);
}

// out = T[kappa f]: out_b = sum_{a <= b} kappa_a f_{b-a} (per variable) on the
// coefficients of need <= J, kappa_a read from plane a of the kappa array at
// node n0.
template <int D, int M, bool VEL, int J, class S>
__device__ __forceinline__ void tprod(const typename S::View& kv, uint32_t n0, const typename S::C* f,
                                      typename S::C* out) {
  using T = typename S::C;
  constexpr int NP = VK<D, M>::NP;
#pragma unroll
  for (int b = 0; b < NP; ++b) out[b] = T(0);
  tprod_terms<D, M, VEL, J, S>(kv, n0, f, out, std::make_integer_sequence<int, NP>{});
}

// out = sc Lap f in coefficient space: sc sum_i (b_i + 1)(b_i + 2) / h_i^2 f_{b + 2 e_i}.
// On the coefficients of need <= J.
template <int D, int M, bool VEL, int J, typename T>
__device__ __forceinline__ void lap_coef(const T* f, T* out, const T* ih, T sc) {
  constexpr int N2 = 2 * M + 2, NP = VK<D, M>::NP;
  const T ix2 = sc * ih[0] * ih[0], iy2 = sc * ih[1] * ih[1], iz2 = sc * ih[2] * ih[2];
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    const int bx = b % N2, by = (b / N2) % N2, bz = b / (N2 * N2);
    if (kNeed<D, M, VEL>.n[b] > J) continue;
    T v = T(0);
    if (bx + 2 < N2) v = fma(T((bx + 1) * (bx + 2)) * ix2, f[b + 2], v);
    if (D > 1 && by + 2 < N2) v = fma(T((by + 1) * (by + 2)) * iy2, f[b + 2 * N2], v);
    if (D > 2 && bz + 2 < N2) v = fma(T((bz + 1) * (bz + 2)) * iz2, f[b + 2 * N2 * N2], v);
    out[b] = v;
  }
}

// Index of the cell-polynomial coefficient s + delta (s in {0..m}^D in the
// data's order, delta a shift per dimension) in the (2m+2)^D layout.
template <int D, int M>
__host__ __device__ constexpr int poly_index(int s, int dx, int dy, int dz) {
  constexpr int MP = M + 1, N2 = 2 * M + 2;
  const int sx = s % MP, sy = D > 1 ? (s / MP) % MP : 0, sz = D > 2 ? s / (MP * MP) : 0;
  return (sx + dx) + N2 * ((sy + dy) + N2 * (sz + dz));
}

// t_k = T[kappa (w_k / w_{k-1}) Lap t_{k-1}] for k = 1 .. kmax, each handed to
// add: a loop while the products are full, then one unrolled step per J.
template <int D, int M, bool VEL, int J, class S, class F>
__device__ __forceinline__ void var_series_tail(const typename S::View& kv, uint32_t n0, typename S::C* t,
                                                const VarArgs<typename S::C>& va, F& add) {
  if constexpr (J >= 0) {
    using T = typename S::C;
    T l[VK<D, M>::NP];
    lap_coef<D, M, VEL, J>(t, l, va.ih, va.ratio[VK<D, M>::KMAX - J]);
    tprod_fwd<D, M, VEL, J, S>(kv, n0, l, t);
    add(t);
    var_series_tail<D, M, VEL, J - 1, S>(kv, n0, t, va, add);
  }
}
// Steps taken unrolled (m >= 4: none, full products throughout: one copy of an
// already long product; the last steps' own copies spill) and in the loop.
template <int D, int M, bool VEL>
constexpr int kSeriesTop = M >= 4 ? 0 : kNeedTop<D, M, VEL>;
template <int D, int M, bool VEL>
constexpr int kSeriesLoops = VK<D, M>::KMAX > kSeriesTop<D, M, VEL> ? VK<D, M>::KMAX - kSeriesTop<D, M, VEL> : 0;
template <int D, int M, bool VEL, class S, class F>
__device__ __forceinline__ void var_series(const typename S::View& kv, uint32_t n0, typename S::C* t,
                                           const VarArgs<typename S::C>& va, F& add) {
  using T = typename S::C;
  constexpr int KMAX = VK<D, M>::KMAX, TOP = kSeriesTop<D, M, VEL>;
#pragma unroll 1
  for (int k = 1; k <= kSeriesLoops<D, M, VEL>; ++k) {
    T l[VK<D, M>::NP];
    lap_coef<D, M, VEL, KMAX>(t, l, va.ih, va.ratio[k]);
    tprod_fwd<D, M, VEL, KMAX, S>(kv, n0, l, t);
    add(t);
  }
  var_series_tail<D, M, VEL, (TOP - 1 < KMAX - 1 ? TOP - 1 : KMAX - 1), S>(kv, n0, t, va, add);
}

template <int D, int M, class S>
__device__ __forceinline__ void p_half_var_body(typename S::View p, typename S::View u, typename S::View kp,
                                                Grid g, VarArgs<typename S::C> va, int blk) {
  using T = typename S::C;
  constexpr int N2 = 2 * M + 2, MP = M + 1, NP = VK<D, M>::NP, NC = Dims<D, M>::NC;
  static_assert(VK<D, M>::KMAX <= kVarMaxK, "series longer than the ratio table");
  int32_t j[3];
  if (!node_of_block<D>(g, blk, j)) return;
  uint32_t cn[1 << D];
  corner_nodes<D>(g, j, cn);  // dual q = j - 1 + e
  const uint32_t n0 = out_index<D>(g, j);
  T div[NP];  // w_0 div c
#pragma unroll
  for (int b = 0; b < NP; ++b) div[b] = T(0);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    T c[NP];
    interp_full<D, M, S>(u, i, cn, c);
    const int st = i == 0 ? 1 : i == 1 ? N2 : N2 * N2;
    const T f = va.w0 * va.ih[i];
#pragma unroll
    for (int b = 0; b < NP; ++b) {
      const int bi = (b / st) % N2;
      if (bi + 1 < N2) div[b] = fma(T(bi + 1) * f, c[b + st], div[b]);
    }
  }
  T t[NP], acc[NC];
  tprod_fwd<D, M, false, VK<D, M>::KMAX, S>(kp, n0, div, t);  // t_0 = w_0 r_0
#pragma unroll
  for (int s = 0; s < NC; ++s) acc[s] = t[poly_index<D, M>(s, 0, 0, 0)];
  auto add = [&](const T* x) {
#pragma unroll
    for (int s = 0; s < NC; ++s) acc[s] += x[poly_index<D, M>(s, 0, 0, 0)];
  };
  var_series<D, M, false, S>(kp, n0, t, va, add);
  finish_pressure<D, M, S>(g, p, n0, acc);
}

template <int D, int M, class S>
__global__ void __launch_bounds__(256) p_half_var(typename S::View p, typename S::View u, typename S::View kp,
                                                  Grid g, VarArgs<typename S::C> va) {
  p_half_var_body<D, M, S>(p, u, kp, g, va, blockIdx.x);
}

template <int D, int M, class S>
__device__ __forceinline__ void u_half_var_body(typename S::View u, typename S::View p, typename S::View ku,
                                                Grid g, VarArgs<typename S::C> va, typename S::C wscale, int blk) {
  using T = typename S::C;
  constexpr int N2 = 2 * M + 2, MP = M + 1, NP = VK<D, M>::NP, NC = Dims<D, M>::NC;
  int32_t j[3];
  if (!node_of_block<D>(g, blk, j)) return;
  uint32_t cn[1 << D];
  corner_nodes<D>(g, j, cn);  // primal j = q + e
  const uint32_t n0 = out_index<D>(g, j);
  T gk[NP], q[NP];  // gk: t_k = w_k g_k; q: their sum on the output set (need 0)
  interp_full<D, M, S>(p, 0, cn, gk);
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    gk[b] *= va.w0;
    q[b] = gk[b];
    // rounded before the first t_k is added also where that addition is not in
    // a loop (which keeps them apart by itself, but 2D m = 3 FP32 is 3% faster
    // pinned, m = 4 6% slower); with a single term the product and the sum are
    // one multiply-add, which rounds less
    if constexpr (VK<D, M>::KMAX > 1 && (M < 4 || kSeriesLoops<D, M, true> < 2)) pin(q[b]);
  }
  auto add = [&](const T* x) {
#pragma unroll
    for (int b = 0; b < NP; ++b)
      if (kNeed<D, M, true>.n[b] == 0) q[b] += x[b];
  };
  var_series<D, M, true, S>(ku, n0, gk, va, add);
  // u_i[s] -= wscale (s_i + 1) / h_i q[s + e_i]
  T f[D];
#pragma unroll
  for (int i = 0; i < D; ++i) f[i] = wscale * va.ih[i];
  update_outputs_as<D, S, D * NC, false>(u, n0, [](int t) { return t; }, [&](int t, T x) {
    const int i = t / NC, s = t % NC;
    const T a = -(T)(digit(s, MP, i) + 1) * f[i];
    return fma(a, q[poly_index<D, M>(s, i == 0, i == 1, i == 2)], x);
  });
}

template <int D, int M, class S>
__global__ void __launch_bounds__(256) u_half_var(typename S::View u, typename S::View p, typename S::View ku,
                                                  Grid g, VarArgs<typename S::C> va, typename S::C wscale) {
  u_half_var_body<D, M, S>(u, p, ku, g, va, wscale, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Variable kappa, 3D m = 2 and 3: one wavefront per node.  The cell
// polynomial has (2m+2)^3 coefficients per field (216 at m = 2, 512 at
// m = 3): two of them (the current term and its Laplacian) no longer fit in
// one work-item's registers, so the 64 work-items of a workgroup share one
// node.  Its polynomials live in LDS, and in the products and Laplacians
// lane l < (2m+2)^2 owns the x-pencil b_y = l mod (2m+2), b_z = l div (2m+2)
// (2m+2 coefficients along x, held in registers).  The arithmetic is that of
// the per-node kernels above (the same tensor-product passes, and the same
// products kappa_a f_{b-a}), except that a pencil's sum is formed from partial
// sums over chunks of its terms (below).
// ---------------------------------------------------------------------------
template <int M>
struct VW {
  static constexpr int MP = M + 1, N2 = 2 * M + 2, NP = N2 * N2 * N2, NPEN = N2 * N2, NC = MP * MP * MP;
  static_assert(NPEN <= 64 && 8 * NC == NP && 4 * MP * MP == NPEN, "one pencil and one line per lane");
};

// Wavefronts per SIMD asked for.  FP64 (8.3 KB of LDS per node at m = 2) takes
// 120 to 128 registers and 4 of them (5 spill: velocity 56^3 1160 us against
// 1065); FP32 fits 8 with a few words of scratch (64^3 1280 + 1080 us; 5 of
// them 1340 + 1113).
template <class S>
constexpr int kVarWaves = sizeof(typename S::C) == 8 ? 4 : 8;

// Node of workgroup blk when every workgroup updates one node: consecutive
// node numbers (x fastest) go to one XCD, so neighbours share its L2.
__device__ __forceinline__ bool wave_node(const Grid& g, int blk, int32_t per_xcd, int32_t* j) {
  const int64_t t = (int64_t)(blk % kXcds) * per_xcd + blk / kXcds;
  if (t >= (int64_t)g.K[0] * g.K[1] * g.K[2]) return false;
  j[0] = (int32_t)(t % g.K[0]);
  j[1] = (int32_t)((t / g.K[0]) % g.K[1]);
  j[2] = (int32_t)(t / ((int64_t)g.K[0] * g.K[1]));
  return true;
}

// Corner e of the node's cell (bit k of e: upper side in dimension k), wrapped
// as corner_nodes wraps it.
__device__ __forceinline__ uint32_t corner_node_of(const Grid& g, const int32_t* j, int e) {
  int32_t c[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    int32_t lo = j[k] + g.soff, hi = lo + 1;
    if (lo < 0) lo += g.sext[k];
    if (hi == g.sext[k]) hi = 0;
    c[k] = ((e >> k) & 1) ? hi : lo;
  }
  return node_index<3>(c[0], c[1], c[2], g.sext);
}

// This lane's corner words of one component: corner lane mod 8, coefficients
// lane div 8 + 8 i.  All of a node's words (and kappa's, and the outputs' old
// values) are loaded before the first is used: loaded where they are used,
// each component waited for memory by itself, and each output plane for the
// store of the one before it.  m = 2 56^3 FP64 1365 + 1137 -> 1250 + 1065 us,
// 64^3 FP32 1400 + 1220 -> 1280 + 1080 us.
template <int M>
constexpr int kCornerWords = (VW<M>::NC + 7) / 8;
template <int M, class S>
__device__ __forceinline__ void corner_words(const typename S::View& f, int comp, uint32_t cnl, int lane,
                                             typename S::C* w) {
  constexpr int NC = VW<M>::NC;
#pragma unroll
  for (int i = 0; i < kCornerWords<M>; ++i) w[i] = S::load(f, comp * NC + min((lane >> 3) + 8 * i, NC - 1), cnl);
}
template <int M, class S>
struct KappaWords {
  static constexpr int NP = VW<M>::NP, W = (NP + 63) / 64;
  typename S::C w[W];
  __device__ __forceinline__ void load(const typename S::View& kv, uint32_t n0, int lane) {
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = S::load(kv, min(lane + 64 * i, NP - 1), n0);
  }
  __device__ __forceinline__ void put(int lane, typename S::C* KA) const {
#pragma unroll
    for (int i = 0; i < W; ++i)
      if (lane + 64 * i < NP) KA[lane + 64 * i] = w[i];
  }
};

// Full interpolant of one component (its corner words w) into
// B[b_x + N2 (b_y + N2 b_z)], through A: the raw corner data A[e + 8 a], the x pass into B (line ey + 2 ez + 4
// (ay + MP az), entries b_x), the y pass into A (line ez + 2 (az + MP b_x),
// entries b_y), the z pass into B.  Every line is one lane's.
template <int M, typename T>
__device__ __forceinline__ void interp_wave(const T* w, int lane, T* A, T* B) {
  constexpr int MP = VW<M>::MP, N2 = VW<M>::N2, NC = VW<M>::NC, NL = VW<M>::NPEN;
#pragma unroll
  for (int i = 0; i < kCornerWords<M>; ++i)
    if ((lane >> 3) + 8 * i < NC) A[(lane & 7) + 8 * ((lane >> 3) + 8 * i)] = w[i];
  __syncthreads();
  if (lane < NL) {
    const int ey = lane & 1, ez = (lane >> 1) & 1, ay = (lane >> 2) % MP, az = (lane >> 2) / MP;
    T L[MP], R[MP], o[N2];
#pragma unroll
    for (int ax = 0; ax < MP; ++ax) {
      const int a = ax + MP * (ay + MP * az);
      L[ax] = A[2 * ey + 4 * ez + 8 * a];
      R[ax] = A[1 + 2 * ey + 4 * ez + 8 * a];
    }
    pass1d<M, 0>(L, R, o);
#pragma unroll
    for (int b = 0; b < N2; ++b) B[lane * N2 + b] = o[b];
  }
  __syncthreads();
  if (lane < NL) {
    const int ez = lane & 1, az = (lane >> 1) % MP, bx = (lane >> 1) / MP;
    T L[MP], R[MP], o[N2];
#pragma unroll
    for (int ay = 0; ay < MP; ++ay) {
      L[ay] = B[(2 * ez + 4 * (ay + MP * az)) * N2 + bx];
      R[ay] = B[(1 + 2 * ez + 4 * (ay + MP * az)) * N2 + bx];
    }
    pass1d<M, 0>(L, R, o);
#pragma unroll
    for (int b = 0; b < N2; ++b) A[lane * N2 + b] = o[b];
  }
  __syncthreads();
  if (lane < NL) {
    const int bx = lane % N2, by = lane / N2;
    T L[MP], R[MP], o[N2];
#pragma unroll
    for (int az = 0; az < MP; ++az) {
      L[az] = A[(2 * (az + MP * bx)) * N2 + by];
      R[az] = A[(1 + 2 * (az + MP * bx)) * N2 + by];
    }
    pass1d<M, 0>(L, R, o);
#pragma unroll
    for (int b = 0; b < N2; ++b) B[bx + N2 * (by + N2 * b)] = o[b];
  }
  __syncthreads();
}

// Work split of one truncated product over the 64 lanes.  The product is
// formed on the pencils with a coefficient of need <= J (above), on the first
// XL coefficients of each (the most any of them needs).  Pencil (by, bz) sums
// over the (by+1)(bz+1) pairs (a_y, a_z) <= (by, bz) (a_z outer), 1 to
// (2m+2)^2 of them; one lane per pencil would wait on the longest.  Instead
// every pencil's pairs are cut into chunks of at most C consecutive pairs, one
// chunk per lane, C the smallest length that needs at most 64 chunks (m = 2:
// C = 10 for a full product, 1 for the last), and each pencil then adds its
// chunks' partial sums in chunk order.  Pairs the longest lane walks in one
// half-step: m = 2 pressure 70 with full products, 49 so; m = 3 640 with
// full products, 453 so.
template <int M, bool VEL, int J>
struct WaveSched {
  static constexpr int N2 = 2 * M + 2;
  using ND = Need<3, M, VEL>;
  int C, n, xl, pairs;
  uint32_t chunk[64];  // lane -> by, bz, first pair, pairs (a byte each)
  uint32_t pen[64];    // pencil -> its first chunk, chunks
  static constexpr bool needed(int q) { return ND::of(0, q % N2, q / N2) <= J; }
  static constexpr int weight(int q) { return (q % N2 + 1) * (q / N2 + 1); }
  constexpr WaveSched() : C(1), n(0), xl(0), pairs(0), chunk(), pen() {
    for (int b = 0; b < N2; ++b)
      if (ND::of(b, 0, 0) <= J) xl = b + 1;
    for (;; ++C) {
      int k = 0;
      for (int q = 0; q < N2 * N2; ++q)
        if (needed(q)) k += (weight(q) + C - 1) / C;
      if (k <= 64) break;
    }
    for (int q = 0; q < N2 * N2; ++q) {
      if (!needed(q)) continue;
      const int w = weight(q);
      pen[q] = (uint32_t)(n | ((w + C - 1) / C) << 8);
      for (int i = 0; i < w; i += C, ++n) {
        const int cnt = w - i < C ? w - i : C;
        chunk[n] = (uint32_t)(q % N2 | (q / N2) << 8 | i << 16 | cnt << 24);
        pairs += cnt;
      }
    }
  }
  // every needed pencil's pairs covered once, in order, by its chunks
  constexpr bool ok() const {
    if (n > 64) return false;
    int total = 0;
    for (int q = 0; q < N2 * N2; ++q) {
      if (!needed(q)) continue;
      int next = 0;
      const int first = pen[q] & 255, nch = pen[q] >> 8;
      for (int c = first; c < first + nch; ++c) {
        if ((int)(chunk[c] & 255) != q % N2 || (int)((chunk[c] >> 8) & 255) != q / N2) return false;
        if ((int)((chunk[c] >> 16) & 255) != next) return false;
        const int cnt = chunk[c] >> 24;
        if (cnt < 1 || cnt > C) return false;
        next += cnt;
      }
      if (next != weight(q)) return false;
      total += next;
    }
    return total == pairs;
  }
};
template <int M, bool VEL, int J>
__device__ constexpr WaveSched<M, VEL, J> kWaveSched{};
static_assert(kWaveSched<2, false, 6>.ok() && kWaveSched<2, false, 6>.C == 10 && kWaveSched<2, false, 6>.n == 60, "");
static_assert(kWaveSched<2, false, 0>.ok() && kWaveSched<2, false, 0>.C == 1 && kWaveSched<2, false, 0>.xl == 3, "");
static_assert(kWaveSched<2, true, 1>.ok() && kWaveSched<3, false, 6>.ok() && kWaveSched<3, true, 2>.ok(), "");

// Partial sum of pencil (by, bz) of T[kappa f] over the pairs i0 .. i0+cnt-1:
// out[b_x] = sum of kappa_a f_{b-a}, a_x <= b_x < XL, K and F in LDS.
template <int M, int XL, typename T>
__device__ __forceinline__ void tprod_chunk(const T* KA, const T* F, uint32_t chunk, T* out) {
  constexpr int N2 = VW<M>::N2;
  const int by = chunk & 255, bz = (chunk >> 8) & 255, i0 = (chunk >> 16) & 255, cnt = chunk >> 24;
#pragma unroll
  for (int b = 0; b < XL; ++b) out[b] = T(0);
  int ay = i0 % (by + 1), az = i0 / (by + 1);
  for (int i = 0; i < cnt; ++i) {
    T kp[XL], fp[XL];
    const T* kr = KA + N2 * (ay + N2 * az);
    const T* fr = F + N2 * ((by - ay) + N2 * (bz - az));
#pragma unroll
    for (int b = 0; b < XL; ++b) {
      kp[b] = kr[b];
      fp[b] = fr[b];
    }
#pragma unroll
    for (int bx = 0; bx < XL; ++bx)
#pragma unroll
      for (int ax = 0; ax <= bx; ++ax) out[bx] = fma(kp[ax], fp[bx - ax], out[bx]);
    if (++ay > by) {
      ay = 0;
      ++az;
    }
  }
}

// This lane's pencil, and its chunk of every product (one schedule per J up to
// the first full product).
template <int M, bool VEL>
struct WaveLane {
  static constexpr int TOP = kNeedTop<3, M, VEL>, N2 = VW<M>::N2;
  int lane;
  bool pen;  // lane < (2m+2)^2 owns pencil (by, bz) = (lane mod N2, lane div N2)
  int by, bz;
  uint32_t chunk[TOP + 1], tot[TOP + 1];
  template <int... J>
  __device__ __forceinline__ void load(std::integer_sequence<int, J...>) {
    ((chunk[J] = kWaveSched<M, VEL, J>.chunk[lane], tot[J] = kWaveSched<M, VEL, J>.pen[lane]), ...);
  }
  __device__ __forceinline__ explicit WaveLane(int l) : lane(l) {
    pen = l < VW<M>::NPEN;
    by = pen ? l % N2 : 0;
    bz = pen ? l / N2 : 0;
    load(std::make_integer_sequence<int, TOP + 1>{});
  }
};

// t = pencil (by, bz) of T[kappa F] on the owning lanes, its first XL
// coefficients; RED: 64 (2m+2) partial sums.  Begins and ends with LDS reads
// only; callers separate it from the next writes of F and RED by a barrier.
template <int M, bool VEL, int J, typename T>
__device__ __forceinline__ void tprod_wave(const T* KA, const T* F, T* RED, const WaveLane<M, VEL>& w, T* t) {
  constexpr int N2 = VW<M>::N2, JJ = J < kNeedTop<3, M, VEL> ? J : kNeedTop<3, M, VEL>;
  constexpr int XL = kWaveSched<M, VEL, JJ>.xl;
  T part[XL];
  tprod_chunk<M, XL>(KA, F, w.chunk[JJ], part);
#pragma unroll
  for (int b = 0; b < XL; ++b) RED[w.lane * N2 + b] = part[b];
  __syncthreads();
#pragma unroll
  for (int b = 0; b < XL; ++b) t[b] = T(0);
  const int first = w.tot[JJ] & 255, nch = w.tot[JJ] >> 8;
  for (int q = 0; q < nch; ++q) {
#pragma unroll
    for (int b = 0; b < XL; ++b) t[b] += RED[(first + q) * N2 + b];
  }
}

// Pencil (by, bz) of sc Lap t (coefficient space), t in LDS.
template <int M, int XL, typename T>
__device__ __forceinline__ void lap_pencil(const T* t, int by, int bz, const T* ih, T sc, T* out) {
  constexpr int N2 = VW<M>::N2;
  const T ix2 = sc * ih[0] * ih[0], iy2 = sc * ih[1] * ih[1], iz2 = sc * ih[2] * ih[2];
  const T* r0 = t + N2 * (by + N2 * bz);
#pragma unroll
  for (int bx = 0; bx < XL; ++bx) {
    T v = T(0);
    if (bx + 2 < N2) v = fma(T((bx + 1) * (bx + 2)) * ix2, r0[bx + 2], v);
    if (by + 2 < N2) v = fma(T((by + 1) * (by + 2)) * iy2, r0[bx + 2 * N2], v);
    if (bz + 2 < N2) v = fma(T((bz + 1) * (bz + 2)) * iz2, r0[bx + 2 * N2 * N2], v);
    out[bx] = v;
  }
}

// One step of the series at J: t <- T[kappa r Lap t] on the lane's pencil, for
// the pencils and coefficients of need <= J.  Coefficients beyond hold no
// defined value and reach none that is needed.
template <int M, bool VEL, int J, typename T>
__device__ __forceinline__ void wave_step(const T* KA, T* F, T* Tc, T* RED, const WaveLane<M, VEL>& w, const T* ih,
                                          T ratio, T* t) {
  constexpr int N2 = VW<M>::N2, TOP = kNeedTop<3, M, VEL>;
  constexpr int XL = kWaveSched<M, VEL, (J < TOP ? J : TOP)>.xl;
  constexpr int XT = kWaveSched<M, VEL, (J + 1 < TOP ? J + 1 : TOP)>.xl;
  if (w.pen) {
#pragma unroll
    for (int b = 0; b < XT; ++b) Tc[N2 * (w.by + N2 * w.bz) + b] = t[b];
  }
  __syncthreads();
  if (w.pen) {
    T l[XL];
    lap_pencil<M, XL>(Tc, w.by, w.bz, ih, ratio, l);
#pragma unroll
    for (int b = 0; b < XL; ++b) F[N2 * (w.by + N2 * w.bz) + b] = l[b];
  }
  __syncthreads();
  tprod_wave<M, VEL, J>(KA, F, RED, w, t);
}
template <int M, bool VEL, int J, typename T, class FA>
__device__ __forceinline__ void wave_series_tail(const T* KA, T* F, T* Tc, T* RED, const WaveLane<M, VEL>& w,
                                                 const VarArgs<T>& va, T* t, FA& add) {
  if constexpr (J >= 0) {
    wave_step<M, VEL, J>(KA, F, Tc, RED, w, va.ih, va.ratio[VK<3, M>::KMAX - J], t);
    add(t);
    wave_series_tail<M, VEL, J - 1>(KA, F, Tc, RED, w, va, t, add);
  }
}
template <int M, bool VEL, typename T, class FA>
__device__ __forceinline__ void wave_series(const T* KA, T* F, T* Tc, T* RED, const WaveLane<M, VEL>& w,
                                            const VarArgs<T>& va, T* t, FA& add) {
  constexpr int KMAX = VK<3, M>::KMAX, TOP = kNeedTop<3, M, VEL>;
#pragma unroll 1
  for (int k = 1; k <= KMAX - TOP; ++k) {
    wave_step<M, VEL, KMAX>(KA, F, Tc, RED, w, va.ih, va.ratio[k], t);
    add(t);
  }
  wave_series_tail<M, VEL, (TOP < KMAX ? TOP : KMAX) - 1>(KA, F, Tc, RED, w, va, t, add);
}

template <int M, class S>
__device__ __forceinline__ void p_half_var_wave_body(typename S::View p, typename S::View u, typename S::View kp,
                                                     Grid g, VarArgs<typename S::C> va, int32_t per_xcd, int blk) {
  using T = typename S::C;
  constexpr int MP = VW<M>::MP, N2 = VW<M>::N2, NP = VW<M>::NP;
  static_assert(VK<3, M>::KMAX <= kVarMaxK, "series longer than the ratio table");
  __shared__ T A[NP], B[NP], KA[NP], RED[64 * N2];
  int32_t j[3];
  if (!wave_node(g, blk, per_xcd, j)) return;  // uniform over the workgroup
  const int lane = threadIdx.x;
  const WaveLane<M, false> w(lane);
  const uint32_t n0 = out_index<3>(g, j);
  const uint32_t cnl = corner_node_of(g, j, lane & 7);  // dual q = j - 1 + e
  const bool pen = w.pen;
  const int by = w.by, bz = w.bz;
  const bool own = pen && by < MP && bz < MP;  // pencil holds data entries (b_x < MP)
  KappaWords<M, S> kw;
  T cw[3][kCornerWords<M>], old[MP];
  kw.load(kp, n0, lane);
#pragma unroll
  for (int i = 0; i < 3; ++i) corner_words<M, S>(u, i, cnl, lane, cw[i]);
  if (own) {
#pragma unroll
    for (int bx = 0; bx < MP; ++bx) old[bx] = S::load(p, bx + MP * (by + MP * bz), n0);
  }
  kw.put(lane, KA);
  T dv[N2];  // w_0 div c on the lane's pencil
#pragma unroll
  for (int b = 0; b < N2; ++b) dv[b] = T(0);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    interp_wave<M>(cw[i], lane, A, B);
    if (pen) {
      const T f = va.w0 * va.ih[i];
      const T* r = B + N2 * (by + N2 * bz);
#pragma unroll
      for (int bx = 0; bx < N2; ++bx) {
        if (i == 0 && bx + 1 < N2) dv[bx] = fma(T(bx + 1) * f, r[bx + 1], dv[bx]);
        if (i == 1 && by + 1 < N2) dv[bx] = fma(T(by + 1) * f, r[bx + N2], dv[bx]);
        if (i == 2 && bz + 1 < N2) dv[bx] = fma(T(bz + 1) * f, r[bx + N2 * N2], dv[bx]);
      }
    }
    __syncthreads();
  }
  T* F = A;  // Laplacian of the current term (input of the product)
  T* Tc = B;  // current term t_k
  if (pen) {
#pragma unroll
    for (int b = 0; b < N2; ++b) F[N2 * (by + N2 * bz) + b] = dv[b];
  }
  __syncthreads();
  T acc[MP], t[N2];
#pragma unroll
  for (int b = 0; b < N2; ++b) t[b] = T(0);
  tprod_wave<M, false, VK<3, M>::KMAX>(KA, F, RED, w, t);  // t_0 = w_0 r_0
#pragma unroll
  for (int b = 0; b < MP; ++b) acc[b] = t[b];
  auto add = [&](const T* x) {
#pragma unroll
    for (int b = 0; b < MP; ++b) acc[b] += x[b];
  };
  wave_series<M, false>(KA, F, Tc, RED, w, va, t, add);
  if (own) {
#pragma unroll
    for (int bx = 0; bx < MP; ++bx) S::store(p, bx + MP * (by + MP * bz), n0, old[bx] - acc[bx]);
  }
}

template <int M, class S>
__device__ __forceinline__ void u_half_var_wave_body(typename S::View u, typename S::View p, typename S::View ku,
                                                     Grid g, VarArgs<typename S::C> va, typename S::C wscale,
                                                     int32_t per_xcd, int blk) {
  using T = typename S::C;
  constexpr int MP = VW<M>::MP, N2 = VW<M>::N2, NP = VW<M>::NP, NC = VW<M>::NC;
  __shared__ T A[NP], B[NP], KA[NP], RED[64 * N2];
  int32_t j[3];
  if (!wave_node(g, blk, per_xcd, j)) return;  // uniform over the workgroup
  const int lane = threadIdx.x;
  const WaveLane<M, true> w(lane);
  const uint32_t n0 = out_index<3>(g, j);
  const uint32_t cnl = corner_node_of(g, j, lane & 7);  // primal j = q + e
  const bool pen = w.pen;
  const int by = w.by, bz = w.bz;
  // u_i[s] takes q[s + e_i]: the pencil holding that updates it
  const bool own[3] = {pen && by < MP && bz < MP, pen && by >= 1 && by <= MP && bz < MP,
                       pen && by < MP && bz >= 1 && bz <= MP};
  const int pl[3] = {MP * (by + MP * bz), NC + MP * ((by - 1) + MP * bz), 2 * NC + MP * (by + MP * (bz - 1))};
  KappaWords<M, S> kw;
  T cw[kCornerWords<M>], old[3][MP];
  kw.load(ku, n0, lane);
  corner_words<M, S>(p, 0, cnl, lane, cw);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (own[i]) {
#pragma unroll
      for (int sx = 0; sx < MP; ++sx) old[i][sx] = S::load(u, pl[i] + sx, n0);
    }
  }
  kw.put(lane, KA);
  interp_wave<M>(cw, lane, A, B);
  T* F = A;  // Laplacian of the current term (input of the product)
  T* Tc = B;  // current term g_k
  T gk[N2], q[N2];
#pragma unroll
  for (int b = 0; b < N2; ++b) gk[b] = T(0);
  if (pen) {
#pragma unroll
    for (int b = 0; b < N2; ++b) gk[b] = Tc[N2 * (by + N2 * bz) + b] * va.w0;
  }
#pragma unroll
  for (int b = 0; b < N2; ++b) q[b] = gk[b];
  __syncthreads();
  auto add = [&](const T* x) {  // q[0 .. m + 1] is what the outputs take
#pragma unroll
    for (int b = 0; b <= MP; ++b) q[b] += x[b];
  };
  wave_series<M, true>(KA, F, Tc, RED, w, va, gk, add);
  // u_i[s] -= wscale (s_i + 1) / h_i q[s + e_i]
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (own[i]) {
      const T f = wscale * va.ih[i];
#pragma unroll
      for (int sx = 0; sx < MP; ++sx) {
        const T a = -(T)(i == 0 ? sx + 1 : i == 1 ? by : bz) * f;
        S::store(u, pl[i] + sx, n0, fma(a, q[i == 0 ? sx + 1 : sx], old[i][sx]));
      }
    }
  }
}

template <int M, class S>
__global__ void __launch_bounds__(64, kVarWaves<S>) p_half_var_wave(typename S::View p, typename S::View u, typename S::View kp,
                                                      Grid g, VarArgs<typename S::C> va, int32_t per_xcd) {
  p_half_var_wave_body<M, S>(p, u, kp, g, va, per_xcd, blockIdx.x);
}

template <int M, class S>
__global__ void __launch_bounds__(64, kVarWaves<S>) u_half_var_wave(typename S::View u, typename S::View p, typename S::View ku,
                                                      Grid g, VarArgs<typename S::C> va, typename S::C wscale,
                                                      int32_t per_xcd) {
  u_half_var_wave_body<M, S>(u, p, ku, g, va, wscale, per_xcd, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Variable kappa: transposed half-steps and the gradient with respect to the
// kappa data.  The increment of a half-step at one node, paired with adjoint
// data y spread onto the cell polynomial, is
//   S = <y, sum_k t_k>,   t_0 = T[kappa f] (pressure) or f (velocity),
//   t_k = r_k T[kappa Lap t_{k-1}],   r_k = w_k / w_{k-1},
// with f = w_0 div c (pressure) or w_0 c (velocity).  With the adjoint series
//   lam_kmax = y,   lam_{k-1} = y + r_k Lap^T T^T[kappa] lam_k
// (T^T[kappa] g: b -> sum_a kappa_a g_{a+b}) one has S = <lam_0, t_0>, so
//   dS/df = T^T[kappa] lam_0 (pressure), lam_0 (velocity), and
//   dS/dkappa_a = sum_k sum_b lam_k[a + b] g_k[b],
//   g_k = r_k Lap t_{k-1} (k >= 1), g_0 = f (pressure side only).
// The transposed interpolation then spreads dS/dc onto the 2^d corner blocks
// (a gather over the neighbouring cells, second kernel).  t_{k-1} is
// recomputed from t_0 for each k: no per-node stack of kmax polynomials; where
// they fit in registers (below) the lam_k, which depend on y and kappa alone,
// are formed first and kept, and t_k is formed once.
// ---------------------------------------------------------------------------

// Cell-polynomial slots on which the adjoint data y of a node can be nonzero:
// b in {0..m}^D (pressure side: the node's data block) or b = s + e_i with s
// in {0..m}^D (velocity side: the derivatives of Q that the velocity takes).
// y is held compactly on these slots.
template <int D, int M, bool PSIDE>
struct YSupport {
  static constexpr int N2 = 2 * M + 2, NP = VK<D, M>::NP;
  static constexpr bool in(int b) {
    const int dg[3] = {b % N2, D > 1 ? (b / N2) % N2 : 0, D > 2 ? b / (N2 * N2) : 0};
    int over = 0, top = 0, sum = 0;
    for (int k = 0; k < D; ++k) {
      if (dg[k] > M + 1) return false;
      top += dg[k] == M + 1;
      over += dg[k] > M;
      sum += dg[k];
    }
    return PSIDE ? over == 0 : top <= 1 && sum > 0;
  }
  static constexpr int count() {
    int c = 0;
    for (int b = 0; b < NP; ++b) c += in(b);
    return c;
  }
  static constexpr int idx(int b) {  // compact slot of b, -1 off the support
    int c = 0;
    for (int x = 0; x < b; ++x) c += in(x);
    return in(b) ? c : -1;
  }
  static constexpr int NY = count();
};

// Per-work-item arrays in LDS, slot (a, b) of lane l at [(a NP + b) 64 + l]:
// the adjoint kernels run 64 work-items per workgroup, consecutive lanes in
// consecutive banks.
template <typename T>
struct LaneLds {
  T* base;
  int lane;
  __device__ __forceinline__ T& operator()(int a, int b, int np) const { return base[(a * np + b) * 64 + lane]; }
};

// The gradient accumulators live in LDS (slot GS); t_0 and, on the pressure
// side, f as well when a cell polynomial takes 512 bytes or more (FP64 at
// 2D m = 3), where registers would spill to scratch.
template <int D, int M, typename T>
constexpr bool kGradStage = sizeof(T) * VK<D, M>::NP >= 512;
// The lam_k kept in registers: polynomials of at most 288 bytes (up to FP64 2D
// m = 2 and FP32 3D m = 1); longer ones would spill, and recompute.  One
// transposed step, recomputed / kept: 2D m = 2 192 x 160 FP64 111 / 100 us, FP32
// 98 / 78 us; 512^2 FP64 564 / 531 us, FP32 302 / 266 us; 3D m = 1 40^3 FP32
// 343 / 288 us.
template <int D, int M, typename T>
constexpr bool kKeepLam = sizeof(T) * VK<D, M>::NP <= 288 && VK<D, M>::KMAX <= 4;
// Whether g_1 of the kept form waits in LDS (grad_forward).
template <int D, int M, typename T>
constexpr bool kKeepG1 = kKeepLam<D, M, T> && (VK<D, M>::KMAX > 1);
// Wavefronts per SIMD asked for: 2D FP32 fits its kept lam_k in half the
// registers to within two (left to itself the compiler takes those two and one
// wavefront runs per SIMD: 326 us at 512^2).
template <int D, int M, typename T>
constexpr int kGradWaves = D == 2 && sizeof(T) == 4 && kKeepLam<D, M, T> ? 2 : 1;

// grad_A += sum_b lam_{A+b} g_b (the kappa_A derivative of <lam, T[kappa g]>).
// lam and g on the coefficients of need <= J.  OWN: the sum over b is formed by
// itself and then added.
template <int D, int M, bool VEL, int J, bool OWN, int A, typename T>
__device__ __forceinline__ void corr_term(const T* lam, const T* g, const LaneLds<T>& L, int gs) {
  if constexpr (kNeed<D, M, VEL>.n[A] > J) return;
  constexpr int N2 = 2 * M + 2, AX = A % N2, AY = (A / N2) % N2, AZ = A / (N2 * N2);
  constexpr int NY = D > 1 ? N2 : 1, NZ = D > 2 ? N2 : 1, NP = VK<D, M>::NP;
  const T before = L(gs, A, NP);
  T acc = OWN ? T(0) : before;
#pragma unroll
  for (int bz = 0; bz + AZ < NZ; ++bz)
#pragma unroll
    for (int by = 0; by + AY < NY; ++by)
#pragma unroll
      for (int bx = 0; bx + AX < N2; ++bx) {
        const int hi = (bx + AX) + N2 * ((by + AY) + N2 * (bz + AZ));
        if (kNeed<D, M, VEL>.n[hi] <= J) acc = fma(lam[hi], g[bx + N2 * (by + N2 * bz)], acc);
      }
  L(gs, A, NP) = OWN ? before + acc : acc;
}

template <int D, int M, bool VEL, int J, bool OWN, typename T, int... A>
__device__ __forceinline__ void corr_terms(const T* lam, const T* g, const LaneLds<T>& L, int gs,
                                           std::integer_sequence<int, A...>) {
  (corr_term<D, M, VEL, J, OWN, A>(lam, g, L, gs), ...);
}

template <int D, int M, bool VEL, int J, bool OWN = false, typename T>
__device__ __forceinline__ void corr(const T* lam, const T* g, const LaneLds<T>& L, int gs) {
  corr_terms<D, M, VEL, J, OWN>(lam, g, L, gs, std::make_integer_sequence<int, VK<D, M>::NP>{});
}

// out = sc Lap^T f: sc sum_i (b_i - 1) b_i / h_i^2 f_{b - 2 e_i}; f zero off
// need <= J, out formed on need <= J + 1.
template <int D, int M, bool VEL, int J, typename T>
__device__ __forceinline__ void lapT_coef(const T* f, T* out, const T* ih, T sc) {
  constexpr int N2 = 2 * M + 2, NP = VK<D, M>::NP;
  const T ix2 = sc * ih[0] * ih[0], iy2 = sc * ih[1] * ih[1], iz2 = sc * ih[2] * ih[2];
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    const int bx = b % N2, by = (b / N2) % N2, bz = b / (N2 * N2);
    T v = T(0);
    if (kNeed<D, M, VEL>.n[b] > J + 1) continue;
    auto in = [](int x) { return kNeed<D, M, VEL>.n[x] <= J; };
    if (bx >= 2 && in(bx >= 2 ? b - 2 : 0)) v = fma(T((bx - 1) * bx) * ix2, f[b - 2], v);
    if (D > 1 && by >= 2 && in(by >= 2 ? b - 2 * N2 : 0)) v = fma(T((by - 1) * by) * iy2, f[b - 2 * N2], v);
    if (D > 2 && bz >= 2 && in(bz >= 2 ? b - 2 * N2 * N2 : 0)) v = fma(T((bz - 1) * bz) * iz2, f[b - 2 * N2 * N2], v);
    out[b] = v;
  }
}

// The series part shared by both sides: given t_0 (registers t0r, or LDS
// slot t0s when staged) and y (compact on its support), returns lam_0 in lam
// and adds sum_{k >= 1} sum_b lam_k[a + b] g_k[b] to the gradient (LDS slot gs).
//
// Kept form: lam_k lives on need <= J = kmax - k, so with g_k on the same set
// each product is formed on it; lam_kmax .. lam_0 in registers, then one pass
// over t_k.  Multiply-adds of 2D m = 2 against recomputing t_k with full
// products: 3933 of 7497 (pressure), 3522 of 6174.
template <int D, int M, bool PSIDE, int K, class S>
__device__ __forceinline__ void lam_back(const typename S::View& kv, uint32_t n0, const typename S::C* yc,
                                         const VarArgs<typename S::C>& va, typename S::C (*lam)[VK<D, M>::NP]) {
  if constexpr (K >= 1) {  // lam[K - 1] from lam[K]
    using T = typename S::C;
    using Y = YSupport<D, M, PSIDE>;
    constexpr int NP = VK<D, M>::NP, J = VK<D, M>::KMAX - K;
    T t[NP], l[NP];
    tprod_grouped<D, M, !PSIDE, J, true, S>(kv, n0, lam[K], t);
    lapT_coef<D, M, !PSIDE, J>(t, l, va.ih, va.ratio[K]);
#pragma unroll
    for (int b = 0; b < NP; ++b) {
      const int yi = Y::idx(b);
      lam[K - 1][b] = (yi >= 0 ? yc[yi < 0 ? 0 : yi] : T(0)) + (kNeed<D, M, !PSIDE>.n[b] <= J + 1 ? l[b] : T(0));
    }
    lam_back<D, M, PSIDE, K - 1, S>(kv, n0, yc, va, lam);
  }
}
template <int D, int M, bool PSIDE, int K, class S>
__device__ __forceinline__ void grad_forward(const typename S::View& kv, uint32_t n0, const LaneLds<typename S::C>& L,
                                             int gs, const VarArgs<typename S::C>& va,
                                             const typename S::C (*lam)[VK<D, M>::NP], typename S::C* t) {
  if constexpr (K <= VK<D, M>::KMAX) {
    using T = typename S::C;
    constexpr int NP = VK<D, M>::NP, J = VK<D, M>::KMAX - K;
    T l[NP];
    lap_coef<D, M, !PSIDE, J>(t, l, va.ih, va.ratio[K]);  // g_k
    // The terms fall with k, and adding a later k's products to the sum of an
    // earlier one would round at the size of that sum: k = 1 comes last, its
    // g_1 waiting in the LDS slot after gs (FP32 3D m = 1, gradient of the
    // velocity side off FP64: 1.6e-7 so, 2.4e-7 with k ascending).
    if constexpr (K == 1 && kKeepG1<D, M, T>) {
#pragma unroll
      for (int b = 0; b < NP; ++b)
        if (kNeed<D, M, !PSIDE>.n[b] <= J) L(gs + 1, b, NP) = l[b];
    } else {
      corr<D, M, !PSIDE, J, (K > 2)>(lam[K], l, L, gs);
    }
    if constexpr (K < VK<D, M>::KMAX) tprod_grouped<D, M, !PSIDE, J, false, S>(kv, n0, l, t);
    grad_forward<D, M, PSIDE, K + 1, S>(kv, n0, L, gs, va, lam, t);
    if constexpr (K == 1 && kKeepG1<D, M, T>) {
#pragma unroll
      for (int b = 0; b < NP; ++b)
        if (kNeed<D, M, !PSIDE>.n[b] <= J) l[b] = L(gs + 1, b, NP);
      corr<D, M, !PSIDE, J>(lam[1], l, L, gs);
    }
  }
}

template <int D, int M, bool PSIDE, class S>
__device__ __forceinline__ void adjoint_series(const typename S::View& kv, uint32_t n0,
                                               const LaneLds<typename S::C>& L, const typename S::C* t0r, int t0s,
                                               int gs, const typename S::C* yc, const VarArgs<typename S::C>& va,
                                               typename S::C* lam) {
  using T = typename S::C;
  using Y = YSupport<D, M, PSIDE>;
  constexpr int NP = VK<D, M>::NP, KMAX = VK<D, M>::KMAX;
  constexpr bool STAGE = kGradStage<D, M, T>;
  if constexpr (kKeepLam<D, M, T>) {
    T lk[KMAX + 1][NP], t[NP];
#pragma unroll
    for (int b = 0; b < NP; ++b) {
      const int yi = Y::idx(b);
      lk[KMAX][b] = yi >= 0 ? yc[yi < 0 ? 0 : yi] : T(0);
      t[b] = t0r[b];
    }
    lam_back<D, M, PSIDE, KMAX, S>(kv, n0, yc, va, lk);
    grad_forward<D, M, PSIDE, 1, S>(kv, n0, L, gs, va, lk, t);
#pragma unroll
    for (int b = 0; b < NP; ++b) lam[b] = lk[0][b];
    return;
  }
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    const int yi = Y::idx(b);
    lam[b] = yi >= 0 ? yc[yi < 0 ? 0 : yi] : T(0);
  }
#pragma unroll 1
  for (int k = KMAX; k >= 1; --k) {
    T t[NP], l[NP];
#pragma unroll
    for (int b = 0; b < NP; ++b) t[b] = STAGE ? L(t0s, b, NP) : t0r[b];
#pragma unroll 1
    for (int q = 1; q < k; ++q) {  // t = t_{k-1}
      lap_coef<D, M, !PSIDE, KMAX>(t, l, va.ih, va.ratio[q]);
      tprod_grouped<D, M, !PSIDE, KMAX, false, S>(kv, n0, l, t);
    }
    lap_coef<D, M, !PSIDE, KMAX>(t, l, va.ih, va.ratio[k]);  // g_k
    corr<D, M, !PSIDE, KMAX>(lam, l, L, gs);
    tprod_grouped<D, M, !PSIDE, KMAX, true, S>(kv, n0, lam, t);
    lapT_coef<D, M, !PSIDE, KMAX>(t, l, va.ih, va.ratio[k]);
#pragma unroll
    for (int b = 0; b < NP; ++b) {
      const int yi = Y::idx(b);
      lam[b] = (yi >= 0 ? yc[yi < 0 ? 0 : yi] : T(0)) + l[b];
    }
  }
}

// Pressure side at primal node j: with Pb the adjoint pressure and U_t the
// velocity before the step, gk -= dS/dkappa (FP64 accumulators, one plane per
// kappa coefficient) and rho_i = d S / d c^(i) (D NP planes of scratch).
// 64 work-items per workgroup (a 64 x 1 tile).
template <int D, int M, class S>
__global__ void __launch_bounds__(64, (kGradWaves<D, M, typename S::C>)) grad_p_var(typename S::View pb, typename S::View u, typename S::View kp,
                                                 double* __restrict__ gk, typename S::View rho, Grid g,
                                                 VarArgs<typename S::C> va) {
  static_assert(D <= 2 || M <= 1, "the adjoint of the variable-kappa half-steps: d <= 2, or d = 3 with m <= 1");
  using T = typename S::C;
  using Y = YSupport<D, M, true>;
  constexpr int N2 = 2 * M + 2, MP = M + 1, NP = VK<D, M>::NP, NC = Dims<D, M>::NC;
  constexpr bool STAGE = kGradStage<D, M, T>;
  constexpr int FS = 0, T0S = 1, GS = STAGE ? 2 : 0;  // LDS slots
  __shared__ T lds[(STAGE ? 3 : kKeepG1<D, M, T> ? 2 : 1) * NP * 64];
  const LaneLds<T> L{lds, (int)threadIdx.x};
  int32_t j[3];
  if (!node_of_block<D>(g, blockIdx.x, j)) return;
  uint32_t cn[1 << D];
  corner_nodes<D>(g, j, cn);  // dual q = j - 1 + e
  const uint32_t n0 = out_index<D>(g, j);
  T f[NP], t0[NP];  // f = w_0 div c, t_0 = T[kappa f]
#pragma unroll
  for (int b = 0; b < NP; ++b) f[b] = T(0);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    T c[NP];
    interp_full<D, M, S>(u, i, cn, c);
    const int st = i == 0 ? 1 : i == 1 ? N2 : N2 * N2;
    const T w = va.w0 * va.ih[i];
#pragma unroll
    for (int b = 0; b < NP; ++b) {
      const int bi = digit(b, N2, i);
      if (bi + 1 < N2) f[b] = fma(T(bi + 1) * w, c[b + st], f[b]);
    }
  }
  tprod_grouped<D, M, false, VK<D, M>::KMAX, false, S>(kp, n0, f, t0);
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    if (STAGE) {
      L(FS, b, NP) = f[b];
      L(T0S, b, NP) = t0[b];
    }
    L(GS, b, NP) = T(0);
  }
  T yc[Y::NY];
#pragma unroll
  for (int s = 0; s < NC; ++s) yc[Y::idx(poly_index<D, M>(s, 0, 0, 0))] = S::load(pb, s, n0);
  T lam[NP];
  adjoint_series<D, M, true, S>(kp, n0, L, t0, T0S, GS, yc, va, lam);
  if (STAGE) {
#pragma unroll
    for (int b = 0; b < NP; ++b) f[b] = L(FS, b, NP);
  }
  corr<D, M, false, VK<D, M>::KMAX>(lam, f, L, GS);  // k = 0: t_0 = T[kappa f]
#pragma unroll
  for (int b = 0; b < NP; ++b) gk[(size_t)b * g.onodes + n0] -= (double)L(GS, b, NP);
  T phi[NP];  // dS/df
  tprod_grouped<D, M, false, VK<D, M>::KMAX, true, S>(kp, n0, lam, phi);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const T w = va.w0 * va.ih[i];
    const int st = i == 0 ? 1 : i == 1 ? N2 : N2 * N2;
#pragma unroll
    for (int b = 0; b < NP; ++b) {
      const int bi = digit(b, N2, i);
      const T v = bi >= 1 ? T(bi) * w * phi[b - st] : T(0);
      S::store(rho, i * NP + b, n0, v);
    }
  }
}

// Velocity side at dual node q: with Ub the adjoint velocity and P' the
// pressure after the step's pressure half-step, gk -= dS/dkappa and
// z = dS/dc (NP planes of scratch).  64 work-items per workgroup.
template <int D, int M, class S>
__global__ void __launch_bounds__(64, (kGradWaves<D, M, typename S::C>)) grad_u_var(typename S::View ub, typename S::View p, typename S::View ku,
                                                 double* __restrict__ gk, typename S::View z, Grid g,
                                                 VarArgs<typename S::C> va) {
  static_assert(D <= 2 || M <= 1, "the adjoint of the variable-kappa half-steps: d <= 2, or d = 3 with m <= 1");
  using T = typename S::C;
  using Y = YSupport<D, M, false>;
  constexpr int N2 = 2 * M + 2, MP = M + 1, NP = VK<D, M>::NP, NC = Dims<D, M>::NC;
  constexpr bool STAGE = kGradStage<D, M, T>;
  constexpr int T0S = 0, GS = STAGE ? 1 : 0;  // LDS slots
  __shared__ T lds[(STAGE ? 2 : kKeepG1<D, M, T> ? 2 : 1) * NP * 64];
  const LaneLds<T> L{lds, (int)threadIdx.x};
  int32_t j[3];
  if (!node_of_block<D>(g, blockIdx.x, j)) return;
  uint32_t cn[1 << D];
  corner_nodes<D>(g, j, cn);  // primal j = q + e
  const uint32_t n0 = out_index<D>(g, j);
  T t0[NP];
  interp_full<D, M, S>(p, 0, cn, t0);
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    t0[b] *= va.w0;
    if (STAGE) L(T0S, b, NP) = t0[b];
    L(GS, b, NP) = T(0);
  }
  // S = sum_i sum_s Ub_i[s] (s_i + 1) / h_i Q[s + e_i]
  T yc[Y::NY];
#pragma unroll
  for (int a = 0; a < Y::NY; ++a) yc[a] = T(0);
#pragma unroll
  for (int i = 0; i < D; ++i)
#pragma unroll
    for (int s = 0; s < NC; ++s) {
      const int si = digit(s, MP, i);
      yc[Y::idx(poly_index<D, M>(s, i == 0, i == 1, i == 2))] += T(si + 1) * va.ih[i] * S::load(ub, i * NC + s, n0);
    }
  T lam[NP];
  adjoint_series<D, M, false, S>(ku, n0, L, t0, T0S, GS, yc, va, lam);
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    gk[(size_t)b * g.onodes + n0] -= (double)L(GS, b, NP);
    S::store(z, b, n0, va.w0 * lam[b]);
  }
}

// acc[a] += sum_b H_e(b, a) z[b]: the transposed interpolation onto corner e
// (bit k: upper side in dimension k) of a cell.  H_e(b, a) is the weight of
// corner datum a in coefficient b of the interpolant: pass_coef for the upper
// corner, with the sign of the delta combination for the lower one.
template <int M, int SIDE>
constexpr double hcol(int b, int a) {
  return pass_coef<M, 0>(b, a) * ((SIDE == 0 && ((b + a) & 1)) ? -1.0 : 1.0);
}

template <int D, int M, int E, typename T>
__device__ __forceinline__ void interp_T(const T* z, T* acc) {
  constexpr int N2 = 2 * M + 2, MP = M + 1;
  if constexpr (D == 1) {
#pragma unroll
    for (int a = 0; a < MP; ++a)
#pragma unroll
      for (int b = 0; b < N2; ++b) {
        const double h = hcol<M, E & 1>(b, a);
        if (h != 0.0) acc[a] = fma(T(h), z[b], acc[a]);
      }
  } else if constexpr (D == 3) {
    T zz[N2][N2][MP];  // [b_x][b_y][a_z]
#pragma unroll
    for (int bx = 0; bx < N2; ++bx)
#pragma unroll
      for (int by = 0; by < N2; ++by)
#pragma unroll
        for (int az = 0; az < MP; ++az) {
          T v = T(0);
#pragma unroll
          for (int bz = 0; bz < N2; ++bz) {
            const double h = hcol<M, (E >> 2) & 1>(bz, az);
            if (h != 0.0) v = fma(T(h), z[bx + N2 * (by + N2 * bz)], v);
          }
          zz[bx][by][az] = v;
        }
    T zy[N2][MP][MP];  // [b_x][a_y][a_z]
#pragma unroll
    for (int bx = 0; bx < N2; ++bx)
#pragma unroll
      for (int ay = 0; ay < MP; ++ay)
#pragma unroll
        for (int az = 0; az < MP; ++az) {
          T v = T(0);
#pragma unroll
          for (int by = 0; by < N2; ++by) {
            const double h = hcol<M, (E >> 1) & 1>(by, ay);
            if (h != 0.0) v = fma(T(h), zz[bx][by][az], v);
          }
          zy[bx][ay][az] = v;
        }
#pragma unroll
    for (int az = 0; az < MP; ++az)
#pragma unroll
      for (int ay = 0; ay < MP; ++ay)
#pragma unroll
        for (int ax = 0; ax < MP; ++ax)
#pragma unroll
          for (int bx = 0; bx < N2; ++bx) {
            const double h = hcol<M, E & 1>(bx, ax);
            if (h != 0.0) acc[ax + MP * (ay + MP * az)] = fma(T(h), zy[bx][ay][az], acc[ax + MP * (ay + MP * az)]);
          }
  } else {
    T zy[N2][MP];
#pragma unroll
    for (int bx = 0; bx < N2; ++bx)
#pragma unroll
      for (int ay = 0; ay < MP; ++ay) {
        T v = T(0);
#pragma unroll
        for (int by = 0; by < N2; ++by) {
          const double h = hcol<M, (E >> 1) & 1>(by, ay);
          if (h != 0.0) v = fma(T(h), z[bx + N2 * by], v);
        }
        zy[bx][ay] = v;
      }
#pragma unroll
    for (int ay = 0; ay < MP; ++ay)
#pragma unroll
      for (int ax = 0; ax < MP; ++ax)
#pragma unroll
        for (int bx = 0; bx < N2; ++bx) {
          const double h = hcol<M, E & 1>(bx, ax);
          if (h != 0.0) acc[ax + MP * ay] = fma(T(h), zy[bx][ay], acc[ax + MP * ay]);
        }
  }
}

template <int D, int M, class S, int EP>
__device__ __forceinline__ void gather_corner(const typename S::View& scr, int comp, uint32_t node,
                                              typename S::C* acc) {
  constexpr int NP = VK<D, M>::NP;
  typename S::C z[NP];
#pragma unroll
  for (int b = 0; b < NP; ++b) z[b] = S::load(scr, comp * NP + b, node);
  // slot EP of the output node's stencil is corner E = EP ^ (2^D - 1) of the
  // source node's cell
  interp_T<D, M, EP ^ ((1 << D) - 1)>(z, acc);
}

// In 3D a scheduling barrier after each corner keeps the compiler from
// issuing all 8 corners' (2m+2)^3 loads up front (2 KB of scratch per lane at
// m = 1 in FP64).
template <int D, int M, class S, int EP>
__device__ __forceinline__ void gather_corner_fenced(const typename S::View& scr, int comp, uint32_t node,
                                                     typename S::C* acc) {
  gather_corner<D, M, S, EP>(scr, comp, node, acc);
  if constexpr (D == 3) __builtin_amdgcn_sched_barrier(0);
}

template <int D, int M, class S, int... EP>
__device__ __forceinline__ void gather_corners(const typename S::View& scr, int comp, const uint32_t* cn,
                                               typename S::C* acc, std::integer_sequence<int, EP...>) {
  (gather_corner_fenced<D, M, S, EP>(scr, comp, cn[EP], acc), ...);
}

template <int D, int M, class S, int... EP>
__device__ __forceinline__ void gather_corners_masked(const typename S::View& scr, int comp, const uint32_t* cn,
                                                      const bool* valid, typename S::C* acc,
                                                      std::integer_sequence<int, EP...>) {
  ((valid[EP] ? gather_corner<D, M, S, EP>(scr, comp, cn[EP], acc) : void()), ...);
}

// Second stage of a transposed variable-kappa half-step: out -= the
// transposed interpolation of the per-cell dS/dc held in scr over the
// output node's stencil (the source node's cell has the output node as
// corner 1 - e where the output's stencil has the source as slot e).
//   PTYPE = true:  out = Pb (primal), scr = z over the dual nodes (NP planes)
//   PTYPE = false: out = Ub (dual, D components), scr = rho over the primal
//                  nodes (D NP planes)
template <int D, int M, class S, bool PTYPE>
__global__ void __launch_bounds__(256) var_adjoint_gather(typename S::View out, typename S::View scr, Grid g) {
  using T = typename S::C;
  constexpr int NC = Dims<D, M>::NC, NO = PTYPE ? 1 : D;
  int32_t j[3];
  if (!node_of_block<D>(g, blockIdx.x, j)) return;
  uint32_t cn[1 << D];
  corner_nodes<D>(g, j, cn);
  const uint32_t n0 = out_index<D>(g, j);
  // The output loop stays a loop even for one output (an opaque bound): in 3D,
  // straight-line code let the compiler issue every corner's loads at once.
  int zero = 0;
  if constexpr (D == 3) asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
#pragma unroll 1
  for (int io = 0; io < NO + zero; ++io) {
    T acc[NC];
#pragma unroll
    for (int a = 0; a < NC; ++a) acc[a] = T(0);
    gather_corners<D, M, S>(scr, io, cn, acc, std::make_integer_sequence<int, (1 << D)>{});
#pragma unroll
    for (int a = 0; a < NC; ++a) S::update(out, io * NC + a, n0, [&](T x) { return x - acc[a]; });
  }
}

// Walls, velocity side: scr[s] -= the transposed interpolation of rho over the
// primal corners of padded dual slot s (0..K+1 per dimension, dual node
// q = s - 1) that lie inside [0, K] (corners past a wall are not nodes of the
// walled step and contribute nothing).  The fold G^T (ghost_fold) then adds
// each ghost slot, with its mirror sign, into the node it mirrors.  The grid's
// K are the padded extents, sext the primal extents.
template <int D, int M, class S>
__global__ void __launch_bounds__(256) var_adjoint_gather_walls(typename S::View scr, typename S::View rho, Grid g) {
  using T = typename S::C;
  constexpr int NC = Dims<D, M>::NC;
  int32_t j[3];
  if (!node_of_block<D>(g, blockIdx.x, j)) return;
  uint32_t cn[1 << D];
  bool valid[1 << D];
#pragma unroll
  for (int e = 0; e < (1 << D); ++e) {
    int32_t c3[3] = {0, 0, 0};
    bool ok = true;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      c3[k] = j[k] - 1 + ((e >> k) & 1);
      ok = ok && c3[k] >= 0 && c3[k] < g.sext[k];
    }
    valid[e] = ok;
    cn[e] = ok ? node_index<D>(c3[0], c3[1], c3[2], g.sext) : 0u;
  }
  const uint32_t n0 = node_index<D>(j[0], j[1], j[2], g.oext);
#pragma unroll 1
  for (int io = 0; io < D; ++io) {
    T acc[NC];
#pragma unroll
    for (int a = 0; a < NC; ++a) acc[a] = T(0);
    gather_corners_masked<D, M, S>(rho, io, cn, valid, acc, std::make_integer_sequence<int, (1 << D)>{});
#pragma unroll
    for (int a = 0; a < NC; ++a) S::update(scr, io * NC + a, n0, [&](T x) { return x - acc[a]; });
  }
}

// ---------------------------------------------------------------------------
// Batched shots: one launch per half-step advances many independent problems
// ("shots": the paper's experiments repeated over sources and grids) of the
// same (d, m, storage), each with its own grid, time step, coefficient and
// buffers.  Shot s owns the workgroups [first_block, first_block + 8 per_xcd)
// of the launch; first_block is a multiple of 8, so every shot keeps its own
// XCD band mapping.  A workgroup finds its shot by binary search over the
// descriptor array (uniform, read through the scalar cache).
// ---------------------------------------------------------------------------
template <class S>
struct ShotHalf {
  typename S::View out, in, kap;   // kap: variable-kappa data (unused for constant kappa)
  const typename S::C* tab;        // merged tables (constant kappa)
  Grid g;
  VarArgs<typename S::C> va;       // variable kappa
  typename S::C wscale, ih[3];     // velocity half-step
  int32_t first_block;
  int32_t wave_per_xcd;            // variable kappa, 3D m >= 2: nodes per XCD run (one workgroup per node)
};

// A table pointer read from memory, recast to the constant address space so
// that uniform table reads become scalar loads (a pointer loaded from memory
// is generic, and generic loads are per-lane flat loads).

template <class S>
__device__ __forceinline__ int shot_of(const ShotHalf<S>* __restrict__ sh, int n, int blk) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (__builtin_amdgcn_readfirstlane(sh[mid].first_block) <= blk)
      lo = mid;
    else
      hi = mid - 1;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// The descriptor of this workgroup's shot, every word passed through
// readfirstlane: the values are uniform, and saying so keeps pointers, grid
// and table addresses in scalar registers (otherwise the merged tables are
// read with vector loads, as in a kernel whose table pointer may vary by lane).
template <class S>
__device__ __forceinline__ ShotHalf<S> shot_desc(const ShotHalf<S>* __restrict__ shots, int s) {
  static_assert(sizeof(ShotHalf<S>) % 4 == 0, "descriptor must be whole words");
  ShotHalf<S> d;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(shots + s);
  uint32_t w[sizeof(ShotHalf<S>) / 4];
#pragma unroll
  for (int i = 0; i < (int)(sizeof(ShotHalf<S>) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(src[i]);
  __builtin_memcpy(&d, w, sizeof d);
  return d;
}

// Form of a 3D batch's half-steps for the default tile.  Shots are small grids
// and fill the 64-wide tiles badly.  FP32, m <= 2, loads corners directly: they
// hit in the caches, and a tile's staging is not shared by enough nodes to pay
// for its barriers.  Otherwise the corners are staged, with the default tile's
// LDS (37 KB for the FP64 pressure side at m <= 2, against 61 KB of the any-tile
// form, which fits two workgroups per CU instead of four).  16 steps of 24
// shots, any-tile / default-tile staged / direct: m = 2 FP32 16^3 2822 / 1946 /
// 1496 us, 40x36x30 10196 / 8279 / 7281 us; m = 1 FP64 16^3 1390 / 875 / 1010 us,
// 40x36x30 5720 / 3081 / 3915 us.
template <int M, class S>
constexpr int kBatchForm = sizeof(typename S::C) == 4 && M <= 2 ? (int)kDirect : (int)kOneLayer;

// FORM: of the 3D half-steps with constant kappa.
template <int D, int M, class S, bool VAR, int FORM = kOneLayer>
__global__ void __launch_bounds__((!VAR && D == 3 ? 256 * PShape<M, S, FORM>::NS : 256), HL_WAVES_PER_EU)
    p_half_batch(const ShotHalf<S>* __restrict__ shots, int n) {
  const ShotHalf<S> sh = shot_desc(shots, shot_of(shots, n, blockIdx.x));
  const int blk = (int)blockIdx.x - sh.first_block;
  const ConstPtr<typename S::C> tab = const_ptr(sh.tab);
  using G = typename S::Global;
  const typename G::View out = S::global(sh.out), in = S::global(sh.in), kap = S::global(sh.kap);
  if constexpr (VAR)
    p_half_var_body<D, M, G>(out, in, kap, sh.g, sh.va, blk);
  else if constexpr (D == 3)
    p_half_3d_body<M, G, PShape<M, S, FORM>>(out, in, tab, sh.g, blk);
  else
    p_half_body<D, M, G, kEither>(out, in, tab, sh.g, blk);
}

template <int D, int M, class S, bool VAR, int FORM = kOneLayer>
__global__ void __launch_bounds__((!VAR && D == 3 ? 256 * UShape<M, S, FORM>::NS : 256), HL_WAVES_PER_EU)
    u_half_batch(const ShotHalf<S>* __restrict__ shots, int n) {
  const ShotHalf<S> sh = shot_desc(shots, shot_of(shots, n, blockIdx.x));
  const int blk = (int)blockIdx.x - sh.first_block;
  const ConstPtr<typename S::C> tab = const_ptr(sh.tab);
  using G = typename S::Global;
  const typename G::View out = S::global(sh.out), in = S::global(sh.in), kap = S::global(sh.kap);
  if constexpr (VAR)
    u_half_var_body<D, M, G>(out, in, kap, sh.g, sh.va, sh.wscale, blk);
  else if constexpr (D == 3)
    u_half_3d_body<M, G, UShape<M, S, FORM>>(out, in, tab, sh.g, sh.wscale, sh.ih[0], sh.ih[1], sh.ih[2], blk);
  else
    u_half_body<D, M, G, kEither>(out, in, tab, sh.g, sh.wscale, sh.ih[0], sh.ih[1], sh.ih[2], blk);
}

// Variable kappa, 3D m >= 2, batched: one 64-wide workgroup per node of each
// shot, as in the single-shot launch.
template <int M, class S>
__global__ void __launch_bounds__(64, kVarWaves<S>) p_half_batch_wave(const ShotHalf<S>* __restrict__ shots, int n) {
  const ShotHalf<S> sh = shot_desc(shots, shot_of(shots, n, blockIdx.x));
  using G = typename S::Global;
  p_half_var_wave_body<M, G>(S::global(sh.out), S::global(sh.in), S::global(sh.kap), sh.g, sh.va, sh.wave_per_xcd,
                             (int)blockIdx.x - sh.first_block);
}

template <int M, class S>
__global__ void __launch_bounds__(64, kVarWaves<S>) u_half_batch_wave(const ShotHalf<S>* __restrict__ shots, int n) {
  const ShotHalf<S> sh = shot_desc(shots, shot_of(shots, n, blockIdx.x));
  using G = typename S::Global;
  u_half_var_wave_body<M, G>(S::global(sh.out), S::global(sh.in), S::global(sh.kap), sh.g, sh.va, sh.wscale,
                             sh.wave_per_xcd, (int)blockIdx.x - sh.first_block);
}

// Sources inside a batch (the source term z = r(t) g(x) of Sec. 4, added by
// the midpoint rule after each pressure half-step): entry i adds
// amps[shot][n] * val[i] to word `word` of its shot's pressure array, n the
// batch's step counter (no source from step namps on).  The entries are the
// nodes of each shot's (compactly supported) g, so the launch is small.
struct BatchSource {
  int32_t shot;
  uint32_t word;  // plane * nodes + node in the shot's pressure array
};

template <typename W>
__global__ void __launch_bounds__(256) batch_source_add(W* const* __restrict__ pbase,
                                                        const BatchSource* __restrict__ ent,
                                                        const W* __restrict__ val, const W* __restrict__ amps,
                                                        int64_t namps, const int64_t* __restrict__ counter,
                                                        int64_t nent) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nent) return;
  const int64_t n = counter[0];
  if (n < 0 || n >= namps) return;
  const BatchSource e = ent[i];
  W* q = pbase[e.shot] + e.word;
  *q = fma(amps[(int64_t)e.shot * namps + n], val[i], *q);
}

// The same in FP32_COMP storage: pbase holds each shot's hi base and lo base
// (entries 2s and 2s + 1); values and amplitudes are FP64 (the values as the
// split storage holds them), and the update rounds to hi + lo as every write
// of that storage does.
template <class S>
__global__ void __launch_bounds__(256) batch_source_add_split(void* const* __restrict__ pbase,
                                                              const BatchSource* __restrict__ ent,
                                                              const double* __restrict__ val,
                                                              const double* __restrict__ amps, int64_t namps,
                                                              const int64_t* __restrict__ counter, int64_t nent) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nent) return;
  const int64_t n = counter[0];
  if (n < 0 || n >= namps) return;
  const BatchSource e = ent[i];
  const typename S::View v{static_cast<float*>(pbase[2 * e.shot]), static_cast<uint16_t*>(pbase[2 * e.shot + 1]), 0};
  const double a = amps[(int64_t)e.shot * namps + n], g = val[i];
  S::update(v, 0, e.word, [&](double x) { return fma(a, g, x); });
}

}  // namespace hl
