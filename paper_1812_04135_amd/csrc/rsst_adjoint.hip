// Discrete adjoint of one SSP-RK2 RSST step, FP64, for a fixed dt.
//
// With U1 = U + dt R(U) and U' = (U + U1 + dt R(U1)) / 2 (Sec. 4.1, the
// two-stage scheme), a cotangent lam' = dJ/dU' is pulled back by
//   (a, s1) = VJP(U1, lam'),      mu  = (lam' + dt a) / 2,
//   (b, s2) = VJP(U,  mu),        lam = lam'/2 + mu + dt b,
//   dJ/dxi += dt s1 / 2 + dt s2,
// where VJP(V, w) = (J_R(V)^T w, w . dR/dxi(V)) is the vector-Jacobian
// product of the semi-discrete operator R: MC-limited face states on the
// conservative variables, the LLF flux with c_tot = |V| + a/xi, the flux
// divergence, the RSST correction of the chosen form (eq. pvs_dt and
// App. A) and gravity (App. B).
//
// Derivatives are the branch-frozen ones of the primal values: the MC
// limiter is zero when l r <= 0, else it follows the first minimum among
// (|l+r|/2, 2|l|, 2|r|); the LLF speed is c_L when c_L >= c_R, else c_R;
// d|V| = 0 at |V| = 0.  A reflecting wall is the mirror image S of the
// cell state (normal momentum negated), so the wall face's outer state is
// S of the inner face state and its cotangent returns through S.
//
// On a 1D or 3D grid the VJP runs as the three passes below (a 2D grid
// takes the tiled form of the same passes, rsst_adjoint_tile.hip), each
// writing only its own cells, so the result is deterministic (no atomics):
//   A2 cell   fluxes G = 2 Fhat at the cell's two faces of every axis (a
//             face shared by two cells is formed by both, the same bits),
//             increments Delta, reverse of correction + gravity:
//             Delta_bar, the direct part of U_bar, the f part of xi_bar;
//   A3 face   G_bar from Delta_bar, reverse of the LLF flux into the plus
//             state of the left cell (Pb) and the minus state of the right
//             cell (Mb), the alpha part of xi_bar;
//   A4+A5 cell  U_bar += Pb + Mb, reverse of the MC half slope h = (Pb-Mb):
//             slope cotangents (lb, rb) of the cell, and the -lb of the cell
//             above and +rb of the cell below (formed here as those cells
//             form them); then mu (first VJP) or the new lam (second VJP).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "rsst_adjoint.h"
#include "rsst_adjoint_ops.h"

#pragma clang fp contract(off)

namespace rsstk {

// What bounds the passes: on small 3D grids the latency of the chains of loads
// and reciprocals, on large ones instruction issue and, in the gather, the 55
// values per cell and axis that it reads.  64-bit index arithmetic and boundary
// branches were half of the instructions; now one axis' neighbourhood is five
// selected 32-bit offsets, read once.  us per adjoint step (before, now):
// 45 x 38 x 52 106, 78; 64^3 187, 163; 128^3 1630, 1376; 1D 256 29.6, 23.4.
//
// Values are addressed by 32-bit byte offsets from the (uniform) start of a
// variable's array, one VGPR per neighbour and no 64-bit vector arithmetic; arrays of 4
// GiB or more (Off = unsigned long long) take 64-bit offsets.
template <typename Off>
__device__ __forceinline__ double ld(const double* p, Off o) {
  return *(const double*)((const char*)p + o);
}

template <typename Off>
__device__ __forceinline__ void st(double* p, Off o, double x) {
  *(double*)((char*)p + o) = x;
}

template <int NV, typename Off>
__device__ __forceinline__ void load(const double* U, long long ncell, Off o, double (&u)[NV]) {
#pragma unroll
  for (int v = 0; v < NV; ++v) u[v] = ld<Off>(U + v * ncell, o);
}

// A cell's neighbourhood along axis D: byte offsets of the cells at -2 .. 2
// through the boundary rule, the sign flips of the normal momentum there
// (the mirror image across a wall), and where the cell lies.
template <typename Off>
struct Line {
  Off o[5];
  int flip[5];
  bool lo, hi;        // first, last cell of the axis
  bool wlo, whi;      // and there is a wall
};

template <int D, typename Off>
__device__ __forceinline__ Line<Off> line_of(const AdjArgs& A, unsigned c, const int x[3]) {
  Line<Off> L;
  const int n = A.n[D], stride = (int)A.stride[D];
  L.lo = x[D] == 0;
  L.hi = x[D] == n - 1;
  L.wlo = L.lo && A.refl_lo[D];
  L.whi = L.hi && A.refl_hi[D];
#pragma unroll
  for (int k = -2; k <= 2; ++k) {
    const int q = x[D] + k;
    const bool below = q < 0, above = q >= n;
    const int qb = A.refl_lo[D] ? -1 - q : q + n, qa = A.refl_hi[D] ? 2 * n - 1 - q : q - n;
    const int m = below ? qb : (above ? qa : q);
    L.o[k + 2] = (Off)(unsigned)((int)c + (m - x[D]) * stride) * 8;
    L.flip[k + 2] = ((below && A.refl_lo[D]) || (above && A.refl_hi[D])) ? (int)0x80000000 : 0;
  }
  return L;
}

template <int NDIM, int D, typename Off>
__device__ __forceinline__ void load_at(const AdjArgs& A, const double* U, const Line<Off>& L, int k,
                                        double (&u)[NDIM + 2]) {
  load<NDIM + 2, Off>(U, A.ncell, L.o[k + 2], u);
  u[1 + D] = __hiloint2double(__double2hiint(u[1 + D]) ^ L.flip[k + 2], __double2loint(u[1 + D]));
}

// Cells per workgroup and axes of a cell per thread.  Small 3D grids give
// every axis of a cell to a wave of its own: their passes are bound by the
// latency of the chain of loads and reciprocals, and one axis is a third of
// the chain and three times the waves.  Large ones, bound by instruction
// issue, take all axes of a cell in one thread (us per adjoint step, split and
// not: 45 x 38 x 52 78 and 83, 56^3 133 and 125, 64^3 178 and 163).
constexpr int kCellsSplit = 128;
constexpr long long kSplitMax = 131072;  // largest ncell that is split
template <int NDIM, bool SPLIT>
struct PassShape {
  static constexpr int kCells = SPLIT ? kCellsSplit : kAdjThreads;
  static constexpr int kThreads = SPLIT ? NDIM * kCellsSplit : kAdjThreads;
};
static bool split_axes(int ndim, long long ncell) { return ndim == 3 && ncell <= kSplitMax; }
static int pass_blocks(int ndim, long long ncell) {
  const int n = split_axes(ndim, ncell) ? kCellsSplit : kAdjThreads;
  return (int)((ncell + n - 1) / n);
}

// This thread's cell (workgroups of neighbouring cells on the same XCD) and its
// coordinates, and its axis (the same for its
// whole wave; -1: all of them).
template <int NDIM, bool SPLIT>
__device__ __forceinline__ bool my_cell(const AdjArgs& A, unsigned& c, int x[3], int& axis) {
  using S = PassShape<NDIM, SPLIT>;
  axis = SPLIT ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / S::kCells) : -1;
  c = (unsigned)xcd_tile(blockIdx.x, A.nblock) * (unsigned)S::kCells + (threadIdx.x - (SPLIT ? (unsigned)axis * S::kCells : 0u));
  const unsigned r = c / (unsigned)A.n[0];
  x[0] = (int)(c - r * (unsigned)A.n[0]);
  x[2] = (int)(r / (unsigned)A.n[1]);
  x[1] = (int)(r - (unsigned)x[2] * (unsigned)A.n[1]);
  return c < (unsigned)A.ncell;
}

// f(D) for the thread's axis, or for every axis in turn.
template <int NDIM, bool SPLIT, typename Fn>
__device__ __forceinline__ void each_axis(int axis, Fn f) {
  if (!SPLIT || axis == 0) f(std::integral_constant<int, 0>());
  if constexpr (NDIM >= 3) {
    if (!SPLIT || axis == 1) f(std::integral_constant<int, 1>());
    if (!SPLIT || axis == 2) f(std::integral_constant<int, 2>());
  }
}

template <int NT>
__device__ __forceinline__ void block_partial(double v, double* out) {
  __shared__ double red[NT / 64];
  const double w = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int q = 0; q < NT / 64; ++q) s += red[q];
    out[blockIdx.x] = s;
  }
}

// Split axes: adds the parts of a cell that axes 1 and 2 formed to the one of
// axis 0 (through LDS); every thread of the workgroup calls it.  Returns
// whether this thread goes on with the cell.
template <int NDIM, bool SPLIT>
__device__ __forceinline__ bool join_axes(int axis, double (&part)[NDIM + 2]) {
  if constexpr (SPLIT) {
    constexpr int NV = NDIM + 2, N = kCellsSplit;
    __shared__ double buf[NDIM - 1][NV][N];
    const int q = (int)threadIdx.x - axis * N;
    if (axis > 0) {
#pragma unroll
      for (int v = 0; v < NV; ++v) buf[axis - 1][v][q] = part[v];
    }
    __syncthreads();
    if (axis == 0) {
#pragma unroll
      for (int d = 1; d < NDIM; ++d)
#pragma unroll
        for (int v = 0; v < NV; ++v) part[v] += buf[d - 1][v][q];
    }
    return axis == 0;
  }
  return true;
}

// ---------------------------------------------------------------- passes

// A2, one axis: inc += (G_hi - G_lo) / (2 dx), the fluxes of the cell's two
// faces formed here.  The ghost across a wall is the mirror cell, and its face
// state the mirror of the cell's own.
template <int NDIM, int D, typename Off>
__device__ __forceinline__ void a2_axis(const AdjArgs& A, const Consts& K, unsigned c, const int x[3],
                                        double (&inc)[NDIM + 2]) {
  constexpr int NV = NDIM + 2;
  const Line<Off> N = line_of<D, Off>(A, c, x);
  double u[5][NV];
#pragma unroll
  for (int k = -2; k <= 2; ++k) load_at<NDIM, D, Off>(A, A.V, N, k, u[k + 2]);
  double h[3][NV], Gl[NV], Gh[NV];
#pragma unroll
  for (int k = 0; k < 3; ++k) half_slope<NDIM>(u[k], u[k + 1], u[k + 2], h[k]);
  Face<NV> L, R;
  make_face<NDIM, D>(u[1], h[0], true, K, L);
  make_face<NDIM, D>(u[2], h[1], false, K, R);
  flux2<NDIM, D>(L, R, Gl);
  make_face<NDIM, D>(u[2], h[1], true, K, L);
  make_face<NDIM, D>(u[3], h[2], false, K, R);
  flux2<NDIM, D>(L, R, Gh);
  const double hd = 0.5 * A.inv_dx[D];
#pragma unroll
  for (int v = 0; v < NV; ++v) inc[v] += (Gh[v] - Gl[v]) * hd;
}

template <int NDIM, int FORM, bool SPLIT, typename Off>
__global__ void __launch_bounds__((PassShape<NDIM, SPLIT>::kThreads)) adj_cell_kernel(AdjArgs A) {
  constexpr int NV = NDIM + 2;
  unsigned c;
  int x[3], axis;
  const bool in = my_cell<NDIM, SPLIT>(A, c, x, axis);
  double Dl[NV] = {};
  if (in) {
    const Consts K = adj_consts<NDIM>(A);
    each_axis<NDIM, SPLIT>(axis, [&](auto d) { a2_axis<NDIM, d(), Off>(A, K, c, x, Dl); });
  }
  const bool mine = join_axes<NDIM, SPLIT>(axis, Dl);
  double xib = 0.0;
  if (in && mine) {
    double u[NV], Rb[NV], Db[NV], ub[NV];
    const Off o = (Off)c * 8;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      ub[v] = 0.0;
      Dl[v] = -Dl[v];
    }
    load<NV, Off>(A.V, A.ncell, o, u);
    load<NV, Off>(A.W, A.ncell, o, Rb);
    const double fb = rate_vjp<NDIM, FORM>(u, Dl, Rb, A, Db, ub);
    xib = fb * A.dfdxi;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      st<Off>(A.Db + v * A.ncell, o, Db[v]);
      st<Off>(A.out + v * A.ncell, o, ub[v]);
    }
  }
  block_partial<PassShape<NDIM, SPLIT>::kThreads>(xib, A.xpart);
}

// A3, one axis: the face above the cell, and the one below it at a low wall.
template <int NDIM, int D, typename Off>
__device__ __forceinline__ void a3_axis(const AdjArgs& A, const Consts& K, unsigned c, const int x[3],
                                        double& xib) {
  constexpr int NV = NDIM + 2;
  const double hd = 0.5 * A.inv_dx[D];
  double* Pb = A.Pb + (long long)D * NV * A.ncell;
  double* Mb = A.Mb + (long long)D * NV * A.ncell;
  const Line<Off> N = line_of<D, Off>(A, c, x);
  const Off o = N.o[2];
  double d0[NV], d1[NV], u[4][NV], h0[NV], h1[NV];
#pragma unroll
  for (int k = -1; k <= 2; ++k) load_at<NDIM, D, Off>(A, A.V, N, k, u[k + 1]);
  load<NV, Off>(A.Db, A.ncell, o, d0);
  load<NV, Off>(A.Db, A.ncell, N.o[3], d1);
  half_slope<NDIM>(u[0], u[1], u[2], h0);
  half_slope<NDIM>(u[1], u[2], u[3], h1);
  {
    // face i+1/2: dDelta_i/dG = -hd, dDelta_{i+1}/dG = +hd (none across a
    // wall, whose outer state is the mirror of the inner one)
    Face<NV> L, R;
    make_face<NDIM, D>(u[1], h0, true, K, L);
    make_face<NDIM, D>(u[2], h1, false, K, R);
    double Gb[NV], Lb[NV], Rbar[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Gb[v] = N.whi ? -hd * d0[v] : hd * (d1[v] - d0[v]);
    llf_vjp<NDIM, D>(L, R, Gb, A, Lb, Rbar, xib);
    if (N.whi) {
      mirror_add<NDIM, D>(Lb, Rbar);
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) st<Off>(Mb + v * A.ncell, N.o[3], Rbar[v]);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) st<Off>(Pb + v * A.ncell, o, Lb[v]);
  }
  if (N.wlo) {
    // wall face i-1/2: outer state S M_0, inner M_0; dDelta_0/dG = +hd
    Face<NV> R;
    make_face<NDIM, D>(u[1], h0, false, K, R);
    const Face<NV> L = mirror<NDIM, D>(R);
    double Gb[NV], Lb[NV], Rbar[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Gb[v] = hd * d0[v];
    llf_vjp<NDIM, D>(L, R, Gb, A, Lb, Rbar, xib);
    mirror_add<NDIM, D>(Rbar, Lb);
#pragma unroll
    for (int v = 0; v < NV; ++v) st<Off>(Mb + v * A.ncell, o, Rbar[v]);
  }
}

template <int NDIM, bool SPLIT, typename Off>
__global__ void __launch_bounds__((PassShape<NDIM, SPLIT>::kThreads)) adj_face_rev_kernel(AdjArgs A) {
  unsigned c;
  int x[3], axis;
  double xib = 0.0;
  if (my_cell<NDIM, SPLIT>(A, c, x, axis)) {
    const Consts K = adj_consts<NDIM>(A);
    each_axis<NDIM, SPLIT>(axis, [&](auto d) { a3_axis<NDIM, d(), Off>(A, K, c, x, xib); });
  }
  block_partial<PassShape<NDIM, SPLIT>::kThreads>(xib, A.xpart + A.nblock);
}

// A4 and A5, one axis: U_bar += Pb + Mb + lb - rb of the cell (a wall's ghost
// neighbour is S of this cell: its share comes back here), -lb of the cell
// above (its l is U_above - U_this) and +rb of the cell below (its r is
// U_this - U_below), with lb = (dh/dl) hb, rb = (dh/dr) hb and hb = Pb - Mb,
// the cotangent of a cell's half slope h.
template <int NDIM, int D, typename Off>
__device__ __forceinline__ void gather_axis(const AdjArgs& A, unsigned c, const int x[3], double (&ub)[NDIM + 2]) {
  constexpr int NV = NDIM + 2;
  const double* Pb = A.Pb + (long long)D * NV * A.ncell;
  const double* Mb = A.Mb + (long long)D * NV * A.ncell;
  const Line<Off> N = line_of<D, Off>(A, c, x);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    double u[5], pb[3], mb[3];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      u[k] = ld<Off>(A.V + v * A.ncell, N.o[k]);
      if (v == 1 + D) u[k] = __hiloint2double(__double2hiint(u[k]) ^ N.flip[k], __double2loint(u[k]));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      pb[k] = ld<Off>(Pb + v * A.ncell, N.o[k + 1]);
      mb[k] = ld<Off>(Mb + v * A.ncell, N.o[k + 1]);
    }
    double lb[3], rb[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double dl, dr;
      mc_half_partials(u[k + 1] - u[k], u[k + 2] - u[k + 1], dl, dr);
      const double hb = pb[k] - mb[k];
      lb[k] = dl * hb;
      rb[k] = dr * hb;
    }
    double s = pb[1] + mb[1] + lb[1] - rb[1];
    const double sl = v == 1 + D ? -lb[1] : lb[1], sr = v == 1 + D ? -rb[1] : rb[1];
    s -= N.wlo ? sl : 0.0;
    s += N.whi ? sr : 0.0;
    s -= N.whi ? 0.0 : lb[2];
    s += N.wlo ? 0.0 : rb[0];
    ub[v] += s;
  }
}

// The last pass of a VJP: A4 and A5, then mu or the new lam.  In the second
// VJP its workgroup 0 also folds the xi partials of both VJPs (complete:
// their passes ended before this one began) into dJdxi, after its own cells.
template <int NDIM, bool SPLIT, typename Off>
__global__ void __launch_bounds__((PassShape<NDIM, SPLIT>::kThreads)) adj_gather_kernel(AdjArgs A) {
  constexpr int NV = NDIM + 2;
  unsigned c;
  int x[3], axis;
  const bool in = my_cell<NDIM, SPLIT>(A, c, x, axis);
  double ub[NV] = {};
  if (in) {
    if (!SPLIT || axis == 0) load<NV, Off>(A.out, A.ncell, (Off)c * 8, ub);
    each_axis<NDIM, SPLIT>(axis, [&](auto d) { gather_axis<NDIM, d(), Off>(A, c, x, ub); });
  }
  const bool mine = join_axes<NDIM, SPLIT>(axis, ub);
  if (in && mine) {
    const Off o = (Off)c * 8;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const long long q = v * A.ncell;
      if (A.post == 1) st<Off>(A.mu + q, o, 0.5 * (ld<Off>(A.lam + q, o) + A.dt * ub[v]));
      else if (A.post == 2) st<Off>(A.lam + q, o, 0.5 * ld<Off>(A.lam + q, o) + ld<Off>(A.mu + q, o) + A.dt * ub[v]);
      else st<Off>(A.out + q, o, ub[v]);
    }
  }
  if (A.post == 2 && blockIdx.x == 0)
    xi_reduce<PassShape<NDIM, SPLIT>::kThreads>(A.xp1, A.xp2, A.xm, A.dt, A.dJdxi);
}

template <int NDIM, bool SPLIT, typename Off>
static hipError_t vjp_launch_k(const AdjArgs& A, int form, hipStream_t s) {
  const dim3 grid(A.nblock), block(PassShape<NDIM, SPLIT>::kThreads);
  switch (form) {
    case kEuler: hipLaunchKernelGGL((adj_cell_kernel<NDIM, kEuler, SPLIT, Off>), grid, block, 0, s, A); break;
    case kPVS: hipLaunchKernelGGL((adj_cell_kernel<NDIM, kPVS, SPLIT, Off>), grid, block, 0, s, A); break;
    case kPMS: hipLaunchKernelGGL((adj_cell_kernel<NDIM, kPMS, SPLIT, Off>), grid, block, 0, s, A); break;
    case kDVS: hipLaunchKernelGGL((adj_cell_kernel<NDIM, kDVS, SPLIT, Off>), grid, block, 0, s, A); break;
    case kDMS: hipLaunchKernelGGL((adj_cell_kernel<NDIM, kDMS, SPLIT, Off>), grid, block, 0, s, A); break;
    default: hipLaunchKernelGGL((adj_cell_kernel<NDIM, kPD, SPLIT, Off>), grid, block, 0, s, A); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((adj_face_rev_kernel<NDIM, SPLIT, Off>), grid, block, 0, s, A);
  // the gather has no partial sums of its own, so its workgroups may differ:
  // split on every 3D grid (all axes in one thread take 336 VGPRs)
  constexpr bool GSPLIT = NDIM == 3;
  using S = PassShape<NDIM, GSPLIT>;
  AdjArgs G = A;
  G.nblock = (int)((A.ncell + S::kCells - 1) / S::kCells);
  hipLaunchKernelGGL((adj_gather_kernel<NDIM, GSPLIT, Off>), dim3(G.nblock), dim3(S::kThreads), 0, s, G);
  return hipGetLastError();
}

static hipError_t vjp_launch(const AdjArgs& A, int form, hipStream_t s) {
  if (A.ndim == 1) return vjp_launch_k<1, false, unsigned>(A, form, s);
  if (split_axes(A.ndim, A.ncell)) return vjp_launch_k<3, true, unsigned>(A, form, s);
  return A.ncell < (1ll << 29) ? vjp_launch_k<3, false, unsigned>(A, form, s)
                               : vjp_launch_k<3, false, unsigned long long>(A, form, s);
}

size_t adjoint_workspace_doubles(int ndim, const int n[3], long long ncell) {
  const int nv = ndim + 2;
  if (ndim == 2) {
    // mu; two partial arrays and the run accumulator, one value per tile
    return (size_t)nv * ncell + 3 * (size_t)tile2_nblock(n);
  }
  const long long nblock = pass_blocks(ndim, ncell);
  // Pb, Mb: ndim fields each; Db, a/b, mu: one each; 4 partial arrays
  return (size_t)nv * ncell * (2 * ndim + 3) + 4 * (size_t)nblock;
}

size_t adjoint_zeroed_offset(int ndim, const int n[3], long long ncell) {
  return ndim == 2 ? (size_t)(ndim + 2) * ncell + 2 * (size_t)tile2_nblock(n) : adjoint_workspace_doubles(ndim, n, ncell);
}

hipError_t launch_adjoint_xi_fold(const AdjointPlan& p, double* dJdxi, hipStream_t s) {
  if (p.ndim != 2) return hipSuccess;
  const int nt = tile2_nblock(p.n);
  return launch_xi_acc_fold(p.work + adjoint_zeroed_offset(2, p.n, p.ncell), nt, dJdxi, s);
}

hipError_t launch_adjoint_step(const AdjointPlan& p, const double* U, const double* U1, double* lam, double dt,
                               double* dJdxi, bool defer, hipStream_t s) {
  const int ndim = p.ndim, nv = ndim + 2;
  const long long n = p.ncell, nf = (long long)nv * n;
  const int nblock = ndim == 2 ? 0 : pass_blocks(ndim, n);
  double* w = p.work;
  AdjArgs A{};
  A.ndim = ndim;
  A.nv = nv;
  for (int d = 0; d < 3; ++d) {
    A.n[d] = p.n[d];
    A.refl_lo[d] = p.refl_lo[d];
    A.refl_hi[d] = p.refl_hi[d];
    A.inv_dx[d] = p.inv_dx[d];
    A.g[d] = p.g[d];
  }
  A.stride[0] = 1;
  A.stride[1] = p.n[0];
  A.stride[2] = (long long)p.n[0] * p.n[1];
  A.ncell = n;
  A.gamma = p.gamma;
  A.gm1 = p.gamma - 1.0;
  A.inv_gm1 = 1.0 / (p.gamma - 1.0);
  A.inv_xi = 1.0 / p.xi;
  A.f = 1.0 - 1.0 / (p.xi * p.xi);
  A.dfdxi = 2.0 / (p.xi * p.xi * p.xi);
  A.lam = lam;
  A.dt = dt;
  A.dJdxi = dJdxi;
  if (ndim == 2) {
    // one tiled launch per VJP; each leaves one partial sum of xi_bar per
    // tile, and a one-workgroup launch after the second folds both sets
    const int nt = tile2_nblock(p.n);
    double* const part1 = w + nf;
    double* const part2 = part1 + nt;
    A.mu = w;
    A.nblock = nt;
    A.xp1 = part1;
    A.xp2 = part2;
    A.xacc = defer ? part2 + nt : nullptr;
    A.V = U1;
    A.W = lam;
    A.xpart = part1;
    A.post = 1;
    hipError_t e = launch_vjp_tile2(A, p.form, s);
    if (e != hipSuccess) return e;
    A.V = U;
    A.W = A.mu;
    A.xpart = part2;
    A.post = 2;
    e = launch_vjp_tile2(A, p.form, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
  }
  A.Pb = w;
  A.Mb = A.Pb + ndim * nf;
  A.Db = A.Mb + ndim * nf;
  double* ab = A.Db + nf;
  double* mu = ab + nf;
  double* part1 = mu + nf;
  double* part2 = part1 + 2 * nblock;
  A.nblock = nblock;
  A.mu = mu;
  // each VJP leaves partials of the f part then the alpha part (2 nblock
  // each); the second VJP's last pass folds both sets into dJdxi
  A.xp1 = part1;
  A.xp2 = part2;
  A.xm = 2 * nblock;
  auto vjp = [&](const double* V, const double* Wc, double* out, double* part, int post) {
    A.V = V;
    A.W = Wc;
    A.out = out;
    A.xpart = part;
    A.post = post;
    return vjp_launch(A, p.form, s);
  };
  // (a, s1) = VJP(U1, lam) with mu = (lam + dt a)/2 formed by its last pass
  hipError_t e = vjp(U1, lam, ab, part1, 1);
  if (e != hipSuccess) return e;
  // (b, s2) = VJP(U, mu) with lam = lam/2 + mu + dt b formed by its last pass
  e = vjp(U, mu, ab, part2, 2);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace rsstk
