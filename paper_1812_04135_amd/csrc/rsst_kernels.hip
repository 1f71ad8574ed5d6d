// Fused RSST stage kernels for gfx950 (the kernels themselves are
// instantiated per dimension and storage type in rsst_stage_inst.hip).
//
// One launch computes one SSP-RK2 stage (Sec. 4.1, items 2-8) for the whole
// grid in a single pass over HBM:
//   stage 1: U1 = Un + dt R(Un)
//   stage 2: Un <- (Un + (U1 + dt R(U1))) / 2, plus the CFL reduction of the
//            new state that gives the next dt (item 1).
// R(U) = MC-limited MUSCL reconstruction of the conservative variables, LLF
// flux with c_tot = |V| + a/xi, flux divergence, Delta P, the per-form
// correction (eq. pvs_dt, App. A) and gravity (App. B).
//
// Work decomposition (x = axis 0, contiguous in memory):
//   * lanes run along x.  1D and 3D: a workgroup holds whole rows of nx cells
//     spread over nwx = ceil(nx/64) waves, so x needs no halo.  2D: each wave
//     takes a strip of a row by itself, with halo lanes (rsst_stage2.h), and
//     a run of steps on a grid of few tiles takes both stages in one launch;
//     some single-stage launches hold whole rows (rsst_row2.h);
//   * whole rows in 2D and 3D: x neighbours and x plus-face states go through
//     LDS rows with a ghost slot at each end (periodic wrap or mirror); every
//     x flux is formed once, by the cell right of the face, and reaches the
//     cell on its left by DPP within a wave and through one LDS seam value per
//     wave edge after another barrier (rsst_row2.h, rsst_stage3.h).  1D keeps
//     its row in one workgroup with DPP neighbours and LDS seams, the
//     wave-edge fluxes formed by both waves (rsst_stage1.h);
//   * 3D: each thread owns two adjacent y rows of its column, and a tile of
//     eight waves stacks 2R rows; the y face between a thread's rows is
//     formed in registers, the one between thread-rows once and handed over
//     in LDS, and the tile's two outer faces by each of the two tiles that
//     share them (the same face states and code, so the same bits), from the
//     rows just outside the tile, which the edge thread-rows read from
//     global memory a plane ahead;
//   * the last axis (z in 3D, y in 2D) is marched: each thread keeps its
//     column's planes in registers, so every z face is computed once and
//     carried to the next plane;
//   * every face state (U +- sigma/2, its pressure, c_tot and normal
//     velocity) is computed once, by the cell that owns it;
//   * workgroup ids are remapped so that consecutive tiles (which share
//     halo rows) run on the same XCD and share its L2.
#include <algorithm>
#include <cstdlib>

#include "rsst_row2.h"
#include "rsst_stage1.h"
#include "rsst_stage2.h"
#include "rsst_stage3.h"

#pragma clang fp contract(off)

namespace rsstk {

// ---------------------------------------------------------------- prime

// The largest c_tot of a state per stage-kernel workgroup slot (the grid has
// one workgroup per slot, each taking a strided share of the cells), from
// which the next stage 1 forms the CFL dt; with set_t, also t = t0.
template <int NDIM, typename ST>
__global__ void __launch_bounds__(256) prime_kernel(const StageArgs A, const ST* __restrict__ u,
                                                    double t0, int set_t) {
  constexpr int NV = NDIM + 2;
  const Consts K{A.gamma, A.gm1, A.inv_gm1, A.inv_xi, A.f, A.inv_cmax2, A.vdw_a, A.vdw_b};
  const Geometry& G = A.geo;
  __shared__ double red[4];
  double cm = 0.0;
  unsigned bad = 0;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < A.ncell;
       c += (long long)gridDim.x * blockDim.x) {
    double q[NV];
    const int i = (int)(c % G.nx);
    const long long r = c / G.nx;
    const int j = (int)(r % G.ns);
    const int k = (int)(r / G.ns);
#pragma unroll
    for (int v = 0; v < NV; ++v) q[v] = (double)u[v * A.ncell + c];
    if constexpr (sizeof(ST) == 4) {
      int b = 0;
      if (A.bg_axis == 0) b = i;
      else if (A.bg_axis == 1) b = (NDIM == 3) ? j : k;
      else if (A.bg_axis == 2) b = k;
#pragma unroll
      for (int v = 0; v < NV; ++v) q[v] += A.bg[v * A.nbg + b];
    }
    const double ct = A.eos ? cell_ctot<NDIM, kExtVdw>(q, K)
                      : (A.inv_cmax2 > 0.0 ? cell_ctot<NDIM, kExtCmax>(q, K) : cell_ctot<NDIM>(q, K));
    if (!(q[0] > 0.0)) bad |= kBadRho;
    if (!(ct < INFINITY)) bad |= kNonFinite;
    cm = fmax(cm, ct);
  }
  if (bad) atomicOr((unsigned*)(A.scal + kFlags), bad);
  const double wm = wave_max(cm);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = wm;
  __syncthreads();
  if (threadIdx.x == 0) {
    A.blkmax_out[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    if (set_t && blockIdx.x == 0) *A.t_out = t0;
  }
}

// ---------------------------------------------------------------- diag

constexpr int kDiagThreads = 256;
constexpr int kDiagBlocks = 1024;

// Per-block partial sums (fixed order: strided per thread, tree per block).
template <int NDIM, typename ST>
__global__ void __launch_bounds__(kDiagThreads) diag_partial_kernel(const StageArgs A,
                                                                    const ST* __restrict__ u,
                                                                    double* __restrict__ part) {
  constexpr int NV = NDIM + 2;
  const Consts K{A.gamma, A.gm1, A.inv_gm1, A.inv_xi, A.f, A.inv_cmax2, A.vdw_a, A.vdw_b};
  const Geometry& G = A.geo;
  __shared__ double s[8][kDiagThreads];
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < A.ncell;
       c += (long long)gridDim.x * blockDim.x) {
    double q[NV];
    const int i = (int)(c % G.nx);
    const long long r = c / G.nx;
    const int j = (int)(r % G.ns);
    const int k = (int)(r / G.ns);
#pragma unroll
    for (int v = 0; v < NV; ++v) q[v] = (double)u[v * A.ncell + c];
    if constexpr (sizeof(ST) == 4) {
      int b = 0;
      if (A.bg_axis == 0) b = i;
      else if (A.bg_axis == 1) b = (NDIM == 3) ? j : k;
      else if (A.bg_axis == 2) b = k;
#pragma unroll
      for (int v = 0; v < NV; ++v) q[v] += A.bg[v * A.nbg + b];
    }
    const double rinv = 1.0 / q[0];
    double m2 = 0.0, mv = 0.0;
    acc[0] += q[0];
#pragma unroll
    for (int e = 0; e < NDIM; ++e) {
      acc[1 + e] += q[1 + e];
      m2 = fma(q[1 + e], q[1 + e], m2);
    }
    acc[4] += q[NV - 1];
    acc[5] += 0.5 * m2 * rinv;
    mv = m2 * rinv;
    const double v = sqrt(m2) * rinv;
    double P, a2;
    if (A.eos) eos_pa2<kExtVdw>(q[0], rinv, q[NV - 1] - 0.5 * mv, K, P, a2);
    else eos_pa2<0>(q[0], rinv, q[NV - 1] - 0.5 * mv, K, P, a2);
    const double ae = A.inv_cmax2 > 0.0 ? a_eff_cmax(a2, K) : sqrt(a2) * A.inv_xi;  // a / xi
    acc[6] = fmax(acc[6], v);
    acc[7] = fmax(acc[7], v / ae);
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) s[q][threadIdx.x] = acc[q];
  __syncthreads();
  for (int h = kDiagThreads / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
#pragma unroll
      for (int q = 0; q < 6; ++q) s[q][threadIdx.x] += s[q][threadIdx.x + h];
      s[6][threadIdx.x] = fmax(s[6][threadIdx.x], s[6][threadIdx.x + h]);
      s[7][threadIdx.x] = fmax(s[7][threadIdx.x], s[7][threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x < 8) part[blockIdx.x * 8 + threadIdx.x] = s[threadIdx.x][0];
}

__global__ void __launch_bounds__(kDiagThreads) diag_final_kernel(const double* __restrict__ part,
                                                                  int np, double vol,
                                                                  double* __restrict__ out) {
  __shared__ double s[8][kDiagThreads];
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.x; b < np; b += blockDim.x) {
#pragma unroll
    for (int q = 0; q < 6; ++q) acc[q] += part[b * 8 + q];
    acc[6] = fmax(acc[6], part[b * 8 + 6]);
    acc[7] = fmax(acc[7], part[b * 8 + 7]);
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) s[q][threadIdx.x] = acc[q];
  __syncthreads();
  for (int h = kDiagThreads / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
#pragma unroll
      for (int q = 0; q < 6; ++q) s[q][threadIdx.x] += s[q][threadIdx.x + h];
      s[6][threadIdx.x] = fmax(s[6][threadIdx.x], s[6][threadIdx.x + h]);
      s[7][threadIdx.x] = fmax(s[7][threadIdx.x], s[7][threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x < 8) out[threadIdx.x] = s[threadIdx.x][0] * (threadIdx.x < 6 ? vol : 1.0);
}

// ---------------------------------------------------------------- host side

// Rows (2D) or planes (3D) per march of the planned grid, unless the
// environment variable RSST_KM, read when a solver is made, sets it: the
// results do not depend on it, which a GPU test checks for several lengths.
static int chunk_override(int km) {
  if (const char* e = getenv("RSST_KM")) {
    const int v = atoi(e);
    if (v >= 1 && v <= 4096) return v;
  }
  return km;
}

// About the us of a stage by whole-row workgroups of chunks of q rows (less some
// 4 of launch and first loads): a row takes a wave alone on its SIMD 1.4 (rows
// of several waves, which wait for each other, 1.5), two waves 2.4, each further
// one 0.9 (1.0); four fit a SIMD, and a chunk starts with the time of 1.5 (0.5)
// rows.  Fitted to 128 grids of 1000 to 131072 wave-rows, rows of 1, 2, 3, 4 and
// 8 waves, both storage types: the chunk it picks is within 1% of the best
// measured on average, 6 to 11% off at the worst.
static double rows_cost(int nwx, int nm, int q) {
  const int per = 16 / nwx, p = ((nm + q - 1) / q + 255) / 256;  // workgroups a CU holds, and gets
  const double one = nwx == 1 ? 1.4 : 1.5, more = nwx == 1 ? 0.9 : 1.0, start = nwx == 1 ? 1.5 : 0.5;
  auto row = [&](int wg) {
    const double w = wg * nwx / 4.0;
    return wg == 0 ? 0.0 : (w <= 1.0 ? one : 2.4 + (w - 2.0) * more);
  };
  return (q + start) * ((p / per) * row(per) + row(p % per));
}

// The chunk of the least rows_cost (left in `cost`).  At most 35 rows, or what
// makes one round of all workgroups (more of them read more maxima, each all of
// them: 64 x 10^6 FP64 4.4 ms per step with 24 rows, 2.6 with 257).  From 8 rows
// on odd ones only: chunks whose first rows are a power of two apart meet in the
// same memory channels (128 x 65536 FP64 403 us with 16 rows, 379 with 32, 323
// with 33).
static int rows_chunk(int nwx, int nm, double& cost) {
  const int full = 256 * (16 / nwx), top = std::max(35, (nm + full - 1) / full | 1);
  int km = 1;
  cost = 1e300;
  for (int q = 1; q <= top && q <= nm; q += q < 7 ? 1 : 2) {
    const double c = rows_cost(nwx, nm, q);
    if (c < cost) { cost = c; km = q; }
  }
  return km;
}

Geometry plan_geometry(int ndim, const int n[3], bool x_per) {
  Geometry G{};
  G.ndim = ndim;
  G.nx = n[0];
  G.ns = (ndim == 3) ? n[1] : 1;
  G.nm = (ndim == 3) ? n[2] : (ndim == 2 ? n[1] : 1);
  G.nwx = (G.nx + 63) / 64;
  G.ts = 1;
  G.km = 1;
  if (ndim == 2) {
    // One stage per launch.  A chunk of km rows costs a wave about km + 1/2
    // rows (it re-reads four and forms one extra face to start), a row 1.05
    // us on a SIMD of its own and 0.8 us where waves share one (1024 SIMDs),
    // and the slowest SIMD decides: the cheapest km.  Measured against the
    // best of 16 lengths when the rule was made: 22.3 us per step (km 5) at
    // 512^2, best 22.3; 54.2 (10) at 1024^2, best 54.2; 133 (10) at 1000 x
    // 3000, best 131 (the last two now take 49 and 110)
    G.cols = plan_cols2(G.nx, x_per, 2);
    int km = 1;
    double best = 1e300;
    for (int q = 1; q <= 64 && q <= G.nm; ++q) {
      const long long w = ((long long)G.cols.ncol * ((G.nm + q - 1) / q) + 1023) / 1024;
      const double c = (w == 1 ? 1.05 : 0.8 * (double)w) * (q + 0.5);
      if (c < best) { best = c; km = q; }
    }
    // Whole rows instead (a workgroup of nwx waves holds a row, three barriers
    // per row) where strips would need more waves for it.  Up to four waves per
    // SIMD a step is mostly latency and whole rows are faster (us per step,
    // rows and strips: 256 x 256 10.7 and 13.1, 256 x 1000 18.8 and 20.9, 512 x
    // 512 18.5 and 21.2, 192 x 341 13.0 and 13.2), but rows of five to seven
    // waves only while a CU has one (384 x 256 12.6 and 13.6, 384 x 341 18.1 and
    // 16.2).  On larger grids rows of one, two and four waves, which fill the
    // SIMDs, and of three on the largest, by what either costs: strips 1.04 us
    // per row and SIMD, of whose lanes they waste a fifth to a half there (64
    // cells between walls: 64 x 8000 FP64 35 and 40, 64 x 65536 165 and 240; 128
    // x 30000 139 and 178; 256 x 16384 151 and 172, but 256 x 1100 24.5 and 21.2;
    // 192 x 20000 150 and 160, but 192 x 5000 48.7 and 47.9).  Rows of eight
    // stay with strips there (512 x 16384 FP64 314 and 331, but FP32, by a kernel
    // of three waves per SIMD, 314 and 295).
    const long long waves = (long long)G.nwx * G.nm;
    if (G.cols.ncol > G.nwx && G.nwx <= 8) {
      double cost;
      const int q = rows_chunk(G.nwx, G.nm, cost);
      if (waves <= 4096) G.rows = G.nwx <= 4 || G.nwx == 8 || G.nm <= 256;
      else G.rows = (G.nwx == 1 || G.nwx == 2 || G.nwx == 4 || (G.nwx == 3 && waves >= 32768)) &&
                    cost < 0.2 + 1.04 * G.cols.ncol * (double)G.nm / 1024.0;
      if (G.rows) km = q;
    }
    km = chunk_override(km);
    G.km = km < G.nm ? km : G.nm;
    G.ntile_s = 1;
    G.nchunk = (G.nm + G.km - 1) / G.km;
    if (G.rows) {
      G.nblk = G.nchunk;
      G.threads = 64 * G.nwx;
      G.lds_bytes = (size_t)carve2(G.nwx).total * sizeof(double);
    } else {
      G.nblk = (G.cols.ncol * G.nchunk + kWaves2 - 1) / kWaves2;
      G.threads = 64 * kWaves2;
      G.lds_bytes = (size_t)(kRed2 + kWaves2) * sizeof(double);
    }
    // Both stages in one launch: tiles of 4 r rows, one per CU (256) at a
    // time, each 4.4 us and 0.85 us per row of its SIMDs (r + 1 rows of stage
    // 1, r of stage 2): the smallest r that needs one round.  It saves a
    // launch, the stage's start-up and the way of U1 through memory, and
    // repeats the halo: with one tile per CU it is the faster one (us per
    // step, against one stage per launch: 64^2 8.5 and 9.7, 389 x 301 13.9 and
    // 16.4, 512^2 18.8 and 19.4, 700 x 500 21.3 and 24.1), with more the tiles'
    // start-ups come one after the other (1024^2: 56 and 50)
    G.colsF = plan_cols2(G.nx, x_per, 4);
    G.rF = 1;
    while (G.rF < kMaxRF && (long long)G.colsF.ncol * ((G.nm + 4 * G.rF - 1) / (4 * G.rF)) > 256) ++G.rF;
    G.fused = (long long)G.colsF.ncol * ((G.nm + 4 * G.rF - 1) / (4 * G.rF)) <= 256;
    if (const int r = chunk_override(0)) G.rF = r < kMaxRF ? r : kMaxRF;
    G.nblkF = G.colsF.ncol * ((G.nm + 4 * G.rF - 1) / (4 * G.rF));
    G.nslot = G.nblk > G.nblkF ? G.nblk : G.nblkF;
    return G;
  }
  if (ndim == 3) {
    // 3D rows of 5-8 waves run as rows of 8 (the waves past the row's end
    // compute on clamped cells and store nothing)
    if (G.nwx > 4) G.nwx = 8;
    // an even number of rows (two per thread), at most the grid's (>= 4)
    G.ts = tile_rows3(G.nwx) < (G.ns & ~1) ? tile_rows3(G.nwx) : (G.ns & ~1);
  }
  G.ntile_s = (G.ns + G.ts - 1) / G.ts;
  if (ndim == 3) {
    // A CU holds eight waves (two per SIMD), one full tile or several of a grid
    // with fewer rows than a tile (two of up to four waves, four of two), so the
    // grid runs in rounds of that many workgroups per CU, each as long as its
    // chunk of km planes plus about 0.7 plane of start-up (a chunk re-reads 4
    // planes and forms one extra face): the cheapest km.
    // (Halving 128 planes until there were 256 workgroups left 187 x 141 x 230
    // at 288, two rounds of 32 planes where one of 33 does: FP32 1.04 ms per
    // step, 0.55 with it.  One workgroup per CU whatever its size left SIMDs
    // empty: 8 x 8 x 2000 FP64 83 us with chunks of 8, 66 with 4; 64 x 4 x 2000
    // 76 with 8, 45 with 2; halved until 256 workgroups, 66 and 61 with 4.)
    const int per_cu = 8 / (G.nwx * G.ts / 2);
    int km = 1;
    double best = 1e300;
    for (int q = 1; q <= 128 && q <= G.nm; ++q) {
      const long long round = 256ll * per_cu, rounds = ((long long)G.ntile_s * ((G.nm + q - 1) / q) + round - 1) / round;
      const double c = (double)rounds * (q + 0.7);
      if (c < best) { best = c; km = q; }
    }
    km = chunk_override(km);
    G.km = km < G.nm ? km : G.nm;
  }
  G.nchunk = (G.nm + G.km - 1) / G.km;
  G.nblk = G.nslot = G.ntile_s * G.nchunk;
  G.threads = 64 * G.nwx * (ndim == 3 ? G.ts / 2 : G.ts);
  G.lds_bytes = (size_t)(ndim == 3 ? carve3(G.ts, G.nwx).total : carve1(G.nwx).total) * sizeof(double);
  return G;
}

template <typename ST>
static hipError_t launch_stage_p(const StageArgs& a, int stage, hipStream_t s) {
  switch (a.geo.ndim) {
    case 1: return launch_stage_n<1, ST, false>(a, stage, s);
    case 2: return launch_stage_n<2, ST, false>(a, stage, s);
    default: return a.big ? launch_stage_n<3, ST, true>(a, stage, s) : launch_stage_n<3, ST, false>(a, stage, s);
  }
}

hipError_t launch_stage(const StageArgs& a, int stage, hipStream_t s) {
  return a.prec ? launch_stage_p<float>(a, stage, s) : launch_stage_p<double>(a, stage, s);
}

template <typename ST>
static hipError_t launch_prime_p(const StageArgs& a, const void* u, double t0, int set_t,
                                 hipStream_t s) {
  const dim3 grid((unsigned)a.nslot), block(256);
  switch (a.geo.ndim) {
    case 1: hipLaunchKernelGGL((prime_kernel<1, ST>), grid, block, 0, s, a, (const ST*)u, t0, set_t); break;
    case 2: hipLaunchKernelGGL((prime_kernel<2, ST>), grid, block, 0, s, a, (const ST*)u, t0, set_t); break;
    default: hipLaunchKernelGGL((prime_kernel<3, ST>), grid, block, 0, s, a, (const ST*)u, t0, set_t); break;
  }
  return hipGetLastError();
}

hipError_t launch_prime(const StageArgs& a, const void* u, double t0, int set_t, hipStream_t s) {
  return a.prec ? launch_prime_p<float>(a, u, t0, set_t, s)
                : launch_prime_p<double>(a, u, t0, set_t, s);
}

// The next CFL step's dt, for reporting: one workgroup runs the grid maximum
// and the dt formula of stage 1 over the stored maxima.
__global__ void __launch_bounds__(256) next_dt_kernel(const StageArgs A) {
  __shared__ double red[4];
  GridMax gm;
  gm.begin(A, red);
  const double m = gm.finish(A, red);
  if (threadIdx.x == 0) A.scal[kDtNext] = m > 0.0 ? cfl_dt_of_max(A, m) : 0.0;
}

hipError_t launch_next_dt(const StageArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(next_dt_kernel, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

int diag_partials(long long ncell) {
  long long nb = (ncell + kDiagThreads - 1) / kDiagThreads;
  return (int)(nb < kDiagBlocks ? nb : kDiagBlocks);
}

template <typename ST>
static hipError_t launch_diag_p(const StageArgs& a, const void* u, double* part, int np,
                                double* out8, hipStream_t s) {
  const dim3 grid((unsigned)np), block(kDiagThreads);
  switch (a.geo.ndim) {
    case 1: hipLaunchKernelGGL((diag_partial_kernel<1, ST>), grid, block, 0, s, a, (const ST*)u, part); break;
    case 2: hipLaunchKernelGGL((diag_partial_kernel<2, ST>), grid, block, 0, s, a, (const ST*)u, part); break;
    default: hipLaunchKernelGGL((diag_partial_kernel<3, ST>), grid, block, 0, s, a, (const ST*)u, part); break;
  }
  double vol = 1.0;
  for (int d = 0; d < a.geo.ndim; ++d) vol /= a.inv_dx[d];
  hipLaunchKernelGGL(diag_final_kernel, dim3(1), dim3(kDiagThreads), 0, s, part, np, vol, out8);
  return hipGetLastError();
}

hipError_t launch_diag(const StageArgs& a, const void* u, double* part, int np, double* out8,
                       hipStream_t s) {
  return a.prec ? launch_diag_p<float>(a, u, part, np, out8, s)
                : launch_diag_p<double>(a, u, part, np, out8, s);
}

}  // namespace rsstk
