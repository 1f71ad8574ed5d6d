// Stage kernels of one dimension and storage type, instantiated for every
// form (with and without xi from the sound speed), row width and stage.
// Compiled once per (RSST_INST_NDIM, RSST_INST_ST, RSST_INST_BIG) so the
// library builds in parallel objects; RSST_INST_BIG = 1 builds the 3D
// kernels that address states of 2 GiB or more (Field64).
#include "rsst_row2.h"
#include "rsst_stage1.h"
#include "rsst_stage2.h"
#include "rsst_stage3.h"

#pragma clang fp contract(off)

#ifndef RSST_INST_NDIM
#error "RSST_INST_NDIM (1, 2 or 3) must be defined"
#endif
#ifndef RSST_INST_ST
#error "RSST_INST_ST (double or float) must be defined"
#endif
#ifndef RSST_INST_BIG
#define RSST_INST_BIG 0
#endif

namespace rsstk {

// FORM: the correction form, plus kExtCmax when xi follows the sound speed
// (eq. cx), kExtVdw for the van der Waals gas, kExtHydro for hydrostatic walls.
// 3D workgroups are at most 512 threads (8 waves at ~200 VGPRs, two waves per
// SIMD); 1D and 2D rows take up to 1024.
constexpr int kMaxThreads3 = 512;

constexpr bool kBig = RSST_INST_BIG != 0;

// The step's dt: given, or (stage 1) formed from the maxima and
// recorded for a separate stage 2.  begin() and finish() as GridMax's.
template <int STAGE>
struct StepDt {
  const StageArgs& A;
  double* red;
  GridMax gm;
  __device__ __forceinline__ void begin() {
    if constexpr (STAGE == 1) {
      if (!(A.dt_fixed > 0.0)) gm.begin(A, red);
    }
  }
  __device__ __forceinline__ double finish() const {
    if (A.dt_fixed > 0.0) return A.dt_fixed;
    if constexpr (STAGE == 1) {
      const double dt = cfl_dt_of_max(A, gm.finish(A, red));
      if (blockIdx.x == 0 && threadIdx.x == 0) A.scal[kDtCur] = dt;
      return dt;
    } else {
      return A.scal[kDtCur];
    }
  }
};

template <int NDIM, int STAGE, typename ST, int FORM, int NWXC, bool BIG>
__global__ void __launch_bounds__(NDIM == 3 ? kMaxThreads3 : 1024) stage_kernel(const StageArgs A) {
  extern __shared__ double lds[];
  static_assert(NDIM != 2, "2D grids run stage_kernel2d");
  const Geometry& G = A.geo;
  double* red = lds + (NDIM == 3 ? carve3(G.ts, NWXC).red : carve1(G.nwx).red);
  StepDt<STAGE> sd{A, red, {}};
  sd.begin();
  unsigned bad = 0;
  double cmax, dt = 0.0;
  if constexpr (NDIM == 3) {
    const int L = xcd_tile(blockIdx.x, G.nblk);
    cmax = stage_body3<STAGE, ST, FORM, NWXC, BIG>(A, lds, L % G.ntile_s, L / G.ntile_s,
                                                   [&]() { return dt = sd.finish(); }, bad);
  } else {
    dt = sd.finish();
    cmax = stage_body1<STAGE, ST, FORM>(A, lds, dt, bad);
  }
  if (bad) atomicOr((unsigned*)(A.scal + kFlags), bad);
  if constexpr (STAGE == 2) cfl_epilogue(A, red, cmax, dt, A.nslot);
}

// 2D grids, one stage: a workgroup is four independent waves, each one strip
// of a chunk (rsst_stage2.h).  Four waves per SIMD (128 VGPRs) hide a row's
// latencies.
template <int STAGE, typename ST, int FORM>
__global__ void __launch_bounds__(64 * kWaves2) __attribute__((amdgpu_waves_per_eu(4))) stage_kernel2d(
    const StageArgs A) {
  extern __shared__ double lds[];
  fetch_args2(A);
  const Geometry& G = A.geo;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int task = xcd_tile(blockIdx.x, G.nblk) * kWaves2 + w, ntask = G.cols.ncol * G.nchunk;
  const bool work = task < ntask;
  const int t = work ? task : ntask - 1;
  const int k0 = (t / G.cols.ncol) * G.km;
  const int k1 = work ? min(k0 + G.km, G.nm) : k0 + 1;
  unsigned bad = 0;
  double dt = 0.0;
  const Tile2 none{nullptr, 0, 0};
  StepDt<STAGE> sd{A, lds + kRed2, {}};
  sd.begin();
  const double cmax = march2<kSplit, STAGE, ST, FORM>(
      A, lane_of(G.cols, G.nx, A.bc_lo[0] == 0, t % G.cols.ncol), lds + w * kLds2, none, k0, k1, k0, k1, work,
      [&]() { return dt = sd.finish(); }, bad);
  if (bad) atomicOr((unsigned*)(A.scal + kFlags), bad);
  if constexpr (STAGE == 2) cfl_epilogue(A, lds + kRed2, cmax, dt, A.nslot);
}

// 2D grids, one stage, a workgroup per whole row (rsst_row2.h): up to 8 waves.
// (16, for rows of 961 to 1024 cells, would hold every form to 128 VGPRs, which
// some exceed: FP32 512 x 512 19.1 us per step instead of 18.1, 256 x 256 11.3
// and 11.1; 1024 x 32768 FP64, 1222 instead of 1319, was the only gain.)
template <int STAGE, typename ST, int FORM>
__global__ void __launch_bounds__(512) row_kernel2d(const StageArgs A) {
  extern __shared__ double lds[];
  double* red = lds + carve2(A.geo.nwx).red;
  StepDt<STAGE> sd{A, red, {}};
  sd.begin();
  unsigned bad = 0;
  double dt = 0.0;
  const double cmax = stage_body2<STAGE, ST, FORM>(A, lds, xcd_tile(blockIdx.x, A.geo.nblk),
                                                   [&]() { return dt = sd.finish(); }, bad);
  if (bad) atomicOr((unsigned*)(A.scal + kFlags), bad);
  if constexpr (STAGE == 2) cfl_epilogue(A, red, cmax, dt, A.nslot);
}

// 2D grids, both stages of a step (rsst_stage2.h): one workgroup per CU, two
// waves per SIMD with all the registers.
template <typename ST, int FORM>
__global__ void __launch_bounds__(64 * kWavesF) __attribute__((amdgpu_waves_per_eu(2, 2)))
step_kernel2d(const StageArgs A) {
  extern __shared__ double lds[];
  fetch_args2(A);
  asm volatile("" ::"s"(A.geo.nslot));
  double* red = lds + lds_doublesF(A.geo.rF) - kWavesF;
  unsigned bad = 0;
  double dt = 0.0;
  StepDt<1> sd{A, red, {}};
  sd.begin();
  const double cmax = step_tile2<ST, FORM>(A, lds, xcd_tile(blockIdx.x, A.geo.nblkF),
                                           [&]() { return dt = sd.finish(); }, bad);
  if (bad) atomicOr((unsigned*)(A.scal + kFlags), bad);
  cfl_epilogue(A, red, cmax, dt, A.geo.nslot);
}

// One launch of a stage kernel over the geometry's grid.  The kernel's LDS
// limit is raised only when a larger tile needs it (lds_set: the limit set
// so far per device, owned by the kernel's launcher), so launches of a known
// shape (e.g. under HIP graph capture) make no attribute call.
static hipError_t launch_geo(void (*kern)(StageArgs), int* lds_set, int nblk, int threads, size_t lds_bytes,
                             const StageArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)nblk), block((unsigned)threads);
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if ((int)lds_bytes > lds_set[dev]) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
    lds_set[dev] = (int)lds_bytes;
  }
  hipLaunchKernelGGL(kern, grid, block, lds_bytes, s, a);
  return hipGetLastError();
}

template <int NDIM, int STAGE, typename ST, int FORM, int NWXC>
static hipError_t launch_stage_k(const StageArgs& a, hipStream_t s) {
  static int lds_set[64] = {0};
  return launch_geo(stage_kernel<NDIM, STAGE, ST, FORM, NWXC, kBig>, lds_set, a.geo.nblk, a.geo.threads, a.geo.lds_bytes,
                    a, s);
}

template <int STAGE, typename ST, int FORM>
static hipError_t launch_rows_2d(const StageArgs& a, hipStream_t s) {
  static int lds_set[64] = {0};
  return launch_geo(row_kernel2d<STAGE, ST, FORM>, lds_set, a.geo.nblk, a.geo.threads, a.geo.lds_bytes, a, s);
}

template <int STAGE, typename ST, int FORM>
static hipError_t launch_stage_2d(const StageArgs& a, hipStream_t s) {
  if (a.geo.rows) return launch_rows_2d<STAGE, ST, FORM>(a, s);
  static int lds_set[64] = {0};
  return launch_geo(stage_kernel2d<STAGE, ST, FORM>, lds_set, a.geo.nblk, a.geo.threads, a.geo.lds_bytes, a, s);
}

template <typename ST, int FORM>
static hipError_t launch_step_2d(const StageArgs& a, hipStream_t s) {
  static int lds_set[64] = {0};
  return launch_geo(step_kernel2d<ST, FORM>, lds_set, a.geo.nblkF, 64 * kWavesF,
                    (size_t)lds_doublesF(a.geo.rF) * sizeof(double), a, s);
}

// STAGE 0: both stages of a 2D step.
template <int NDIM, int STAGE, typename ST, int FORM>
static hipError_t launch_stage_t(const StageArgs& a, hipStream_t s) {
  if constexpr (NDIM == 3) {
    switch (a.geo.nwx) {
      case 1: return launch_stage_k<NDIM, STAGE, ST, FORM, 1>(a, s);
      case 2: return launch_stage_k<NDIM, STAGE, ST, FORM, 2>(a, s);
      case 3: return launch_stage_k<NDIM, STAGE, ST, FORM, 3>(a, s);
      case 4: return launch_stage_k<NDIM, STAGE, ST, FORM, 4>(a, s);
      case 8: return launch_stage_k<NDIM, STAGE, ST, FORM, 8>(a, s);
      default: return hipErrorInvalidValue;
    }
  } else if constexpr (NDIM == 2) {
    if constexpr (STAGE == 0) return launch_step_2d<ST, FORM>(a, s);
    else return launch_stage_2d<STAGE, ST, FORM>(a, s);
  } else {
    return launch_stage_k<NDIM, STAGE, ST, FORM, 0>(a, s);
  }
}

template <int NDIM, int STAGE, typename ST, int X>
static hipError_t launch_stage_x(const StageArgs& a, hipStream_t s) {
  switch (a.form) {
    case kEuler: return launch_stage_t<NDIM, STAGE, ST, kEuler | X>(a, s);
    case kPVS: return launch_stage_t<NDIM, STAGE, ST, kPVS | X>(a, s);
    case kPMS: return launch_stage_t<NDIM, STAGE, ST, kPMS | X>(a, s);
    case kDVS: return launch_stage_t<NDIM, STAGE, ST, kDVS | X>(a, s);
    case kDMS: return launch_stage_t<NDIM, STAGE, ST, kDMS | X>(a, s);
    default: return launch_stage_t<NDIM, STAGE, ST, kPD | X>(a, s);
  }
}

// The van der Waals and hydrostatic-wall kernels exist for FP64 storage only
// (the C ABI rejects the other combinations before any launch); 1D grids
// need no hydrostatic variant (their walls are x walls, allowed only without
// a force along x, where they are mirror walls).
template <int NDIM, int STAGE, typename ST, int H>
static hipError_t launch_stage_g(const StageArgs& a, hipStream_t s) {
  if (a.eos) return launch_stage_x<NDIM, STAGE, ST, kExtVdw | H>(a, s);
  return a.inv_cmax2 > 0.0 ? launch_stage_x<NDIM, STAGE, ST, kExtCmax | H>(a, s)
                           : launch_stage_x<NDIM, STAGE, ST, H>(a, s);
}

template <int NDIM, int STAGE, typename ST>
static hipError_t launch_stage_f(const StageArgs& a, hipStream_t s) {
  if constexpr (sizeof(ST) == 8) {
    if constexpr (NDIM >= 2) {
      if (a.hydro) return launch_stage_g<NDIM, STAGE, ST, kExtHydro>(a, s);
    }
    return launch_stage_g<NDIM, STAGE, ST, 0>(a, s);
  } else {
    if (a.eos || a.hydro) return hipErrorInvalidValue;
    return a.inv_cmax2 > 0.0 ? launch_stage_x<NDIM, STAGE, ST, kExtCmax>(a, s)
                             : launch_stage_x<NDIM, STAGE, ST, 0>(a, s);
  }
}

template <int NDIM, typename ST, bool BIG>
hipError_t launch_stage_n(const StageArgs& a, int stage, hipStream_t s) {
  static_assert(BIG == kBig, "one addressing per object");
  return stage == 1 ? launch_stage_f<NDIM, 1, ST>(a, s) : launch_stage_f<NDIM, 2, ST>(a, s);
}

#if RSST_INST_NDIM == 2
template <typename ST>
hipError_t launch_step2d(const StageArgs& a, hipStream_t s) {
  return launch_stage_f<2, 0, ST>(a, s);
}

template hipError_t launch_step2d<RSST_INST_ST>(const StageArgs&, hipStream_t);
#endif

template hipError_t launch_stage_n<RSST_INST_NDIM, RSST_INST_ST, kBig>(const StageArgs&, int, hipStream_t);

#if RSST_INST_NDIM == 1 && !RSST_INST_BIG
// nsteps whole steps of a 1D grid in one launch.  A 1D grid is one workgroup
// (a row of at most 16 waves), so both stages and the CFL maximum of every
// step run in that workgroup with barriers in between, and each lane keeps
// its own cell in registers from the first load to the last store: the
// stage bodies are those of stage_kernel in their register-resident form
// (stage input, step-start state and output in registers, each equal to
// what storing and reloading would give; neighbours come by DPP and LDS as
// always), each step's dt is formed from the previous step's maximum as
// stage 1 forms it from the stored maxima, and t and dt stay in registers.
// So the state, t and the next dt after each step are bitwise those of the
// per-stage launches.  U is written once, at the end (and the stage buffer
// not at all).  With a CFL step and an end time, the steps after t reaches
// t_end (dt = 0, which would leave U unchanged) are skipped.  a1: stage 1
// (U -> U1), a2: stage 2.
template <typename ST, int FORM>
__global__ void __launch_bounds__(1024) steps1d_kernel(const StageArgs a1, const StageArgs a2, int nsteps) {
  constexpr int NV = 3;
  extern __shared__ double lds[];
  const Geometry& G = a1.geo;
  double* red = lds + carve1(G.nwx).red;
  const bool cfl = !(a1.dt_fixed > 0.0);
  double t = *a1.t_in;
  double dt = a1.dt_fixed;
  if (cfl) {  // from the one stored maximum (a 1D grid is one workgroup), as stage 1 forms it
    dt = a1.cfl_h / a1.blkmax[0];
    if (a1.t_end > 0.0) dt = fmin(dt, fmax(a1.t_end - t, 0.0));
  }
  // this lane's cell (lanes past the row hold the last cell and store nothing)
  const int i = min((int)threadIdx.x, G.nx - 1);
  RegCell<NV> c;
  {
    ST raw[NV];
    load_cell_raw<1, ST>(make_field<false>(a1.uin, a1.ncell, NV, (int)sizeof(ST), G.nx * (int)sizeof(ST)), 0,
                         i * (int)sizeof(ST), raw);
    const int b = (sizeof(ST) == 4 && !a1.bg_uniform) ? bg_index<1>(a1, i, 0, 0) : 0;
    finish_cell<1, ST>(a1, raw, -1, b, c.in);
  }
  double stu[NV];  // stored values of the state after the last step
  unsigned bad = 0;
  double mlast = -1.0;
  for (int q = 0; q < nsteps; ++q) {
    if (cfl && a1.t_end > 0.0 && !(dt > 0.0)) break;
#pragma unroll
    for (int v = 0; v < NV; ++v) c.out[v] = c.in[v];
    stage_body1<1, ST, FORM, true>(a1, lds, dt, bad, &c);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      c.un[v] = c.in[v];
      c.in[v] = c.out[v];
    }
    const double cm = stage_body1<2, ST, FORM, true>(a2, lds, dt, bad, &c);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      c.in[v] = c.out[v];
      stu[v] = c.st[v];
    }
    const double wm = wave_max(cm);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = wm;
    __syncthreads();
    double m = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, red[w]);
    mlast = m;
    t = t + dt;
    if (cfl) {
      dt = a1.cfl_h / m;
      if (a1.t_end > 0.0) dt = fmin(dt, fmax(a1.t_end - t, 0.0));
    }
    __syncthreads();
  }
  if (mlast >= 0.0 && (int)threadIdx.x < G.nx) {
    ST* u = (ST*)a2.uout;
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v * a2.ncell + i] = (ST)stu[v];
  }
  if (bad) atomicOr((unsigned*)(a1.scal + kFlags), bad);
  if (threadIdx.x == 0) {
    *a1.t_out = t;
    if (mlast >= 0.0) a1.blkmax_out[0] = mlast;  // the maximum of the state left in U
  }
}

// The same run by waves with halo lanes (rsst_stage1.h), rows of at most
// kMaxHalo1 cells: LDS holds the cells and the waves' maxima twice, by the
// parity of the step, so that one barrier per step orders a step's writes
// before its reads and those before the writes two steps on.  The same bits.
template <typename ST, int FORM>
__global__ void __launch_bounds__(1024) steps1d_halo_kernel(const StageArgs A, int nsteps) {
  constexpr int NV = 3;
  constexpr int EXT = FORM & (kExtCmax | kExtVdw);
  constexpr bool F32 = sizeof(ST) == 4;
  extern __shared__ double lds[];
  const int nx = A.geo.nx, nw = blockDim.x >> 6, cw = (nx + nw - 1) / nw;
  double* const cells = lds;                 // [2][NV][nx]
  double* const maxima = lds + 2 * NV * nx;  // [2][nw]
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool x_per = A.bc_lo[0] == 0;
  // the lane's cell, and whether it is a wall's ghost
  const int x0 = w * cw, q = min(x0 + lane - kHalo1, nx + kHalo1 - 1);
  const int i = q < 0 ? (x_per ? q + nx : -1 - q) : (q >= nx ? (x_per ? q - nx : 2 * nx - 1 - q) : q);
  const bool ghost = !x_per && (q < 0 || q >= nx);
  const bool own = lane >= kHalo1 && lane < kHalo1 + min(cw, nx - x0);
  const int flip = ghost ? (int)0x80000000 : 0;
  auto mirrored = [&](double x) { return __hiloint2double(__double2hiint(x) ^ flip, __double2loint(x)); };
  const Consts K{A.gamma, A.gm1, A.inv_gm1, A.inv_xi, A.f, A.inv_cmax2, A.vdw_a, A.vdw_b};
  const double g[3] = {mirrored(A.g[0]), 0.0, 0.0};
  const double hx = 0.5 * A.inv_dx[0];
  double bg[NV] = {}, u[NV], st[NV] = {};
  const ST* in = (const ST*)A.uin;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    if constexpr (F32) bg[v] = A.bg[v * A.nbg + (A.bg_axis == 0 ? i : 0)];
    u[v] = (double)in[v * A.ncell + i];
    if constexpr (F32) u[v] += bg[v];
  }
  u[1] = mirrored(u[1]);
  const bool cfl = !(A.dt_fixed > 0.0);
  double t = *A.t_in, dt = A.dt_fixed;
  double m = A.blkmax[0], mlast = -1.0;
  unsigned bad = 0;
  for (int n = 0; n < nsteps; ++n) {
    if (cfl) {
      dt = A.cfl_h / m;
      if (A.t_end > 0.0) {
        dt = fmin(dt, fmax(A.t_end - t, 0.0));
        if (!(dt > 0.0)) break;
      }
    }
    // a lane's stored value and what the next stage reads back from it
    // (rounded to the storage type; a ghost's rounds to its cell's mirror
    // image: its background momentum is its cell's)
    double y[NV], u1[NV];
    unsigned b = lane_stage1<FORM>(u, K, g, hx, dt, y);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if constexpr (F32) {
        const double x = v == 1 ? mirrored(y[v]) : y[v];
        const double r = (double)(ST)(x - bg[v]) + bg[v];
        u1[v] = v == 1 ? mirrored(r) : r;
      } else {
        u1[v] = y[v];
      }
    }
    b |= lane_stage1<FORM>(u1, K, g, hx, dt, y);
    double out[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      y[v] = 0.5 * (u[v] + y[v]);
      const ST r = (ST)(y[v] - bg[v]);
      st[v] = (double)r;
      if constexpr (F32) out[v] = st[v] + bg[v];
      else out[v] = y[v];
    }
    if (own) bad |= b;
    // publish the new cells and the wave's largest c_tot, then read the cell
    // (a halo lane's from the wave that owns it) and the maxima
    double* const c = cells + (n & 1) * NV * nx;
    double* const mx = maxima + (n & 1) * nw;
    const double wm = wave_max(own ? cell_ctot<1, EXT>(out, K) : 0.0);
    if (own) {
#pragma unroll
      for (int v = 0; v < NV; ++v) c[v * nx + i] = out[v];
    }
    if (lane == 0) mx[w] = wm;
    t = t + dt;
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = c[v * nx + i];
    u[1] = mirrored(u[1]);
    m = 0.0;
    for (int k = 0; k < nw; ++k) m = fmax(m, mx[k]);
    mlast = m;
  }
  if (mlast >= 0.0 && own) {
    ST* out = (ST*)A.uout;
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v * A.ncell + i] = (ST)st[v];
  }
  if (bad) atomicOr((unsigned*)(A.scal + kFlags), bad);
  if (threadIdx.x == 0) {
    *A.t_out = t;
    if (mlast >= 0.0) A.blkmax_out[0] = mlast;  // the maximum of the state left in U
  }
}

template <typename ST, int FORM>
static hipError_t launch_steps1d_halo(const StageArgs& a1, const StageArgs& a2, int nsteps, hipStream_t s) {
  const int nw = (a1.geo.nx + kTile1 - 1) / kTile1;
  const size_t lds = (size_t)(2 * 3 * a1.geo.nx + 2 * nw) * sizeof(double);  // at most 43 KiB
  StageArgs a = a1;
  a.uout = a2.uout;
  hipLaunchKernelGGL((steps1d_halo_kernel<ST, FORM>), dim3(1), dim3((unsigned)(64 * nw)), lds, s, a, nsteps);
  return hipGetLastError();
}

template <typename ST, int FORM>
static hipError_t launch_steps1d_k(const StageArgs& a1, const StageArgs& a2, int nsteps, hipStream_t s) {
  const Geometry& G = a1.geo;
  if (G.nx <= kMaxHalo1) return launch_steps1d_halo<ST, FORM>(a1, a2, nsteps, s);
  auto kern = steps1d_kernel<ST, FORM>;
  static int lds_set[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if ((int)G.lds_bytes > lds_set[dev]) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)G.lds_bytes);
    if (e != hipSuccess) return e;
    lds_set[dev] = (int)G.lds_bytes;
  }
  hipLaunchKernelGGL(kern, dim3(1), dim3((unsigned)G.threads), G.lds_bytes, s, a1, a2, nsteps);
  return hipGetLastError();
}

template <typename ST, int X>
static hipError_t launch_steps1d_x(const StageArgs& a1, const StageArgs& a2, int n, hipStream_t s) {
  switch (a1.form) {
    case kEuler: return launch_steps1d_k<ST, kEuler | X>(a1, a2, n, s);
    case kPVS: return launch_steps1d_k<ST, kPVS | X>(a1, a2, n, s);
    case kPMS: return launch_steps1d_k<ST, kPMS | X>(a1, a2, n, s);
    case kDVS: return launch_steps1d_k<ST, kDVS | X>(a1, a2, n, s);
    case kDMS: return launch_steps1d_k<ST, kDMS | X>(a1, a2, n, s);
    default: return launch_steps1d_k<ST, kPD | X>(a1, a2, n, s);
  }
}

template <typename ST>
hipError_t launch_steps1d(const StageArgs& a1, const StageArgs& a2, int nsteps, hipStream_t s) {
  if (a1.geo.ndim != 1 || a1.geo.nblk != 1) return hipErrorInvalidValue;
  if constexpr (sizeof(ST) == 8) {
    if (a1.eos) return launch_steps1d_x<ST, kExtVdw>(a1, a2, nsteps, s);
  }
  if (a1.eos) return hipErrorInvalidValue;
  return a1.inv_cmax2 > 0.0 ? launch_steps1d_x<ST, kExtCmax>(a1, a2, nsteps, s)
                            : launch_steps1d_x<ST, 0>(a1, a2, nsteps, s);
}

template hipError_t launch_steps1d<RSST_INST_ST>(const StageArgs&, const StageArgs&, int, hipStream_t);
#endif

}  // namespace rsstk
