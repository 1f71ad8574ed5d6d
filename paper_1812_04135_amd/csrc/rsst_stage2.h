// Device code of the RSST stages on 2D grids, shared by the per-grid 2D
// kernels and the batched persistent kernel.
//
// One wave works alone on a strip of 64 columns and marches y over a chunk
// of rows, one row per iteration.  The strip is either a whole periodic x row
// of at most 64 cells (the neighbours of its two ends wrap inside the strip)
// or fewer cells with halo lanes on each side, whose lanes hold the cells
// there (through the x boundary rule: a wall's ghost is the mirror cell with
// m_x negated) and repeat the face states the outer cells need: two lanes per
// side for one stage, four for the two stages of a step.  So within a stage
// nothing crosses waves and the march has no workgroup barrier: a wave's x
// neighbours and x plus-face states go through its own LDS slots, which a
// wave reads back in order without a barrier, and the flux at a cell's right
// face comes from the lane right of it by DPP.  y is marched: every y face
// is formed once and carried to the next row.
//
// What bounds it: FP64 issue (4 cycles per wave instruction on gfx950, 16
// for a reciprocal or square-root seed; 345 instructions per row and stage
// in FP64, 390 in FP32 storage: 0.7 us) and, on grids too small to fill the
// SIMDs, the latency of the chain through a row, 1.05 us for a wave alone on
// its SIMD.  Measured: 0.8 us per row where waves share a SIMD.  Whole rows
// per workgroup with three barriers each (rsst_row2.h) leave the SIMDs idle
// half of the time on large grids: 1024^2 FP64 62 us per step, 50 with strips.
#pragma once

#include "rsst_stage.h"

#pragma clang fp contract(off)

namespace rsstk {

constexpr int kWaves2 = 4;                 // waves (strips) per workgroup of a single stage
constexpr int kLds2 = 7 * 64;              // LDS doubles per wave: cell states, then x plus-face states
constexpr int kRed2 = kWaves2 * kLds2;     // per-workgroup reduction slots follow

// Strips of a 2D row for a given halo: one where a periodic row fits a wave,
// else strips of at most 64 - 2 halo cells, evenly filled.
__host__ __device__ inline Cols2 plan_cols2(int nx, bool x_per, int halo) {
  Cols2 c;
  if (x_per && nx <= 64) {
    c.ncol = 1;
    c.cw = nx;
    c.halo = 0;
  } else {
    const int w = 64 - 2 * halo;
    c.ncol = (nx + w - 1) / w;
    c.cw = (nx + c.ncol - 1) / c.ncol;
    c.halo = halo;
  }
  return c;
}

// Orders a wave's LDS writes before its later LDS reads of other lanes' slots
// (and the reverse): the hardware executes one wave's LDS accesses in order,
// so this only keeps the compiler from moving them.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Value held by lane l+1 (lane 63: lane 0's).
__device__ __forceinline__ double rotate_left(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x134, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x134, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// Reads the arguments that a 2D kernel needs first in one go: the compiler
// otherwise loads each where it is used, a chain of scalar-cache misses
// before the first state load.
__device__ __forceinline__ void fetch_args2(const StageArgs& A) {
  asm volatile("" ::"s"(A.geo.nx), "s"(A.geo.nm), "s"(A.geo.km), "s"(A.geo.rF), "s"(A.geo.cols.ncol), "s"(A.geo.cols.cw),
               "s"(A.geo.cols.halo), "s"(A.geo.colsF.ncol), "s"(A.geo.colsF.cw), "s"(A.geo.colsF.halo), "s"(A.geo.nblk), "s"(A.geo.nblkF),
               "s"(A.bc_lo[0]), "s"(A.bc_lo[1]), "s"(A.bc_hi[1]), "s"(A.ncell), "s"(A.uin), "s"(A.un), "s"(A.uout),
               "s"(A.blkmax), "s"(A.nslot), "s"(A.t_in), "s"(A.dt_fixed));
}

// A lane's place in strip `col`.
struct Lane2 {
  int i;           // its cell (through the x boundary rule)
  int so, sl, sr;  // LDS slots: its own, its left and its right neighbour's
  int sm;          // slot of the lane that owns its cell (itself but for a wall's ghost)
  int mxs;         // sign flip of m_x (a wall's ghost)
  bool own;        // the strip stores this cell
  bool pub;        // the lane's values are its cell's (a whole row's spare lanes end at the wrong neighbour)
};

__device__ __forceinline__ Lane2 lane_of(const Cols2& C, int nx, bool x_per, int col) {
  const int lane = threadIdx.x & 63;
  Lane2 L;
  bool mx = false;
  if (C.halo) {
    const int x0 = col * C.cw;
    const int q = min(x0 + lane - C.halo, nx + C.halo - 1);
    L.i = q;
    if (q < 0) {
      L.i = x_per ? q + nx : -1 - q;
      mx = !x_per;
    } else if (q >= nx) {
      L.i = x_per ? q - nx : 2 * nx - 1 - q;
      mx = !x_per;
    }
    L.so = lane;
    L.sl = max(lane - 1, 0);
    L.sr = min(lane + 1, 63);
    L.sm = mx ? min(max(L.i - x0 + C.halo, 0), 63) : lane;
    L.own = lane >= C.halo && lane < C.halo + min(C.cw, nx - x0);
    L.pub = true;
  } else {
    // lanes past the row repeat its first cells: the lane right of the last
    // cell then holds cell 0, whose left face is the last cell's right face
    L.i = lane % nx;
    L.so = L.sm = L.i;
    L.sl = L.i == 0 ? nx - 1 : L.i - 1;
    L.sr = L.i == nx - 1 ? 0 : L.i + 1;
    L.own = L.pub = lane < nx;
  }
  L.mxs = mx ? (int)0x80000000 : 0;
  return L;
}

// The stage values U1 of a tile in LDS: rows [k_lo, k_lo + nrow), each
// [value][64 slots].
struct Tile2 {
  double* u1;
  int k_lo, nrow;
};

// How a stage takes its input and leaves its output.
//   kSplit: input A.uin, output A.uout (one stage per launch);
//   kFused: stage 1 reads A.uin and leaves U1 in the tile (and in A.u1out, if
//     given); stage 2 reads the tile and A.un, and writes A.uout.
enum Mode2 { kSplit = 0, kFused = 1 };

// One stage of R over rows [k0, k1) of a strip, by one wave (lds: the wave's
// kLds2 doubles), returning the lane's largest c_tot of the stage-2 output
// (0 in stage 1) and or-ing non-physical flags into `bad`.  store: false for
// a wave without work, which runs one row and stores nothing.  Fused stage 1:
// rows are unwrapped indices, at most two outside [0, ny) and only across a
// periodic boundary; rows [own0, own1) go to A.u1out.
// dtf() gives the step's dt; it is called once, before the first row.  LDAUX: cache policy of the state loads.
template <int MODE, int STAGE, typename ST, int FORMX, int LDAUX = 0, typename DtFn>
__device__ __forceinline__ double march2(const StageArgs& A, const Lane2& L, double* lds, const Tile2& T, int k0,
                                         int k1, int own0, int own1, bool store, DtFn dtf, unsigned& bad) {
  constexpr int NDIM = 2, NV = 4;
  constexpr int FORM = FORMX & 7;
  constexpr int EXT = FORMX & (kExtCmax | kExtVdw);
  constexpr bool HYD = (FORMX & kExtHydro) != 0;
  constexpr bool F32 = sizeof(ST) == 4;
  constexpr int SZ = (int)sizeof(ST);
  constexpr bool IN_TILE = MODE == kFused && STAGE == 2;
  constexpr bool OUT_TILE = MODE == kFused && STAGE == 1;
  const Geometry& G = A.geo;
  const int nm = G.nm;
  const int rm_lo = A.bc_lo[1], rm_hi = A.bc_hi[1];
  const bool own = L.own && store;
  const int plane = G.nx * SZ;  // bytes per y row
  const int colb = L.i * SZ;
  double* const Uo = lds + L.so;
  double* const Ul = lds + L.sl;
  double* const Ur = lds + L.sr;

  const Consts K{A.gamma, A.gm1, A.inv_gm1, A.inv_xi, A.f, A.inv_cmax2, A.vdw_a, A.vdw_b};
  const double g[3] = {A.g[0], A.g[1], A.g[2]};
  const double hx = 0.5 * A.inv_dx[0], hy = 0.5 * A.inv_dx[1];
  const Field32 uin = make_field<false>(A.uin, A.ncell, NV, SZ, plane);
  const Field32 unp = make_field<false>(A.un ? A.un : A.uin, A.ncell, NV, SZ, plane);
  const Field32 uout = make_field<false>(OUT_TILE ? A.u1out : A.uout, A.ncell, NV, SZ, plane);

  // FP32 perturbation form: the background of a row (profile along y, kk its
  // mapped index) or of the lane's column (uniform, along x)
  const __amdgpu_buffer_rsrc_t bgr = field_rsrc(A.bg, F32 ? (long long)NV * A.nbg * 8 : 0);
  const int bg_fix = A.bg_axis == 0 ? L.i : 0;
  auto bg_row = [&](int kk, double (&b)[NV]) {
    if constexpr (F32) load_bg<NV>(bgr, A.nbg, A.bg_axis == 1 ? kk : bg_fix, b);
  };
  // a row to load: its mapped index, the sign of m_y there, the hydrostatic
  // lever of a wall's ghost, and (tile) its row in the tile
  struct Row {
    int kk;
    bool neg;
    double lev;
  };
  auto row_of = [&](int q) {
    Row r;
    r.kk = map_index(q, nm, rm_lo, rm_hi, r.neg);
    r.lev = HYD ? hydro_lever(q, nm, rm_lo, rm_hi, A.dx[1], A.g[1]) : 0.0;
    // the tile holds a wall's ghost rows nowhere (they mirror rows that it
    // holds) and a periodic neighbour's rows unwrapped
    if constexpr (IN_TILE) r.kk = min(max((r.neg ? r.kk : q) - T.k_lo, 0), T.nrow - 1);
    return r;
  };
  // the stored values of a row (tile: already FP64, background included)
  typedef typename std::conditional<IN_TILE, double, ST>::type RT;
  constexpr bool WIDEN = F32 && !IN_TILE;
  auto load_row = [&](const Row& r, RT (&raw)[NV], double (&bz)[NV]) {
    if constexpr (IN_TILE) {
      const double* t = T.u1 + r.kk * (NV * 64) + L.sm;
#pragma unroll
      for (int v = 0; v < NV; ++v) raw[v] = t[v * 64];
    } else {
      load_cell_raw<NDIM, ST, LDAUX>(uin, r.kk, colb, raw);
      if constexpr (WIDEN) bg_row(r.kk, bz);
    }
  };
  auto fin = [&](const RT (&raw)[NV], const Row& r, const double (&bz)[NV], double (&u)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = (double)raw[v];
    if constexpr (WIDEN) {
#pragma unroll
      for (int v = 0; v < NV; ++v) u[v] += bz[v];
    }
    u[1] = __hiloint2double(__double2hiint(u[1]) ^ L.mxs, __double2loint(u[1]));
    u[2] = __hiloint2double(__double2hiint(u[2]) ^ (r.neg ? (int)0x80000000 : 0), __double2loint(u[2]));
    if constexpr (HYD) {
      if (r.lev != 0.0) {
        const double dedp = A.eos ? (1.0 - A.vdw_b * u[0]) * A.inv_gm1 : A.inv_gm1;
        u[NDIM + 1] = u[NDIM + 1] + u[0] * r.lev * dedp;
      }
    }
  };

  // the march window: rows k, k + 1, k + 2 (finished), the slope at k and
  // the flux at k - 1/2
  double q0[NV], q1[NV], q2[NV], sm0[NV], Fm_lo[NV];
  double cmax = 0.0;
  {
    RT ra[5][NV];
    double bz[5][NV];
    Row rw[5];
#pragma unroll
    for (int p = 0; p < 5; ++p) {
      rw[p] = row_of(k0 - 2 + p);
      load_row(rw[p], ra[p], bz[p]);
    }
    double qa[NV], qb[NV], ha[NV];
    fin(ra[0], rw[0], bz[0], qa);
    fin(ra[1], rw[1], bz[1], qb);
    fin(ra[2], rw[2], bz[2], q0);
    fin(ra[3], rw[3], bz[3], q1);
    fin(ra[4], rw[4], bz[4], q2);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      ha[v] = mc_half(qb[v] - qa[v], q0[v] - qb[v]);
      sm0[v] = mc_half(q0[v] - qb[v], q1[v] - q0[v]);
    }
    Face<NV> fl, fr;
    make_face<NDIM, 1, EXT>(qb, ha, true, K, fl);
    make_face<NDIM, 1, EXT>(q0, sm0, false, K, fr);
    flux2<NDIM, 1>(fl, fr, Fm_lo);
  }

  const double dt = dtf();
  // both stages in one launch: two waves share a SIMD and wait for each other
  // between the stages, so the one with fewer rows left yields (wave_prio;
  // 512^2 19.3 to 18.8 us per step; nothing to gain below three rows)
  const int kp = k1 - k0 > 2 ? k1 - 4 : k1;
  for (int k = k0; k < k1; ++k) {
    if (MODE == kFused && k >= kp) wave_prio(k1 - 1 - k);
    // loads: the row three ahead (the window's row k + 2 of the next
    // iteration) and the step-start state
    RT rn[NV];
    ST unr[NV];
    double bn[NV], bc[NV];
    const Row r3 = row_of(min(k + 3, nm + (MODE == kFused ? 3 : 1)));
    load_row(r3, rn, bn);
    const int kc = OUT_TILE ? row_of(k).kk : k;  // the row's own index
    if constexpr (STAGE == 2) load_cell_raw<NDIM, ST, LDAUX>(unp, k, colb, unr);
    bg_row(kc, bc);

    // publish the cell state
#pragma unroll
    for (int v = 0; v < NV; ++v) Uo[v * 64] = q0[v];
    wave_lds_fence();
    double ul[NV], ur[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      ul[v] = Ul[v * 64];
      ur[v] = Ur[v * 64];
    }

    // y: the slope at k + 1 and the flux at k + 1/2
    double Dl[NV], sm1[NV], Fm_hi[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) sm1[v] = mc_half(q1[v] - q0[v], q2[v] - q1[v]);
    {
      Face<NV> fl, fr;
      make_face<NDIM, 1, EXT>(q0, sm0, true, K, fl);
      make_face<NDIM, 1, EXT>(q1, sm1, false, K, fr);
      flux2<NDIM, 1>(fl, fr, Fm_hi);
    }
    // (y first: it covers the LDS reads, which the scheduler would otherwise
    // wait for at once)
    __builtin_amdgcn_sched_barrier(0);

    // x: the plus-face state (published over the cell states, which every
    // lane has read), the flux at the left face, and the right neighbour's
    // for the right face
    double h[NV], Fx_lo[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) h[v] = mc_half(q0[v] - ul[v], ur[v] - q0[v]);
    {
      Face<NV> fp, fm, pl;
      make_face<NDIM, 0, EXT>(q0, h, true, K, fp);
      wave_lds_fence();
      put_face(Uo, 64, fp);
      make_face<NDIM, 0, EXT>(q0, h, false, K, fm);
      wave_lds_fence();
      get_face(Ul, 64, pl);
      flux2<NDIM, 0>(pl, fm, Fx_lo);
    }
    wave_lds_fence();
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double Fx_hi = rotate_left(Fx_lo[v]);
      Dl[v] = -(Fx_hi - Fx_lo[v]) * hx;
      Dl[v] = fma(-(Fm_hi[v] - Fm_lo[v]), hy, Dl[v]);
      Fm_lo[v] = Fm_hi[v];
      sm0[v] = sm1[v];
    }

    // the rate, the RK update and the store
    double Rt[NV];
    const unsigned b = rsst_rate<NDIM, FORM, EXT>(q0, Dl, K, g, Rt);
    ST st[NV];
    double out[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double y = fma(dt, Rt[v], q0[v]);
      if constexpr (STAGE == 2) {
        double un = (double)unr[v];
        if constexpr (F32) un += bc[v];
        y = 0.5 * (un + y);
      }
      if constexpr (F32) {
        st[v] = (ST)(y - bc[v]);
        out[v] = (double)st[v] + bc[v];
      } else {
        st[v] = (ST)y;
        out[v] = y;
      }
    }
    if constexpr (OUT_TILE) {
      if (store && L.pub) {
        double* t = T.u1 + (k - T.k_lo) * (NV * 64) + L.so;
#pragma unroll
        for (int v = 0; v < NV; ++v) t[v * 64] = out[v];
      }
    }
    if (own && (!OUT_TILE || (k >= own0 && k < own1))) {
      bad |= b;
      if (!OUT_TILE || A.u1out) {
#pragma unroll
        for (int v = 0; v < NV; ++v) buf_store<ST>(uout.r, colb, uout.soff(v, k), st[v]);
      }
      if constexpr (STAGE == 2) cmax = fmax(cmax, cell_ctot<NDIM, EXT>(out, K));
    }
    // the window moves one row
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      q0[v] = q1[v];
      q1[v] = q2[v];
    }
    fin(rn, r3, bn, q2);
  }
  return cmax;
}

// ---- both stages of a step in one launch --------------------------------
//
// A workgroup of eight waves takes one strip and a tile of 4 r rows.  Stage
// 1: the waves march the 4 (r + 1) rows of U1 that these need, into LDS; a
// barrier; stage 2: they march the tile's rows.  Waves w and w + 4 share a
// SIMD, and each SIMD gets r + 1 and r rows.  U1 never goes to memory, unless
// the caller keeps it.
constexpr int kWavesF = 8;
__host__ __device__ constexpr int lds_doublesF(int r) { return kWavesF * kLds2 + 4 * (r + 1) * 4 * 64 + kWavesF; }
constexpr int kMaxRF = 15;  // 156 KB of LDS

// The rows [a, b) of wave w when every SIMD gets n rows.
__device__ __forceinline__ void wave_rows(int w, int n, int& a, int& b) {
  const int hi = (n + 1) >> 1, lo = n >> 1;
  a = w < 4 ? w * hi : 4 * hi + (w - 4) * lo;
  b = a + (w < 4 ? hi : lo);
}

template <typename ST, int FORMX, typename DtFn>
__device__ __forceinline__ double step_tile2(const StageArgs& A, double* lds, int tile, DtFn dtf, unsigned& bad) {
  const Geometry& G = A.geo;
  const Cols2& C = G.colsF;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int R = 4 * G.rF;
  const int col = tile % C.ncol;
  const int kb = (tile / C.ncol) * R, ke = min(kb + R, G.nm);
  double* const mine = lds + w * kLds2;
  const Tile2 T{lds + kWavesF * kLds2, kb - 2, R + 4};
  const Lane2 L = lane_of(C, G.nx, A.bc_lo[0] == 0, col);
  double dt = 0.0;
  {
    const int lo = A.bc_lo[1] ? 0 : -2, hi = A.bc_hi[1] ? G.nm : G.nm + 2;
    int k0, k1;
    wave_rows(w, G.rF + 1, k0, k1);
    k0 = max(kb - 2 + k0, lo);
    k1 = min(min(kb - 2 + k1, ke + 2), hi);
    const bool work = k0 < k1;
    if (!work) {
      k0 = kb;
      k1 = kb + 1;
    }
    march2<kFused, 1, ST, FORMX>(A, L, mine, T, k0, k1, kb, ke, work, [&]() { return dt = dtf(); }, bad);
  }
  __syncthreads();
  int k0, k1;
  wave_rows(w, G.rF, k0, k1);
  k0 += kb;
  k1 = min(k1 + kb, ke);
  double cmax = 0.0;
  if (k0 < k1)
    cmax = march2<kFused, 2, ST, FORMX>(A, L, mine, T, k0, k1, kb, ke, true, [&]() { return dt; }, bad);
  return cmax;
}

}  // namespace rsstk
