// Device code of one RSST stage over whole 2D rows, for the single-stage
// launches whose rows fill their waves better than strips with halo lanes do
// (rsst_stage2.h; plan_geometry says which).
//
// A workgroup holds an x row of nx cells (nwx waves) and marches y over its
// chunk of rows, one per iteration.  x neighbours and x plus-face states are
// exchanged through LDS rows with one ghost slot at each end (periodic wrap or
// mirror), and every x face flux is formed once, by the cell right of the face, and
// handed to the cell on its left after a third barrier (by DPP within a wave,
// one LDS seam value per wave edge).
// y is marched: every y face is formed once and carried to the next row.
//
// Two rows per iteration (half the barriers, twice the independent work per
// thread, but 160 VGPRs and so three waves per SIMD instead of four) were no
// faster than one with chunks of as many rows: us per step, two and one, 512 x
// 500 FP64 19.9, 19.3, FP32 19.5, 19.3; 256 x 1000 19.5, 19.4 and 19.1, 19.5;
// 128 x 4000 31.0, 30.7 and 30.9, 31.7.
#pragma once

#include "rsst_stage.h"

#pragma clang fp contract(off)

namespace rsstk {

// LDS carve-up of a 2D workgroup (doubles): a row of nwx waves.
struct Carve2 {
  int u, fp, fxs, red, total;
};

__host__ __device__ inline Carve2 carve2(int nwx) {
  constexpr int NV = 4, PL = NV + 3;
  const int px = 64 * nwx + 2;
  Carve2 c;
  int o = 0;
  c.u = o;   o += NV * px;   // cell states [value][slot], slot 1 + i; 0, nx + 1: ghosts
  c.fp = o;  o += PL * px;  // x plus-face states, slot 1 + i; slot 0: the left ghost's
  c.fxs = o; o += NV * nwx;  // x flux at the left edge of each wave
  c.red = o; o += 16;
  c.total = o;
  return c;
}

// One stage of R over a chunk of rows, returning the thread's largest c_tot of
// the stage-2 output (0 in stage 1) and or-ing non-physical flags into `bad`.
// dtf() gives the step's dt; it is called once, after the first rows are loaded.
template <int STAGE, typename ST, int FORMX, typename DtFn>
__device__ __forceinline__ double stage_body2(const StageArgs& A, double* lds, int chunk, DtFn dtf,
                                              unsigned& bad) {
  constexpr int NDIM = 2, NV = 4, PL = NV + 3;
  constexpr int FORM = FORMX & 7;
  constexpr int EXT = FORMX & (kExtCmax | kExtVdw);
  constexpr bool HYD = (FORMX & kExtHydro) != 0;
  constexpr bool F32 = sizeof(ST) == 4;
  constexpr int SZ = (int)sizeof(ST);
  const Geometry& G = A.geo;
  const int nwx = G.nwx;
  const int PX = 64 * nwx + 2;
  const Carve2 C = carve2(nwx);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wx = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i_raw = tid;
  const bool xin = i_raw < G.nx;
  const int i = xin ? i_raw : G.nx - 1;
  const int k0 = chunk * G.km, k1 = min(k0 + G.km, G.nm);
  const bool last_x = i_raw == G.nx - 1;
  const bool first_x = i_raw == 0;
  const bool x_per = A.bc_lo[0] == 0;
  const int rm_lo = A.bc_lo[1], rm_hi = A.bc_hi[1];
  const int plane = G.nx * SZ;  // bytes per y row
  const int col = i * SZ;

  // the thread's LDS addresses: its cell slot minus one (its left neighbour),
  // its plus-face slot minus one, and its wave's x seam
  double* const Urow = lds + C.u;
  double* const Frow = lds + C.fp;
  double* const ub = Urow + i;            // + v PX + {0, 1, 2}
  double* const fb = Frow + i;            // + q PX + {0, 1}
  double* const xs = lds + C.fxs + wx;    // + v nwx

  // FP32 perturbation form: the background in registers, along y (the march
  // axis: bgc for row k of the iteration, bgn for the row the iteration loads,
  // k + 2) or fixed for the march (uniform, along x: bgc)
  const bool bg_on_m = F32 && A.bg_axis == 1;
  double bgc[NV], bgn[NV];
  const __amdgpu_buffer_rsrc_t bgr = field_rsrc(A.bg, F32 ? (long long)NV * A.nbg * 8 : 0);
  if constexpr (F32) {
    if (!bg_on_m) load_bg<NV>(bgr, A.nbg, A.bg_axis == 0 ? i : 0, bgc);
  }
  // FP64 state of stored values: FP32 with the background bz; FP64 with the
  // mirror sign and a hydrostatic wall's carried pressure (lever)
  auto fin = [&](const ST (&raw)[NV], int neg, const double (&bz)[NV], double lev, double (&u)[NV]) {
    if constexpr (F32) finish_cell_bgv<NDIM, ST>(raw, neg, bz, u);
    else finish_cell<NDIM, ST>(A, raw, neg, 0, u, lev);
  };

  const Consts K{A.gamma, A.gm1, A.inv_gm1, A.inv_xi, A.f, A.inv_cmax2, A.vdw_a, A.vdw_b};
  const double g[3] = {A.g[0], A.g[1], A.g[2]};
  const double hx = 0.5 * A.inv_dx[0], hy = 0.5 * A.inv_dx[1];
  const Field32 uin = make_field<false>(A.uin, A.ncell, NV, SZ, plane);
  const Field32 unp = make_field<false>(A.un ? A.un : A.uin, A.ncell, NV, SZ, plane);
  // stage 2 writes the new state in place over the step-start state
  const Field32 uout = make_field<false>(A.uout, A.ncell, NV, SZ, plane);

  // the march window: rows k and k + 1 (finished), the slope at k and the
  // flux at k - 1/2
  double q0[NV], q1[NV], sm0[NV], Fm_lo[NV];
  double cmax = 0.0;
  // (k0 is in range anyway; that the compiler is told so here is worth 3%: 256 x
  // 256 10.6 us per step without, 10.3 with)
  const int k0l = min(k0, G.nm - 1);
  {
    double qa[NV], qb[NV], ha[NV];
    auto ld = [&](int q, double (&u)[NV]) {  // row k0 + q of the thread's column, through the y walls
      bool n;
      const int kk = map_index(k0l + q, G.nm, rm_lo, rm_hi, n);
      ST raw[NV];
      load_cell_raw<NDIM, ST>(uin, kk, col, raw);
      double bz[NV];
      if constexpr (F32) {
        if (bg_on_m) load_bg<NV>(bgr, A.nbg, kk, bz);
        else {
#pragma unroll
          for (int v = 0; v < NV; ++v) bz[v] = bgc[v];
        }
      }
      fin(raw, n ? NDIM : -1, bz, HYD ? hydro_lever(k0l + q, G.nm, rm_lo, rm_hi, A.dx[1], A.g[1]) : 0.0, u);
    };
    ld(-2, qa);
    ld(-1, qb);
    ld(0, q0);
    ld(1, q1);
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

  for (int k = k0; k < k1; ++k) {
    // ---- loads for this iteration: the row two ahead and the step-start
    // state (stored values now, finished where first used)
    ST wr[NV], unr[NV];
    bool wn;
    const int kk = map_index(k + 2, G.nm, rm_lo, rm_hi, wn);
    const double wlev = HYD ? hydro_lever(k + 2, G.nm, rm_lo, rm_hi, A.dx[1], A.g[1]) : 0.0;
    if constexpr (F32) {
      if (bg_on_m) {
        load_bg<NV>(bgr, A.nbg, k, bgc);
        load_bg<NV>(bgr, A.nbg, kk, bgn);
      }
    }
    load_cell_raw<NDIM, ST>(uin, kk, col, wr);
    if constexpr (STAGE == 2) load_cell_raw<NDIM, ST>(unp, k, col, unr);

    // ---- P1: publish the cell states, and the x ghosts
    if (xin) {
#pragma unroll
      for (int v = 0; v < NV; ++v) ub[v * PX + 1] = q0[v];
    }
    if (first_x || last_x) {
      // cell 0: periodic, the ghost right of the last cell; wall, the mirror
      // left of cell 0.  The last cell: periodic, the ghost left of cell 0;
      // wall, the mirror right of the last cell.
      double* ur = Urow + (first_x == x_per ? G.nx + 1 : 0);
#pragma unroll
      for (int v = 0; v < NV; ++v) ur[v * PX] = (v == 1 && !x_per) ? -q0[v] : q0[v];
    }
    __syncthreads();  // B1

    // (the reads of the neighbours' slots form their addresses anew: kept over
    // the march they put half of the forms beyond 128 VGPRs, three waves per SIMD)
    int pitch = PX;
    asm volatile("" : "+s"(pitch));

    // ---- P2: the x slopes and the plus-face states (published)
    double h[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) h[v] = mc_half(q0[v] - ub[v * pitch], ub[v * pitch + 2] - q0[v]);
    {
      Face<NV> fp;
      make_face<NDIM, 0, EXT>(q0, h, true, K, fp);
      if (xin) put_face(fb + 1, PX, fp);
      if (x_per && last_x) put_face(Frow, PX, fp);  // the periodic ghost left of cell 0
    }
    __syncthreads();  // B2

    // ---- P3: the x flux at each cell's left face, published at wave edges
    double Fx_lo[NV];
    {
      Face<NV> fm, pl;
      make_face<NDIM, 0, EXT>(q0, h, false, K, fm);
      get_face(fb, pitch, pl);  // slot i: the plus face of cell i - 1
      if (!x_per) {
        if (first_x) pl = mirror<NDIM, 0>(fm);
      }
      flux2<NDIM, 0>(pl, fm, Fx_lo);
      if (lane == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) xs[v * nwx] = Fx_lo[v];
      }
    }
    __syncthreads();  // B3

    // ---- P4: the flux at each cell's right face, the y direction, then the
    // rate, the RK update and the store
    double Dl[NV];
    {
      double Fx_hi[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) Fx_hi[v] = from_right(Fx_lo[v]);
      if (last_x) {
        if (x_per) {
#pragma unroll
          for (int v = 0; v < NV; ++v) Fx_hi[v] = xs[v * nwx - wx];
        } else {
          Face<NV> fp;
          get_face(fb + 1, PX, fp);
          flux2<NDIM, 0>(fp, mirror<NDIM, 0>(fp), Fx_hi);
        }
      } else if (lane == 63 && xin) {
#pragma unroll
        for (int v = 0; v < NV; ++v) Fx_hi[v] = xs[v * nwx + 1];
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) Dl[v] = -(Fx_hi[v] - Fx_lo[v]) * hx;
    }
    // the row two ahead, finished; the slope at k + 1 and the flux at k + 1/2
    double q2[NV];
    if (F32 && bg_on_m) fin(wr, wn ? NDIM : -1, bgn, 0.0, q2);
    else fin(wr, wn ? NDIM : -1, bgc, wlev, q2);
    double sm1[NV], Fm_hi[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) sm1[v] = mc_half(q1[v] - q0[v], q2[v] - q1[v]);
    {
      Face<NV> fl, fr;
      make_face<NDIM, 1, EXT>(q0, sm0, true, K, fl);
      make_face<NDIM, 1, EXT>(q1, sm1, false, K, fr);
      flux2<NDIM, 1>(fl, fr, Fm_hi);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      Dl[v] = fma(-(Fm_hi[v] - Fm_lo[v]), hy, Dl[v]);
      Fm_lo[v] = Fm_hi[v];
      sm0[v] = sm1[v];
    }
    double Rt[NV];
    const unsigned b = rsst_rate<NDIM, FORM, EXT>(q0, Dl, K, g, Rt);
    double un[NV];
    if constexpr (STAGE == 2) fin(unr, -1, bgc, 0.0, un);
    if (xin) {
      bad |= b;
      double out[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        double y = fma(dt, Rt[v], q0[v]);
        if constexpr (STAGE == 2) y = 0.5 * (un[v] + y);
        double bgv = 0.0;
        if constexpr (F32) bgv = bgc[v];
        const ST st = (ST)(y - bgv);
        buf_store<ST>(uout.r, col, uout.soff(v, k), st);
        out[v] = (double)st + bgv;
      }
      if constexpr (STAGE == 2) cmax = fmax(cmax, cell_ctot<NDIM, EXT>(out, K));
    }
    // the window moves one row
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      q0[v] = q1[v];
      q1[v] = q2[v];
    }
  }
  return cmax;
}

}  // namespace rsstk
