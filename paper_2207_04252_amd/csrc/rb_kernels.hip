// Device kernels of the bi-fluid finite-volume library for gfx950 (MI355X).
//
// One RK2 stage is one launch per group of fields (k_gas, and k_dust for each species): a
// workgroup owns a 64 (theta) x 8 (r) tile of cells and marches through a chunk of z planes.
// Each z plane of the tile, with a two-cell halo, is staged in LDS; every thread solves the
// Riemann problems at the upper theta and r faces of its own cell (the tile's lower-edge
// faces are solved by the first 72 threads), exchanges the fluxes through LDS, and keeps its
// column of the z direction to itself.  Fluxes, divergence, sources, drag and the update are
// fused: the state is read once per stage (plus the L2-resident halo) and written once.
#include "rb_device.h"

namespace rb {

// ------------------------------------------------------------------------------------
// the gas stage kernel (FP64).  The groups of fields interact only through the cell-local drag,
// which each kernel evaluates from the other group's centre state of the same stage input.
//
// Bound by the issue of FP64 instructions (four cycles each) and the latency of the face
// solves, at two waves per SIMD (256 VGPRs); 1690 -> 1290 lane-instructions per cell by the
// faces' short form (gas_face64) with the general form behind one inlined copy per plane.
// LDS holds two planes (160760 of the CU's 163840 bytes, which two waves per SIMD leave free):
// one barrier per plane, so that a wavefront that ends its faces early goes on with
// the update, and what the update needs per row is read there in batches (as scalar loads
// each value waited for its own).  The older wave of a SIMD is served first, so the younger
// ones end a plane: the first two wavefronts, which solve the tile's edge faces, and the
// first one's partner take no halo cells.  Gas disc 128 x 256 x 64: 235 -> 157 us per
// launch (two barriers and scalar loads 194); bi-fluid disc 256 x 512 x 64, 800 -> 600; 50
// steps of the 2D disc 3.32 -> 2.18 ms.

template <int ND, bool G75, bool EXT>
__global__ void __launch_bounds__(NTM, 2) k_gas(StageArgs a) {
  __shared__ int s_stop;
  if (threadIdx.x == 0) s_stop = __atomic_load_n(&a.c.ctrl->status, __ATOMIC_RELAXED);
  __syncthreads();
  if (s_stop & FL_HARD) return;
  constexpr int NG = 5, HW = TJ + 4, NHALO = 4 * HW + 4 * TM;
  static_assert(NHALO <= NTM - 3 * 64, "one halo cell per thread");
  // plane k's W' in the half k & 1; its r faces and the theta faces at the tile's lower edge
  // likewise (read by the update behind the next barrier); the own theta faces
  __shared__ double s_pl[2][NG][TM + 4][HW];
  __shared__ double s_fr[2][NG][TM + 1][TJ];
  __shared__ double s_fe[2][NG][TM];
  // (s_ft in one copy: its readers are its writer's wavefront, ordered by wave_order)
  __shared__ double s_ft[NG][NTM];
  __shared__ double s_rm[NG][NTM];
  __shared__ double s_red[NTM / 64][3];
  // Newton counts of the faces the wavefront owns (bins 0..7, 7: seven or more)
  __shared__ int s_nh[NTM / 64][8];
  __shared__ GasCount s_cnt;
  // per-plane tables: the stationary velocity, pressure and density (NF) at the rows'
  // centres, r faces and upper z faces; density and velocity at the centres of the rows and
  // their halo, two planes ahead; the update's conservative state, gravity and residual
  constexpr int NF = 3, NFACE = (3 * TM + 1) * NF, NCEN = (TM + 4) * 2, NU = 12, NUPD = TM * NU;
  constexpr int T_CEN = NFACE, T_UPD = T_CEN + NCEN, NTAB = T_UPD + NUPD;
  static_assert(NTAB <= NTM, "one table entry per thread");
  __shared__ double s_face[4][NFACE];
  __shared__ double s_cen[4][NCEN];
  __shared__ double s_upd[4][NUPD];
  // per row, the same in every plane: parabola weights of the cells on both sides of the r
  // face below it (first entry: of the tile's lower edge), geometry of the update
  __shared__ double s_wt[TM + 1][8];
  enum { RW_AR0 = 0, RW_AR1, RW_ATH, RW_AZ, RW_V, RW_INVV, RW_INVRC, RW_OMK, RW_N };
  __shared__ double s_row[TM][RW_N];

  const Geo& g = a.g;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int tjb = tile % a.ntj;
  const int tib = (tile / a.ntj) % a.ntm;
  const int kcb = tile / (a.ntj * a.ntm);
  const int tid = threadIdx.x, tj = tid & (TJ - 1);
  const int ti = __builtin_amdgcn_readfirstlane(tid / TJ);
  const int j0 = tjb * TJ, i0 = tib * TM;
  const int k0 = kcb * a.tk, k1 = min(g.nz, k0 + a.tk);
  const int jg = j0 + tj;
  const int ig = i0 + ti, igc = min(ig, g.nr - 1);
  const bool act = jg < g.nth && ig < g.nr;
  const bool drag = !a.gas_only && ND > 0 && !g.drag_exact;
  const bool twod = g.twod != 0;
  const size_t plane = (size_t)g.nr * g.nth;
  const GasC gc = gas_consts(g.gamma, g.newton_max);
  const RecC recc;
  const unsigned jl = (unsigned)(jg % g.nth);  // (past the grid: as k_dust)
  const size_t row0 = (size_t)igc * g.nth;
  const ctab rt = to_ctab(a.t.rt) + (size_t)igc * RT_N, ar = to_ctab(a.t.ar);
  if (tid < (TM + 1) * 8) {
    const int r = tid / 8, e = tid % 8, i = min(i0 + r - 1 + (e < 4 ? 0 : 1), g.nr);
    // (RC_WPM .. RC_LPP of the lower cell, RC_WMM .. RC_LMP of the upper)
    s_wt[r][e] = a.t.rco[(size_t)(i + 1) * RC_N + e];
  } else if (tid >= 128 && tid < 128 + TM * RW_N) {
    const int r = (tid - 128) / RW_N, e = (tid - 128) % RW_N, i = min(i0 + r, g.nr - 1);
    const double* q = a.t.rt + (size_t)i * RT_N;
    s_row[r][e] = e == RW_AR0   ? a.t.ar[i]
                  : e == RW_AR1 ? a.t.ar[i + 1]
                  : e == RW_ATH ? q[RT_ATH]
                  : e == RW_AZ  ? q[RT_AZ]
                  : e == RW_V   ? q[RT_V]
                  : e == RW_INVV ? q[RT_INVV]
                  : e == RW_INVRC ? q[RT_INVRC]
                                  : q[RT_OMK];
  } else if (tid >= 256 && tid < 256 + NTM / 64 * 8) {
    s_nh[(tid - 256) / 8][tid & 7] = 0;
  }
  if (tid == 0) s_cnt = GasCount{0, 0, 0, 0};
  int maxit = 0;
  auto tally = [&](bool own, int last) {
    const int b = min(last, 7);
    unsigned long long left = __ballot(own);
    while (left) {
      const int at = __builtin_ctzll(left), v = __builtin_amdgcn_readlane(b, at);
      const unsigned long long mk = __ballot(own && b == v);
      if (tj == at) atomicAdd(&s_nh[ti][v], __popcll(mk));
      left &= ~mk;
    }
  };

  // thread NTM - 1 - t stages table entry t: tab_p + plane * tab_stride (the tile's edge faces
  // are the first wavefronts')
  const int tt = NTM - 1 - tid;
  const double* tab_p = nullptr;
  size_t tab_stride = 0;
  if (tt < NTAB) {
    const size_t nr = (size_t)g.nr;
    // (entry e of a face: velocity, pressure, density)
    if (tt < NFACE) {
      const int r = tt / NF, e = tt % NF == 0 ? WB_V : WB_W + tt % NF;
      if (r < TM) {
        tab_p = a.t.wc + (size_t)min(i0 + r, g.nr - 1) * WB_N + e;
        tab_stride = nr * WB_N;
      } else if (r < 2 * TM + 1) {
        tab_p = a.t.wr + (size_t)min(i0 + r - TM, g.nr) * WB_N + e;
        tab_stride = (nr + 1) * WB_N;
      } else {
        tab_p = a.t.wz + (nr + (size_t)min(i0 + r - 2 * TM - 1, g.nr - 1)) * WB_N + e;
        tab_stride = nr * WB_N;
      }
    } else if (tt < T_UPD) {
      const int r = (tt - T_CEN) / 2, e = (tt - T_CEN) % 2 ? WB_V : WB_RHO;
      tab_p = a.t.wc + (size_t)min(max(i0 + r - 2, 0), g.nr - 1) * WB_N + e;
      tab_stride = nr * WB_N;
    } else {
      const int r = (tt - T_UPD) / NU, e = (tt - T_UPD) % NU;
      const size_t i = min(i0 + r, g.nr - 1);
      if (e < 5) { tab_p = a.t.bgc + i * 5 + e; tab_stride = nr * 5; }
      else if (e < 7) { tab_p = a.t.grav + i * 2 + (e - 5); tab_stride = nr * 2; }
      else { tab_p = a.t.r0 + i * 5 + (e - 7); tab_stride = nr * 5; }
    }
  }
  const bool cen_t = tt >= T_CEN && tt < T_UPD;
  auto tab_load = [&](int k) {  // (the centres' entries: of plane k + 2)
    return tt < NTAB ? tab_p[(size_t)min(cen_t ? k + 2 : k, g.nz - 1) * tab_stride] : 0.0;
  };
  auto tab_store = [&](int k, double x) {
    if (tt < NFACE) s_face[k & 3][tt] = x;
    else if (tt < T_UPD) s_cen[(k + 2) & 3][tt - T_CEN] = x;
    else if (tt < NTAB) s_upd[k & 3][tt - T_UPD] = x;
  };

  const double* vin = (const double*)a.in;
  struct Raw { double e[NG]; };
  auto col_fetch = [&](const double* v, int k, Raw& R) {
    const size_t r = (size_t)min(max(k, 0), g.nz - 1) * plane + row0;
#pragma unroll
    for (int f = 0; f < NG; ++f) R.e[f] = at_row(v + (size_t)f * g.N + r, jl);
  };
  // W' of a cell with stationary density and azimuthal velocity c (no other velocity)
  const double gm1 = g.gamma - 1.0;
  auto form = [&](const double* e, const double* c, double* out) {
    const double b[WB_N] = {0.0, c[1], 0.0, 0.0, c[0], 0.0, 0.0, 0.0};
    cell_w(e, b, gm1, out);
  };
  // W' of the thread's cell of plane k, or of the ghost in its place
  auto col_form = [&](int k, const Raw& R, const double* c, double* out) {
    if (EXT && g.bc_z == 1 && (k < 0 || k >= g.nz)) {
      const size_t e = (size_t)((k < 0 ? 0 : 2) + min(k < 0 ? -1 - k : k - g.nz, 1)) * g.nr + igc;
      double s[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) s[f] = R.e[f] * a.t.ozr[e];
      cell_w(s, a.t.ghzw + e * WB_N, gm1, out);
    } else if (k < 0 || k >= g.nz) {
      const size_t l = (k < 0 ? 0 : 2) + min(k < 0 ? -1 - k : k - g.nz, 1);
      const ctab gt = to_ctab(a.t.ghz) + (l * g.nr + igc) * g.nf;
#pragma unroll
      for (int f = 0; f < NG; ++f) out[f] = gt[f];
    } else if (ig >= g.nr) {
      const ctab gt = to_ctab(a.t.ghr) + ((size_t)(2 + min(ig - g.nr, 1)) * g.nz + k) * g.nf;
#pragma unroll
      for (int f = 0; f < NG; ++f) out[f] = gt[f];
    } else {
      form(R.e, c, out);
    }
  };
  auto cen = [&](int k, int row) { return &s_cen[k & 3][row * 2]; };
  // (not by the first two wavefronts, which solve the tile's edge faces, nor by the fifth, on
  // the first one's SIMD)
  const int th = ti < 2 || ti == 4 ? -1 : tid - (ti < 4 ? 2 : 3) * 64;
  const bool halo_t = th >= 0 && th < NHALO;
  int h_rr = 0, h_cc = 0;
  if (!halo_t) {}
  else if (th < 2 * HW) { h_rr = th / HW; h_cc = th % HW; }
  else if (th < 4 * HW) { h_rr = TM + 2 + (th - 2 * HW) / HW; h_cc = (th - 2 * HW) % HW; }
  else if (halo_t) { const int e = th - 4 * HW; h_rr = 2 + e / 4; h_cc = (e & 3) < 2 ? (e & 3) : TJ + (e & 3); }
  const int h_ii = i0 + h_rr - 2;
  const size_t h_off = (size_t)min(max(h_ii, 0), g.nr - 1) * g.nth + (j0 + h_cc - 2 + g.nth) % g.nth;
  auto halo_fetch = [&](int k, Raw& R) {
#pragma unroll
    for (int f = 0; f < NG; ++f) R.e[f] = at_plane(vin + (size_t)f * g.N + (size_t)k * plane, h_off);
  };
  auto halo_store = [&](int k, const Raw& R) {
    double w[NG];
    if (h_ii < 0 || h_ii >= g.nr) {
      const int side = h_ii < 0 ? 0 : 1, layer = min(h_ii < 0 ? -1 - h_ii : h_ii - g.nr, 1);
      const double* gt = a.t.ghr + ((size_t)(side * 2 + layer) * g.nz + k) * g.nf;
#pragma unroll
      for (int f = 0; f < NG; ++f) w[f] = gt[f];
    } else {
      form(R.e, cen(k, h_rr), w);
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) s_pl[k & 1][f][h_rr][h_cc] = w[f];
  };

  // a face by the short form (bp: the stationary velocity, pressure and density there), with
  // its Newton count tallied if the thread owns it; returns false where the general form has
  // to solve it.  (k, i): the lower cell.  Without gamma = 7/5 the general form at once
  auto general = [&](int dir, auto cell, int k, int i, bool own, double* F) {
    TStat st = {0, 0, 0, 0, 0, 0, 0};
    gas_face64_general<G75>(a, gc, recc, dir, k, i, cell, F, st);
    maxit = max(maxit, st.maxit);
    tally(own, st.last);
    if (st.fall) atomicAdd(&s_cnt.fall, (unsigned)st.fall);
    if (st.vac) atomicAdd(&s_cnt.vac, (unsigned)st.vac);
    if (st.noconv) atomicMax(&s_cnt.noconv, 1);
  };
  // (co: the weights of the cells on both sides)
  auto face = [&](auto dirc, auto cell, const double* co, const double* bp, int k, int i, bool own,
                  double* F) {
    constexpr int D = decltype(dirc)::value;
    if constexpr (!G75) {
      general(D, cell, k, i, own, F);
      return true;
    } else {
      double qL[NG], qR[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) {
        face_pair<D>(recc, cell(0, f), cell(1, f), cell(2, f), cell(3, f), co, co, qL[f], qR[f]);
        if (f == 1 || f > 2) {
          qL[f] = bp[f == 1 ? 0 : f - 2] + qL[f];
          qR[f] = bp[f == 1 ? 0 : f - 2] + qR[f];
        }
      }
      int last = 0;
      const bool ok = gas_face64<D>(gc, qL, qR, F, last);
      if (ok) maxit = max(maxit, last);
      tally(own && ok, last);
      return ok;
    }
  };
  using DR = std::integral_constant<int, 0>;
  using DT = std::integral_constant<int, 1>;
  using DZ = std::integral_constant<int, 2>;
  double smax = 0.0, tsmin = 1e300, ledger = 0.0;

  tab_store(k0, tab_load(k0));
  for (int p = k0 - 2; p < k0; ++p)
    if (cen_t) tab_store(p, tab_load(p));
  __syncthreads();
  double rp[NG], fzlo[NG];
  {
    Raw R;
    double r0[NG];
    // (planes below k0 are not in the ring of centre entries)
    auto form_at = [&](int k, double* out) {
      const ctab c = to_ctab(a.t.wc) + ((size_t)min(max(k, 0), g.nz - 1) * g.nr + igc) * WB_N;
      const double cf[2] = {c[WB_RHO], c[WB_V]};
      col_fetch(vin, k, R);
      col_form(k, R, cf, out);
    };
    if (!twod) {
      double e2[NG], rm[NG];
      form_at(k0 - 2, e2);
      form_at(k0 - 1, rm);
      form_at(k0, r0);
      form_at(k0 + 1, rp);
      const ctab c = to_ctab(a.t.wz) + ((size_t)k0 * g.nr + igc) * WB_N;
      const double bp[NF] = {c[WB_V], c[WB_P], c[WB_RHO]};
      auto get = [&](int s, int f) { return s == 0 ? e2[f] : s == 1 ? rm[f] : s == 2 ? r0[f] : rp[f]; };
      if (!face(DZ(), get, nullptr, bp, k0 - 1, igc, act && k0 == 0, fzlo))
        general(2, get, k0 - 1, igc, act && k0 == 0, fzlo);
      if (a.second && k0 == 0 && act) ledger -= rt[RT_AZ] * fzlo[4];
#pragma unroll
      for (int f = 0; f < NG; ++f) s_rm[f][tid] = rm[f];
    } else {
      form_at(0, r0);
#pragma unroll
      for (int f = 0; f < NG; ++f) { rp[f] = 0.0; fzlo[f] = 0.0; }
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) s_pl[k0 & 1][f][ti + 2][tj + 2] = r0[f];
    if (halo_t) {
      halo_fetch(k0, R);
      halo_store(k0, R);
    }
  }
  const double dt = a.dt_idx >= 0 ? a.c.dtlog[a.dt_idx] : 0.0;

  // One barrier per plane: behind the one that ends plane k the update of plane k - 1 and, in
  // the other half of the LDS arrays, the faces of plane k.
  const double* row = s_row[ti];
  Raw base;
  double dvar[ND > 0 ? ND : 1][4], dz[NG];
  for (int kk = k0;; ++kk) {
    __syncthreads();
    // the column's cell kk+2 and the next plane's halo and tables
    const bool more = kk + 1 < k1;
    Raw nraw, hraw;
    double tab_next = 0.0;
    col_fetch(vin, kk + 2, nraw);
    if (more) {
      if (halo_t) halo_fetch(kk + 1, hraw);
      tab_next = tab_load(kk + 1);
    }
    if (kk > k0) {
      const int k = kk - 1;
      // boundary outflow ledger
      if (a.second && act) {
        if (ig == g.nr - 1) ledger += row[RW_AR1] * s_fr[k & 1][4][ti + 1][tj];
        if (ig == 0) ledger -= row[RW_AR0] * s_fr[k & 1][4][0][tj];
        if (!twod && k == g.nz - 1) ledger += row[RW_AZ] * fzlo[4];
      }
      // ---- divergence -sum_s A_s F.n_s (Sect. 2.2), sources (App. B), drag (Sect. 2.9)
      double r0[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) r0[f] = s_pl[k & 1][f][ti + 2][tj + 2];
      const double *upd = &s_upd[k & 3][ti * NU], *fc = &s_face[k & 3][ti * NF];
      // the cell's primitives: stationary flow + W'
      const double rho = fc[2] + r0[4], p = fc[1] + r0[3];
      const double u = r0[0], v = fc[0] + r0[1], w = r0[2];
      const double invrc = row[RW_INVRC], gr = upd[5], gz = upd[6];
      double S[NG];
      S[0] = (rho * v * v + p) * invrc + rho * gr;
      S[1] = -(rho * u * v) * invrc;
      S[2] = rho * gz;
      S[3] = rho * (u * gr + w * gz);
      S[4] = 0.0;
      if (drag) {
        double dx = 0.0, dy = 0.0, dzz = 0.0;
#pragma unroll
        for (int s2 = 0; s2 < ND; ++s2) {
          const double rd = dvar[s2][3];
          double ud = 0.0, vd = 0.0, wd = 0.0;
          if (rd > 0.0) {
            const double id = 1.0 / rd;
            ud = dvar[s2][0] * id;
            vd = dvar[s2][1] * id;
            wd = dvar[s2][2] * id;
          }
          const double its = inv_tstop<EXT>(g, s2, row[RW_OMK], rho, p);
          dx += rd * (ud - u) * its;
          dy += rd * (vd - v) * its;
          dzz += rd * (wd - w) * its;
        }
        S[0] += dx;
        S[1] += dy;
        S[2] += dzz;
        S[3] += u * dx + v * dy + w * dzz;
      }
      // indirect gravity (Sect. 2.10): minus the star's acceleration by the disc
      if (EXT && g.indirect && a.mode != MODE_RESID) {
        const double A = a.t.indab[0], B = a.t.indab[1];
        const double cs = a.t.trig[jl], sn = a.t.trig[g.nth + jl];
        const double acr = -g.GM * (A * cs + B * sn), act_ = -g.GM * (B * cs - A * sn);
        S[0] += rho * acr;
        S[1] += rho * act_;
        S[3] += rho * u * acr + rho * v * act_;
      }
      // boundary damping zones (Sect. 2.4): the gas deviation relaxes to the stationary flow
      if (EXT && g.damp) {
        const double kd = a.t.damp[(size_t)k * g.nr + igc];
        Raw e;
        col_fetch(vin, k, e);
#pragma unroll
        for (int f = 0; f < NG; ++f) S[f] -= kd * e.e[f];
      }
      // (every face and the residual read first, in one batch)
      const double *r_hi = &s_fr[k & 1][0][ti + 1][tj], *r_lo = &s_fr[k & 1][0][ti][tj];
      const double *t_lo = tj ? &s_ft[0][tid - 1] : &s_fe[k & 1][0][ti];
      const int t_st = tj ? NTM : TM;
      double Gt[NG], res[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) res[f] = upd[7 + f];
      const double ar0 = row[RW_AR0], ar1 = row[RW_AR1], ath = row[RW_ATH], vol = row[RW_V];
#pragma unroll
      for (int f = 0; f < NG; ++f) {
        const double dr = ar1 * r_hi[f * (TM + 1) * TJ] - ar0 * r_lo[f * (TM + 1) * TJ];
        const double dth = ath * (s_ft[f][tid] - t_lo[f * t_st]);
        Gt[f] = fma(S[f], vol, -((dr + dth) + dz[f]));
        Gt[f] -= a.mode != MODE_RESID ? res[f] : 0.0;
      }
      if (a.mode == MODE_RESID) {
        if (act && jg == 0) {
#pragma unroll
          for (int f = 0; f < NG; ++f) a.c.r0w[((size_t)k * g.nr + ig) * 5 + f] = Gt[f];
        }
      } else if (a.mode == MODE_OPER) {
        if (act) {
#pragma unroll
          for (int f = 0; f < NG; ++f)
            at_row((double*)a.out + (size_t)f * g.N + (size_t)k * plane + row0, jl) = Gt[f];
        }
      } else if (act) {
        // all loads before any store (the second stage updates in place)
        const double cdt = a.coef * dt * row[RW_INVV];
        double qn[NG];
#pragma unroll
        for (int f = 0; f < NG; ++f) qn[f] = upd[f];
#pragma unroll
        for (int f = 0; f < NG; ++f) {
          const double nv = fma(cdt, Gt[f], base.e[f]);
          qn[f] += nv;
          at_row((double*)a.out + (size_t)f * g.N + (size_t)k * plane + row0, jl) = nv;
        }
        // positivity of the new gas state; CFL of the new state (second stage)
        const double in2 = 1.0 / qn[4];
        const double un = qn[0] * in2, vn = qn[1] * in2, wn = qn[2] * in2;
        const double pn = (g.gamma - 1.0) * (qn[3] - 0.5 * (qn[0] * un + qn[1] * vn + qn[2] * wn));
        if (!(qn[4] > 0.0 && pn > 0.0)) {
          atomicOr(&a.c.ctrl->status, FL_NEG);
          atomicMin(&a.c.ctrl->first_bad, (unsigned long long)((size_t)k * plane + (size_t)ig * g.nth + jg));
          atomicCAS(&a.c.ctrl->bad_step, -1, a.step);
        } else if (a.second) {
          const double spd = sqrt(un * un + vn * vn + wn * wn) + sqrt(g.gamma * pn * in2);
          smax = fmax(smax, spd);
          if (EXT && g.drag_law) {
#pragma unroll
            for (int s2 = 0; s2 < ND; ++s2)
              tsmin = fmin(tsmin, 1.0 / inv_tstop<EXT>(g, s2, row[RW_OMK], qn[4], pn));
          }
        }
      }
      if (kk < k1) {
#pragma unroll
        for (int f = 0; f < NG; ++f) s_rm[f][tid] = r0[f];
      }
    }
    if (kk == k1) break;
    wave_order();
    const int k = kk;
    double (*pl)[TM + 4][HW] = s_pl[k & 1];
    const double* face_c = &s_face[k & 3][ti * NF];
    const double* face_r = &s_face[k & 3][(TM + ti + 1) * NF];
    const double* face_z = &s_face[k & 3][(2 * TM + 1 + ti) * NF];
    unsigned bad = 0;
    // ---- theta face j+1/2
    {
      auto get = [&](int c, int f) { return pl[f][ti + 2][tj + 1 + c]; };
      double F[NG];
      if (!face(DT(), get, nullptr, face_c, k, igc, act, F)) bad |= 1;
#pragma unroll
      for (int f = 0; f < NG; ++f) s_ft[f][tid] = F[f];
    }
    // ---- r face i+1/2
    {
      auto get = [&](int c, int f) { return pl[f][ti + 1 + c][tj + 2]; };
      double F[NG];
      if (!face(DR(), get, s_wt[ti + 1], face_r, k, min(ig, g.nr), act, F)) bad |= 2;
#pragma unroll
      for (int f = 0; f < NG; ++f) s_fr[k & 1][f][ti + 1][tj] = F[f];
    }
    // ---- lower-edge faces of the tile: r face i0-1/2 (threads 0..63) and theta face
    //      j0-1/2 of each row (threads 64..71)
    if (tid < TJ) {
      auto get = [&](int c, int f) { return pl[f][c][tid + 2]; };
      double F[NG];
      // (the upper face of the tile below, which owns it, except at the inner boundary)
      if (!face(DR(), get, s_wt[0], &s_face[k & 3][TM * NF], k, i0 - 1,
                i0 == 0 && jg < g.nth, F))
        bad |= 4;
#pragma unroll
      for (int f = 0; f < NG; ++f) s_fr[k & 1][f][0][tid] = F[f];
    } else if (tid < TJ + TM) {
      const int row = tid - TJ;
      auto get = [&](int c, int f) { return pl[f][row + 2][c]; };
      double F[NG];
      if (!face(DT(), get, nullptr, &s_face[k & 3][row * NF], k,
                min(i0 + row, g.nr - 1), false, F))
        bad |= 4;
#pragma unroll
      for (int f = 0; f < NG; ++f) s_fe[k & 1][f][row] = F[f];
    }
    // the next plane's halo and tables
    if (more) {
      if (halo_t) halo_store(k + 1, hraw);
      tab_store(k + 1, tab_next);
    }
    // the update's base of this cell and the dust its drag needs (raw stored values)
    if (a.mode == MODE_UPDATE && act) col_fetch((const double*)a.base, k, base);
    if (drag) {
      const size_t r = (size_t)k * plane + row0;
#pragma unroll
      for (int s2 = 0; s2 < ND; ++s2)
#pragma unroll
        for (int c = 0; c < 4; ++c) dvar[s2][c] = at_row(vin + (size_t)(5 + 4 * s2 + c) * g.N + r, jl);
    }
    // ---- z face k+1/2
    double rn[NG], fzhi[NG];
    if (!twod) {
      col_form(k + 2, nraw, cen(k + 2, ti + 2), rn);
      auto get = [&](int c, int f) {
        return c == 0 ? s_rm[f][tid] : c == 1 ? pl[f][ti + 2][tj + 2] : c == 2 ? rp[f] : rn[f];
      };
      if (!face(DZ(), get, nullptr, face_z, k, igc, act, fzhi)) bad |= 8;
    } else {
#pragma unroll
      for (int f = 0; f < NG; ++f) { rn[f] = 0.0; fzhi[f] = 0.0; }
    }
    // ---- the faces the short form did not take (rare), one call for all kinds: own theta and
    //      r face, tile edge, z face
    if (G75 && __builtin_expect(!wave_none(bad != 0), 0)) {
#pragma nounroll
      for (int kind = 0; kind < 4; ++kind) {
        if (!(bad >> kind & 1)) continue;
        const bool edge_r = kind == 2 && tid < TJ, along_th = kind == 0 || (kind == 2 && !edge_r);
        const int rr = kind == 0 ? ti + 2 : kind == 1 ? ti + 1 : edge_r ? 0 : tid - TJ + 2;
        const int cc = kind == 0 ? tj + 1 : along_th ? 0 : tj + 2;
        const double* p = &pl[0][rr][cc];
        const int st = along_th ? 1 : HW;
        auto cell = [&](int c, int f) {
          if (kind == 3)
            return c == 0 ? s_rm[f][tid] : c == 1 ? pl[f][ti + 2][tj + 2] : c == 2 ? rp[f] : rn[f];
          return p[f * (TM + 4) * HW + c * st];
        };
        const int i = kind == 1 ? min(ig, g.nr) : kind == 2 ? (edge_r ? i0 - 1 : min(i0 + tid - TJ, g.nr - 1)) : igc;
        double F[NG];
        general(along_th ? 1 : kind == 3 ? 2 : 0, cell, k, i,
                kind == 2 ? edge_r && i0 == 0 && jg < g.nth : act, F);
#pragma unroll
        for (int f = 0; f < NG; ++f) {
          if (kind == 0) s_ft[f][tid] = F[f];
          else if (kind == 1) s_fr[k & 1][f][ti + 1][tj] = F[f];
          else if (kind == 3) fzhi[f] = F[f];
          else if (edge_r) s_fr[k & 1][f][0][tid] = F[f];
          else s_fe[k & 1][f][tid - TJ] = F[f];
        }
      }
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) {
      dz[f] = row[RW_AZ] * (fzhi[f] - fzlo[f]);
      fzlo[f] = fzhi[f];
      if (more) s_pl[(k + 1) & 1][f][ti + 2][tj + 2] = rp[f];
      rp[f] = rn[f];
    }
  }

  // ---- block reductions: counters, CFL partial, boundary outflow partial
  __syncthreads();
  const int wv = tid / 64, ln = tid & 63;
  const int mi = wave_imax(maxit);
  if (ln < 8 && s_nh[wv][ln])
    atomicAdd(&a.c.ctrl->newton_hist[ln], (unsigned long long)s_nh[wv][ln]);
  if (ln == 0 && mi) atomicMax(&a.c.ctrl->maxit, mi);
  if (tid == 0) {
    if (s_cnt.fall) atomicAdd(&a.c.ctrl->nfall, (unsigned long long)s_cnt.fall);
    if (s_cnt.vac) { atomicAdd(&a.c.ctrl->nvac, (unsigned long long)s_cnt.vac); atomicOr(&a.c.ctrl->status, FL_VAC); }
    if (s_cnt.noconv) { atomicOr(&a.c.ctrl->status, FL_NOCONV); atomicCAS(&a.c.ctrl->bad_step, -1, a.step); }
  }
  if (a.second && a.mode == MODE_UPDATE) {
    // the CFL bound of the thread's row decreases with the speed: the largest one's
    const double m = wave_min(smax > 0.0 ? g.cfl * rt[RT_V] / (smax * rt[RT_MAXA]) : 1e300);
    const double ls = wave_sum(ledger);
    const double tm = (EXT && ND > 0) ? wave_min(tsmin) : 1e300;
    if (ln == 0) { s_red[wv][0] = m; s_red[wv][1] = ls; s_red[wv][2] = tm; }
    __syncthreads();
    if (tid == 0) {
      double mm = s_red[0][0], lsum = s_red[0][1], tmm = s_red[0][2];
      for (int w2 = 1; w2 < NTM / 64; ++w2) {
        mm = fmin(mm, s_red[w2][0]);
        lsum += s_red[w2][1];
        tmm = fmin(tmm, s_red[w2][2]);
      }
      a.c.cflp[(size_t)blockIdx.x * 5] = mm;
      a.c.outp[(size_t)blockIdx.x * 5] = lsum;
      if (EXT && g.drag_law) a.c.tsp[blockIdx.x] = tmm;
    }
  }
}

// ------------------------------------------------------------------------------------
// the dust stage kernel

// One RK2 stage of one dust species; tiles, planes and update as k_gas.  Bound by
// instruction issue and by the waits between its barriers, so it is written for two
// workgroups on a CU (four waves per SIMD, 128 VGPRs): while one waits at a barrier or for
// memory the other computes.  What a plane needs between phases therefore lives in LDS
// where it can: the cell below (s_rm) and the current cell (the staged plane itself) of the
// thread's column; registers keep only the cell above, the flux of the z face below and the
// raw loads in flight, all requested before the faces that hide them.  Three-dust disc
// 512 x 1024 x 128, FP32-perturbation form: 1.92 -> 1.74 ms per launch, 1.63 (4.7 GB, 2.9
// TB/s) once its loads no longer counted as LDS accesses; one-dust disc 256 x 512 x 64, FP64:
// 0.30 -> 0.25 ms (1.0 GB, 4.0 TB/s).
template <bool P32, bool EXT>
__global__ void __launch_bounds__(NTM, 4) k_dust(StageArgs a, int species) {
  __shared__ int s_stop;
  if (threadIdx.x == 0) s_stop = __atomic_load_n(&a.c.ctrl->status, __ATOMIC_RELAXED);
  __syncthreads();
  if (s_stop & FL_HARD) return;
  constexpr int NG = 4, HW = TJ + 4, NHALO = 4 * HW + 4 * TM;
  static_assert(NHALO <= NTM, "one halo cell per thread");
  __shared__ double s_pl[NG][TM + 4][HW];
  __shared__ double s_ft[NG][TM][TJ + 1];
  __shared__ double s_fr[NG][TM + 1][TJ];
  __shared__ double s_rm[NG][NTM];
  __shared__ double s_red[NTM / 64][2];
  // per-plane tables: the stationary conservative state and gravity of the tile's rows, one
  // plane ahead; the stationary azimuthal velocity of the rows and their halo, two ahead
  constexpr int NTAB = TM * 7, NV0 = TM + 4;
  __shared__ double s_tab[2][NTAB];
  __shared__ double s_v0[4][NV0];

  const Geo& g = a.g;
  const RecC recc;
  const int F0 = 5 + 4 * species, slot = 1 + species;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int tjb = tile % a.ntj;
  const int tib = (tile / a.ntj) % a.ntm;
  const int kcb = tile / (a.ntj * a.ntm);
  const int tid = threadIdx.x, tj = tid & (TJ - 1);
  const int ti = __builtin_amdgcn_readfirstlane(tid / TJ);
  const int j0 = tjb * TJ, i0 = tib * TM;
  const int k0 = kcb * a.tk_dust, k1 = min(g.nz, k0 + a.tk_dust);
  const int jg = j0 + tj;
  const int ig = i0 + ti, igc = min(ig, g.nr - 1);
  const bool act = jg < g.nth && ig < g.nr;
  const bool drag = !g.drag_exact;
  const bool twod = g.twod != 0;
  const size_t plane = (size_t)g.nr * g.nth;
  TStat st = {0, 0, 0, 0, 0, 0, 0};
  // the thread's column; the threads past the last one go on round the circle, so that every
  // face solved is one of the mesh (their flags and counts are the mesh's) and no slot of the
  // staged plane has two writers
  const unsigned jl = (unsigned)(jg % g.nth);
  const size_t row0 = (size_t)igc * g.nth;  // (a wavefront has one row: scalar)
  // tables of the wavefront's row, by scalar loads
  const ctab rt = to_ctab(a.t.rt) + (size_t)igc * RT_N, ar = to_ctab(a.t.ar), rco = to_ctab(a.t.rco);
  // thread t stages table entry t: tab_p + plane * tab_stride
  const bool tab_t = tid < NTAB, v0_t = P32 && tid >= NTAB && tid < NTAB + NV0;
  const double* tab_p = nullptr;
  unsigned tab_stride = 0;
  if (tid < TM * 5) {
    tab_p = a.t.bgc + (size_t)min(i0 + tid / 5, g.nr - 1) * 5 + tid % 5;
    tab_stride = g.nr * 5u;
  } else if (tab_t) {
    const int e = tid - TM * 5;
    tab_p = a.t.grav + (size_t)min(i0 + e / 2, g.nr - 1) * 2 + e % 2;
    tab_stride = g.nr * 2u;
  } else if (v0_t) {
    tab_p = a.t.wc + (size_t)min(max(i0 + tid - NTAB - 2, 0), g.nr - 1) * WB_N + WB_V;
    tab_stride = g.nr * (unsigned)WB_N;
  }
  auto tab_load = [&](int k) {  // (bgc and gravity of plane k, the velocity of plane k + 2)
    return tab_p[(size_t)min(v0_t ? k + 2 : k, g.nz - 1) * tab_stride];
  };
  auto tab_store = [&](int k, double x) {
    if (tab_t) s_tab[k & 1][tid] = x;
    if (v0_t) s_v0[(k + 2) & 3][tid - NTAB] = x;
  };

  // the state's arrays of this species: FP64 layout, momenta and density; FP32 layout,
  // velocity deviations (FP32) and density
  using VT = typename std::conditional<P32, float, double>::type;
  auto vel_of = [&](const void* s) {
    return (const VT*)s + (size_t)(P32 ? 5 + 3 * species : F0) * g.N;
  };
  auto den_of = [&](const void* s) {
    return (const double*)s + (P32 ? p32_f64_base(g) + (size_t)species * g.N : (size_t)(F0 + 3) * g.N);
  };
  const VT* vin = vel_of(a.in);
  const double* din = den_of(a.in);
  struct Raw { VT m[3]; double rd; };
  // reconstructed variables (velocity, zero where the density is not positive; density)
  // of a stored cell whose stationary azimuthal velocity is v0
  auto form = [&](const Raw& R, double v0, double* out) {
    const bool full = R.rd > 0.0;
    if constexpr (P32) {
      out[0] = full ? (double)R.m[0] : 0.0;
      out[1] = full ? v0 + (double)R.m[1] : 0.0;
      out[2] = full ? (double)R.m[2] : 0.0;
    } else {
      const double id = full ? 1.0 / R.rd : 0.0;
#pragma unroll
      for (int f = 0; f < 3; ++f) out[f] = R.m[f] * id;
    }
    out[3] = R.rd;
  };
  // the thread's cell of plane k of its column; rows and planes outside the grid are
  // clamped into it and replaced when formed
  auto col_fetch = [&](const VT* v, const double* d, int k, Raw& R) {
    const size_t r = (size_t)min(max(k, 0), g.nz - 1) * plane + row0;
#pragma unroll
    for (int f = 0; f < 3; ++f) R.m[f] = at_row(v + (size_t)f * g.N + r, jl);
    R.rd = at_row(d + r, jl);
  };
  auto col_form = [&](int k, const Raw& R, double v0, double* out) {
    if ((k < 0 || k >= g.nz) && !(EXT && g.bc_z == 1)) {
      const int side = k < 0 ? 0 : 1, layer = min(k < 0 ? -1 - k : k - g.nz, 1);
      const ctab gt = to_ctab(a.t.ghz) + ((size_t)(side * 2 + layer) * g.nr + igc) * g.nf + F0;
#pragma unroll
      for (int f = 0; f < NG; ++f) out[f] = gt[f];
    } else if (k >= 0 && k < g.nz && ig >= g.nr) {
      const ctab gt = to_ctab(a.t.ghr) + ((size_t)(2 + min(ig - g.nr, 1)) * g.nz + k) * g.nf + F0;
#pragma unroll
      for (int f = 0; f < NG; ++f) out[f] = gt[f];
    } else {
      form(R, v0, out);  // (outflow: the boundary cell's variables)
    }
  };
  // the thread's cell of the halo ring
  const bool halo_t = tid < NHALO;
  int h_rr = 0, h_cc = 0;
  if (tid < 2 * HW) { h_rr = tid / HW; h_cc = tid % HW; }
  else if (tid < 4 * HW) { h_rr = TM + 2 + (tid - 2 * HW) / HW; h_cc = (tid - 2 * HW) % HW; }
  else if (halo_t) { const int e = tid - 4 * HW; h_rr = 2 + e / 4; h_cc = (e & 3) < 2 ? (e & 3) : TJ + (e & 3); }
  const int h_ii = i0 + h_rr - 2;
  const bool h_gh = h_ii < 0 || h_ii >= g.nr;
  const size_t h_off = (size_t)min(max(h_ii, 0), g.nr - 1) * g.nth + (j0 + h_cc - 2 + g.nth) % g.nth;
  auto halo_fetch = [&](int k, Raw& R) {
#pragma unroll
    for (int f = 0; f < 3; ++f) R.m[f] = at_plane(vin + (size_t)f * g.N + (size_t)k * plane, h_off);
    R.rd = at_plane(din + (size_t)k * plane, h_off);
  };
  auto halo_store = [&](int k, const Raw& R) {
    double w[NG];
    if (h_gh) {
      const int side = h_ii < 0 ? 0 : 1, layer = min(h_ii < 0 ? -1 - h_ii : h_ii - g.nr, 1);
      const double* gt = a.t.ghr + ((size_t)(side * 2 + layer) * g.nz + k) * g.nf + F0;
#pragma unroll
      for (int f = 0; f < NG; ++f) w[f] = gt[f];
    } else {
      form(R, P32 ? s_v0[k & 3][h_rr] : 0.0, w);
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) s_pl[f][h_rr][h_cc] = w[f];
  };

  using DR = std::integral_constant<int, 0>;
  using DT = std::integral_constant<int, 1>;
  using DZ = std::integral_constant<int, 2>;
  double ledger = 0.0, vmax2 = 0.0;

  // column: the cell above the current plane (rp), the flux of the z face below; the
  // current cell goes to the staged plane, the one below to its LDS slot
  double rp[NG], fzlo[NG];
  if (tab_t) tab_store(k0, tab_load(k0));
  for (int p = k0; p < k0 + 3; ++p)
    if (v0_t) tab_store(p - 2, tab_load(p - 2));
  {
    Raw R;
    double r0[NG];
    const ctab wc = to_ctab(a.t.wc) + (size_t)igc * WB_N + WB_V;
    auto vc = [&](int k) { return P32 ? wc[(size_t)min(max(k, 0), g.nz - 1) * g.nr * WB_N] : 0.0; };
    if (!twod) {
      double e2[NG], rm[NG];
      col_fetch(vin, din, k0 - 2, R); col_form(k0 - 2, R, vc(k0 - 2), e2);
      col_fetch(vin, din, k0 - 1, R); col_form(k0 - 1, R, vc(k0 - 1), rm);
      col_fetch(vin, din, k0, R); col_form(k0, R, vc(k0), r0);
      col_fetch(vin, din, k0 + 1, R); col_form(k0 + 1, R, vc(k0 + 1), rp);
      auto get = [&](int c, int f) { return c == 0 ? e2[f] : c == 1 ? rm[f] : c == 2 ? r0[f] : rp[f]; };
      dust_face<DZ::value>(recc, get, nullptr, nullptr, fzlo, st);
      if (a.second && k0 == 0 && act) ledger -= rt[RT_AZ] * fzlo[3];
#pragma unroll
      for (int f = 0; f < NG; ++f) s_rm[f][tid] = rm[f];
    } else {
      col_fetch(vin, din, 0, R); col_form(0, R, vc(0), r0);
#pragma unroll
      for (int f = 0; f < NG; ++f) { rp[f] = 0.0; fzlo[f] = 0.0; }
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) s_pl[f][ti + 2][tj + 2] = r0[f];
    if (P32) __syncthreads();  // the velocity tables, with which the halo is formed
    if (halo_t) {
      halo_fetch(k0, R);
      halo_store(k0, R);
    }
  }
  const double dt = a.dt_idx >= 0 ? a.c.dtlog[a.dt_idx] : 0.0;
  // the parabola weights of the r face above the row (and below it, for the tile's edge)
  auto weights = [&](int i) { return rco + (size_t)(min(max(i, -1), g.nr) + 1) * RC_N; };

  for (int k = k0; k < k1; ++k) {
    const bool more = k + 1 < k1;
    __syncthreads();
    // the column's cell k+2 and the next plane's halo
    Raw nraw, hraw;
    double tab_next = 0.0;
    if (!twod) col_fetch(vin, din, k + 2, nraw);
    if (more) {
      if (halo_t) halo_fetch(k + 1, hraw);
      if (tab_t || v0_t) tab_next = tab_load(k + 1);
    }
    // ---- theta face j+1/2
    {
      auto get = [&](int c, int f) { return s_pl[f][ti + 2][tj + 1 + c]; };
      double F[NG];
      dust_face<DT::value>(recc, get, nullptr, nullptr, F, st);
#pragma unroll
      for (int f = 0; f < NG; ++f) s_ft[f][ti][tj + 1] = F[f];
    }
    // the update's base of this cell and the gas state its drag needs (raw stored values);
    // stage 1 of the FP32 layout has its base in the staged plane
    const bool upd = a.mode == MODE_UPDATE && act;
    const bool base_r0 = P32 && a.base == a.in;
    Raw base;
    VT pg[5];
    if (upd && !base_r0) col_fetch(vel_of(a.base), den_of(a.base), k, base);
    if (drag) {
#pragma unroll
      for (int f = 0; f < 5; ++f)
        pg[f] = at_row((const VT*)a.in + (size_t)f * g.N + (size_t)k * plane + row0, jl);
    }
    // ---- r face i+1/2
    {
      auto get = [&](int c, int f) { return s_pl[f][ti + 1 + c][tj + 2]; };
      double F[NG];
      dust_face<DR::value>(recc, get, weights(ig), weights(ig + 1), F, st);
      if (a.second && act && ig == g.nr - 1) ledger += ar[igc + 1] * F[3];
#pragma unroll
      for (int f = 0; f < NG; ++f) s_fr[f][ti + 1][tj] = F[f];
    }
    // ---- lower-edge faces of the tile: r face i0-1/2 (threads 0..63) and theta face
    //      j0-1/2 of each row (threads 64..71)
    if (tid < TJ) {
      auto get = [&](int c, int f) { return s_pl[f][c][tid + 2]; };
      double F[NG];
      dust_face<DR::value>(recc, get, weights(i0 - 1), weights(i0), F, st);
#pragma unroll
      for (int f = 0; f < NG; ++f) s_fr[f][0][tid] = F[f];
      if (a.second && i0 == 0 && j0 + tid < g.nth) ledger -= ar[0] * F[3];
    } else if (tid < TJ + TM) {
      const int row = tid - TJ;
      auto get = [&](int c, int f) { return s_pl[f][row + 2][c]; };
      double F[NG];
      dust_face<DT::value>(recc, get, nullptr, nullptr, F, st);
#pragma unroll
      for (int f = 0; f < NG; ++f) s_ft[f][row][0] = F[f];
    }
    // ---- z face k+1/2
    double rn[NG], dz[NG];
    if (!twod) {
      double fzhi[NG];
      col_form(k + 2, nraw, P32 ? s_v0[(k + 2) & 3][ti + 2] : 0.0, rn);
      auto get = [&](int c, int f) {
        return c == 0 ? s_rm[f][tid] : c == 1 ? s_pl[f][ti + 2][tj + 2] : c == 2 ? rp[f] : rn[f];
      };
      dust_face<DZ::value>(recc, get, nullptr, nullptr, fzhi, st);
      if (a.second && act && k == g.nz - 1) ledger += rt[RT_AZ] * fzhi[3];
#pragma unroll
      for (int f = 0; f < NG; ++f) {
        dz[f] = rt[RT_AZ] * (fzhi[f] - fzlo[f]);
        fzlo[f] = fzhi[f];
      }
    } else {
#pragma unroll
      for (int f = 0; f < NG; ++f) { rn[f] = 0.0; dz[f] = 0.0; }
    }
    // (the entries it replaces were last read before this plane's first barrier)
    if (more) tab_store(k + 1, tab_next);
    __syncthreads();
    if (halo_t && more) halo_store(k + 1, hraw);
    // ---- divergence -sum_s A_s F.n_s (Sect. 2.2), sources (App. B), drag (Sect. 2.9)
    double r0[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) r0[f] = s_pl[f][ti + 2][tj + 2];
    const double* bgc = &s_tab[k & 1][ti * 5];
    const double gr = s_tab[k & 1][TM * 5 + ti * 2], gz = s_tab[k & 1][TM * 5 + ti * 2 + 1];
    const double v0 = P32 ? s_v0[k & 3][ti + 2] : 0.0;
    const double invrc = rt[RT_INVRC];
    const double rd = r0[3], ud = r0[0], vd = r0[1], wd = r0[2];
    double fx = 0.0, fy = 0.0, fz = 0.0;
    if (drag) {
      double q[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) q[f] = bgc[f] + (double)pg[f];
      const double inv = 1.0 / q[4];
      const double u = q[0] * inv, v = q[1] * inv, w = q[2] * inv;
      const double pq = (EXT && g.drag_law)
          ? (g.gamma - 1.0) * (q[3] - 0.5 * (q[0] * u + q[1] * v + q[2] * w)) : 0.0;
      const double its = inv_tstop<EXT>(g, species, rt[RT_OMK], q[4], pq);
      fx = rd * (ud - u) * its;
      fy = rd * (vd - v) * its;
      fz = rd * (wd - w) * its;
    }
    double S[NG];
    S[0] = (rd * vd * vd) * invrc + rd * gr - fx;
    S[1] = -(rd * ud * vd) * invrc - fy;
    S[2] = rd * gz - fz;
    S[3] = 0.0;
    // indirect gravity (Sect. 2.10): minus the star's acceleration by the disc
    if (EXT && g.indirect) {
      const double A = a.t.indab[0], B = a.t.indab[1];
      const double cs = a.t.trig[jl], sn = a.t.trig[g.nth + jl];
      S[0] += rd * (-g.GM * (A * cs + B * sn));
      S[1] += rd * (-g.GM * (B * cs - A * sn));
    }
    double Gt[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) {
      const double dr = ar[igc + 1] * s_fr[f][ti + 1][tj] - ar[igc] * s_fr[f][ti][tj];
      const double dth = rt[RT_ATH] * (s_ft[f][ti][tj + 1] - s_ft[f][ti][tj]);
      Gt[f] = fma(S[f], rt[RT_V], -((dr + dth) + dz[f]));
    }
    if (a.mode == MODE_OPER) {
      if (act) {
#pragma unroll
        for (int f = 0; f < NG; ++f)
          at_row((VT*)a.out + (size_t)(F0 + f) * g.N + (size_t)k * plane + row0, jl) = (VT)Gt[f];
      }
    } else if (act) {
      // all loads before any store (the second stage updates in place)
      double nv[NG];
      const double cdt = a.coef * dt * rt[RT_INVV];
      if (base_r0) {
        // density times (stored velocity deviation + stationary velocity), the stored
        // deviation being zero where the density is not positive
        nv[0] = rd * ud;
        nv[1] = rd * (rd > 0.0 ? vd : v0);
        nv[2] = rd * wd;
        nv[3] = rd;
      } else if constexpr (P32) {
        nv[0] = base.rd * (double)base.m[0];
        nv[1] = base.rd * (v0 + (double)base.m[1]);
        nv[2] = base.rd * (double)base.m[2];
        nv[3] = base.rd;
      } else {
#pragma unroll
        for (int f = 0; f < 3; ++f) nv[f] = base.m[f];
        nv[3] = base.rd;
      }
#pragma unroll
      for (int f = 0; f < NG; ++f) nv[f] = fma(cdt, Gt[f], nv[f]);
      VT* vo = const_cast<VT*>(vel_of(a.out)) + (size_t)k * plane + row0;
      at_row(const_cast<double*>(den_of(a.out)) + (size_t)k * plane + row0, jl) = nv[3];
      if constexpr (P32) {
        // velocity deviations formed with the new density (zero where it vanishes)
        const bool full = nv[3] > 1e-300;
        const double ir = full ? frcp(nv[3]) : 0.0;
        at_row(vo, jl) = full ? (float)(nv[0] * ir) : 0.0f;
        at_row(vo + g.N, jl) = full ? (float)(nv[1] * ir - v0) : 0.0f;
        at_row(vo + 2 * g.N, jl) = full ? (float)(nv[2] * ir) : 0.0f;
      } else {
#pragma unroll
        for (int f = 0; f < 3; ++f) at_row(vo + (size_t)f * g.N, jl) = nv[f];
      }
      if (a.second && nv[3] < 0.0) {
        st.negd++;
      } else if (a.second && nv[3] > 0.0) {
        const double id = 1.0 / nv[3];
        const double a1 = nv[0] * id, a2 = nv[1] * id, a3 = nv[2] * id;
        vmax2 = fmax(vmax2, a1 * a1 + a2 * a2 + a3 * a3);
      }
    }
    // ---- shift the column
    if (more) {
#pragma unroll
      for (int f = 0; f < NG; ++f) {
        s_rm[f][tid] = r0[f];
        s_pl[f][ti + 2][tj + 2] = rp[f];
        rp[f] = rn[f];
      }
    }
  }

  // ---- block reductions: counters, CFL partial, boundary outflow partial
  const int wv = tid / 64, ln = tid & 63;
  const int nf = wave_isum(st.fall), nd = wave_isum(st.negd);
  if (ln == 0) {
    if (nd) atomicAdd(&a.c.ctrl->nnegd, (unsigned long long)nd);
    if (nf) atomicAdd(&a.c.ctrl->nfall, (unsigned long long)nf);
  }
  if (a.second && a.mode == MODE_UPDATE) {
    // the CFL bound of the thread's row decreases with the speed: the largest one's
    const double smax = sqrt(vmax2);
    const double m = wave_min(smax > 0.0 ? g.cfl * rt[RT_V] / (smax * rt[RT_MAXA]) : 1e300);
    const double ls = wave_sum(ledger);
    if (ln == 0) { s_red[wv][0] = m; s_red[wv][1] = ls; }
    __syncthreads();
    if (tid == 0) {
      double mm = s_red[0][0], lsum = s_red[0][1];
      for (int w2 = 1; w2 < NTM / 64; ++w2) {
        mm = fmin(mm, s_red[w2][0]);
        lsum += s_red[w2][1];
      }
      a.c.cflp[(size_t)blockIdx.x * 5 + slot] = mm;
      a.c.outp[(size_t)blockIdx.x * 5 + slot] = lsum;
    }
  }
}

// ------------------------------------------------------------------------------------
// the gas stage kernel of the FP32-perturbation form

// One RK2 stage of the gas in the FP32-perturbation form; tiles, planes and update as k_gas,
// addressing as k_dust.  Bound by instruction issue and the chains of the face solves: what
// the faces need of the stationary flow is staged a plane ahead (PertBg), azimuthal faces take
// the upwind state and the others the star state alone (gas_face32); the faces that form does
// not take are marked and solved together, by one inlined copy of the general form per plane.
// One barrier per plane and batched reads, as k_gas.  Lane-instructions per cell 1506 -> 1270:
// three-dust disc 512 x 1024 x 128, 4.97 -> 3.9 ms per launch; gas disc 128 x 256 x 64, 182 ->
// 136 us; the results the same to the last bit.  (Polynomials in place of the pressure
// functions took 990 instructions, 3.1 ms and 113 us, with other roundings: see gas_face32.)
// Two waves per SIMD: at three (12-row tiles, 168 VGPRs, the general form called) the largest
// disc gained 4% and the others lost more, at four (128) the general form's registers spilled
// into the faces.

template <int ND, bool EXT>
__global__ void __launch_bounds__(NTM, 2) k_gas32(StageArgs a) {
  __shared__ int s_stop;
  if (threadIdx.x == 0) s_stop = __atomic_load_n(&a.c.ctrl->status, __ATOMIC_RELAXED);
  __syncthreads();
  if (s_stop & FL_HARD) return;
  constexpr int NG = 5, HW = TJ + 4, NHALO = 4 * HW + 4 * TM;
  static_assert(NHALO <= NTM - 3 * 64, "one halo cell per thread");
  // (planes, faces and tables in halves and rings: as k_gas)
  __shared__ float s_pl[2][NG][TM + 4][HW];
  __shared__ float s_fr[2][NG][TM + 1][TJ];
  __shared__ float s_fe[2][NG][TM];
  __shared__ float s_ft[NG][NTM];  // (one copy: as k_gas)
  __shared__ float s_rm[NG][NTM];
  __shared__ double s_red[NTM / 64][3];
  // Newton counts of the faces the wavefront owns (bins 0..7, 7: seven or more)
  __shared__ int s_nh[NTM / 64][8];
  __shared__ GasCount s_cnt;
  // per-plane tables, in doubles: the stationary flow (PertBg) at the rows' centres, r faces
  // and upper z faces; (PertCell) at the centres of the rows and their halo, two planes ahead;
  // the update's (conservative state, gravity, density, velocity)
  constexpr int PFD = PF_D, NFACE = (3 * TM + 1) * PFD, NCEN = (TM + 4) * 2, NUPD = TM * 9;
  constexpr int T_CEN = NFACE, T_UPD = T_CEN + NCEN, NTAB = T_UPD + NUPD;
  static_assert(NTAB <= NTM, "one table entry per thread");
  __shared__ __align__(16) double s_face[4][NFACE];
  __shared__ __align__(16) double s_cen[4][NCEN];
  __shared__ double s_upd[4][NUPD];
  __shared__ __align__(16) float s_wt[TM + 1][8];
  enum { RW_AR0 = 0, RW_AR1, RW_ATH, RW_AZ, RW_V, RW_INVV, RW_INVRC, RW_OMK, RW_N };
  __shared__ double s_row[TM][RW_N];

  const Geo& g = a.g;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int tjb = tile % a.ntj;
  const int tib = (tile / a.ntj) % a.ntm;
  const int kcb = tile / (a.ntj * a.ntm);
  const int tid = threadIdx.x, tj = tid & (TJ - 1);
  const int ti = __builtin_amdgcn_readfirstlane(tid / TJ);
  const int j0 = tjb * TJ, i0 = tib * TM;
  const int k0 = kcb * a.tk, k1 = min(g.nz, k0 + a.tk);
  const int jg = j0 + tj;
  const int ig = i0 + ti, igc = min(ig, g.nr - 1);
  const bool act = jg < g.nth && ig < g.nr;
  const bool drag = ND > 0 && !g.drag_exact;
  const bool twod = g.twod != 0;
  const size_t plane = (size_t)g.nr * g.nth;
  const float gm1f = (float)(g.gamma - 1.0);
  const unsigned jl = (unsigned)(jg % g.nth);  // (past the grid: as k_dust)
  const size_t row0 = (size_t)igc * g.nth;
  const ctab rt = to_ctab(a.t.rt) + (size_t)igc * RT_N, ar = to_ctab(a.t.ar);
  if (tid < (TM + 1) * 8) {
    const int r = tid / 8, e = tid % 8, i = min(i0 + r - 1 + (e < 4 ? 0 : 1), g.nr);
    s_wt[r][e] = a.t.rcf[(size_t)(i + 1) * RC_N + e];
  } else if (tid >= 128 && tid < 128 + TM * RW_N) {
    const int r = (tid - 128) / RW_N, e = (tid - 128) % RW_N, i = min(i0 + r, g.nr - 1);
    const double* q = a.t.rt + (size_t)i * RT_N;
    s_row[r][e] = e == RW_AR0   ? a.t.ar[i]
                  : e == RW_AR1 ? a.t.ar[i + 1]
                  : e == RW_ATH ? q[RT_ATH]
                  : e == RW_AZ  ? q[RT_AZ]
                  : e == RW_V   ? q[RT_V]
                  : e == RW_INVV ? q[RT_INVV]
                  : e == RW_INVRC ? q[RT_INVRC]
                                  : q[RT_OMK];
  } else if (tid >= 256 && tid < 256 + NTM / 64 * 8) {
    s_nh[(tid - 256) / 8][tid & 7] = 0;
  }
  if (tid == 0) s_cnt = GasCount{0, 0, 0, 0};
  int maxit = 0;
  auto tally = [&](bool own, int last) {
    const int b = min(last, 7);
    unsigned long long left = __ballot(own);
    while (left) {
      const int at = __builtin_ctzll(left), v = __builtin_amdgcn_readlane(b, at);
      const unsigned long long mk = __ballot(own && b == v);
      if (tj == at) atomicAdd(&s_nh[ti][v], __popcll(mk));
      left &= ~mk;
    }
  };

  // thread NTM - 1 - t stages table entry t: as k_gas
  const int tt = NTM - 1 - tid;
  const double* tab_p = nullptr;
  size_t tab_stride = 0;
  if (tt < NTAB) {
    const size_t nr = (size_t)g.nr;
    if (tt < NFACE) {
      const int r = tt / PFD, e = tt % PFD;
      if (r < TM) {
        tab_p = a.t.pc + (size_t)min(i0 + r, g.nr - 1) * PFD + e;
        tab_stride = nr * PFD;
      } else if (r < 2 * TM + 1) {
        tab_p = a.t.pr + (size_t)min(i0 + r - TM, g.nr) * PFD + e;
        tab_stride = (nr + 1) * PFD;
      } else {
        tab_p = a.t.pz + (nr + (size_t)min(i0 + r - 2 * TM - 1, g.nr - 1)) * PFD + e;
        tab_stride = nr * PFD;
      }
    } else if (tt < T_UPD) {
      const int r = (tt - T_CEN) / 2, e = (tt - T_CEN) % 2;
      tab_p = a.t.pc + (size_t)min(max(i0 + r - 2, 0), g.nr - 1) * PFD + e;
      tab_stride = nr * PFD;
    } else {
      const int r = (tt - T_UPD) / 9, e = (tt - T_UPD) % 9;
      const size_t i = min(i0 + r, g.nr - 1);
      if (e < 5) { tab_p = a.t.bgc + i * 5 + e; tab_stride = nr * 5; }
      else if (e < 7) { tab_p = a.t.grav + i * 2 + (e - 5); tab_stride = nr * 2; }
      else { tab_p = a.t.wc + i * WB_N + (e == 7 ? WB_RHO : WB_V); tab_stride = nr * WB_N; }
    }
  }
  const bool cen_t = tt >= T_CEN && tt < T_UPD;
  auto tab_load = [&](int k) {  // (the centres' entries: of plane k + 2)
    return tt < NTAB ? tab_p[(size_t)min(cen_t ? k + 2 : k, g.nz - 1) * tab_stride] : 0.0;
  };
  auto tab_store = [&](int k, double x) {
    if (tt < NFACE) s_face[k & 3][tt] = x;
    else if (tt < T_UPD) s_cen[(k + 2) & 3][tt - T_CEN] = x;
    else if (tt < NTAB) s_upd[k & 3][tt - T_UPD] = x;
  };

  const float* vin = (const float*)a.in;
  struct Raw { float e[NG]; };
  auto col_fetch = [&](const float* v, int k, Raw& R) {
    const size_t r = (size_t)min(max(k, 0), g.nz - 1) * plane + row0;
#pragma unroll
    for (int f = 0; f < NG; ++f) R.e[f] = at_row(v + (size_t)f * g.N + r, jl);
  };
  // W' of the thread's cell of plane k; ghosts hold the stationary flow (W' = 0), except the
  // outflow condition's: the boundary cell's deviation scaled by the densities' ratio
  auto col_form = [&](int k, const Raw& R, const PertCell& c, float* out) {
    if (EXT && g.bc_z == 1 && (k < 0 || k >= g.nz)) {
      const size_t e = (size_t)((k < 0 ? 0 : 2) + min(k < 0 ? -1 - k : k - g.nz, 1)) * g.nr + igc;
      float s[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) s[f] = (float)((double)R.e[f] * a.t.ozr[e]);
      cell_w(s, a.t.ghzw + e * WB_N, gm1f, out);
    } else if (k < 0 || k >= g.nz || ig >= g.nr) {
#pragma unroll
      for (int f = 0; f < NG; ++f) out[f] = 0.0f;
    } else {
      cell_w32(R.e, c, gm1f, out);
    }
  };
  auto cen = [&](int k, int row) -> const PertCell& { return *(const PertCell*)&s_cen[k & 3][row * 2]; };
  // (by the wavefronts that k_gas takes)
  const int th = ti < 2 || ti == 4 ? -1 : tid - (ti < 4 ? 2 : 3) * 64;
  const bool halo_t = th >= 0 && th < NHALO;
  int h_rr = 0, h_cc = 0;
  if (!halo_t) {}
  else if (th < 2 * HW) { h_rr = th / HW; h_cc = th % HW; }
  else if (th < 4 * HW) { h_rr = TM + 2 + (th - 2 * HW) / HW; h_cc = (th - 2 * HW) % HW; }
  else if (halo_t) { const int e = th - 4 * HW; h_rr = 2 + e / 4; h_cc = (e & 3) < 2 ? (e & 3) : TJ + (e & 3); }
  const int h_ii = i0 + h_rr - 2;
  const size_t h_off = (size_t)min(max(h_ii, 0), g.nr - 1) * g.nth + (j0 + h_cc - 2 + g.nth) % g.nth;
  auto halo_fetch = [&](int k, Raw& R) {
#pragma unroll
    for (int f = 0; f < NG; ++f) R.e[f] = at_plane(vin + (size_t)f * g.N + (size_t)k * plane, h_off);
  };
  auto halo_store = [&](int k, const Raw& R) {
    float w[NG];
    cell_w32(R.e, cen(k, h_rr), gm1f, w);
    const bool ghost = h_ii < 0 || h_ii >= g.nr;
#pragma unroll
    for (int f = 0; f < NG; ++f) s_pl[k & 1][f][h_rr][h_cc] = ghost ? 0.0f : w[f];
  };

  // a face by the short form (b: the background there), with its Newton count tallied if
  // the thread owns it; returns false where the general form has to solve it
  auto bg_at = [](const double* p) -> const PertBg& { return *(const PertBg*)p; };
  auto face = [&](auto dirc, auto cell, const float* co, const PertBg& b, bool own, float* F) {
    constexpr int D = decltype(dirc)::value;
    float qL[NG], qR[NG];
    recon32<D>(cell, co, co, qL, qR);
    int last = 0;
    const bool ok = gas_face32<D>(b, qL, qR, F, last);
    if (ok) maxit = max(maxit, last);
    tally(own && ok, last);
    return ok;
  };
  // the same by the general form: stencil cells q, direction, lower cell (k, i)
  auto general = [&](int dir, const Face32& q, int k, int i, bool own, float* F) {
    const Face32Out o = gas_face32_general(a, dir, k, i, q);
#pragma unroll
    for (int f = 0; f < NG; ++f) F[f] = o.F[f];
    maxit = max(maxit, o.maxit);
    tally(own, o.last);
    if (o.fall) atomicAdd(&s_cnt.fall, o.fall);
    if (o.vac) atomicAdd(&s_cnt.vac, o.vac);
    if (o.resolve) atomicAdd(&s_cnt.resolve, o.resolve);
    if (o.noconv) atomicMax(&s_cnt.noconv, 1);
  };
  using DR = std::integral_constant<int, 0>;
  using DT = std::integral_constant<int, 1>;
  using DZ = std::integral_constant<int, 2>;
  double smax = 0.0, tsmin = 1e300, ledger = 0.0;

  tab_store(k0, tab_load(k0));
  for (int p = k0 - 2; p < k0; ++p)
    if (cen_t) tab_store(p, tab_load(p));
  __syncthreads();
  float rp[NG], fzlo[NG];
  {
    Raw R;
    float r0[NG];
    // (planes below k0 are not in the ring of centre entries)
    auto form_at = [&](int k, float* out) {
      const PertBg c = pert_at(a.t.pc, (size_t)min(max(k, 0), g.nz - 1) * g.nr + igc);
      col_fetch(vin, k, R);
      col_form(k, R, c.cell, out);
    };
    if (!twod) {
      float e2[NG], rm[NG];
      form_at(k0 - 2, e2);
      form_at(k0 - 1, rm);
      form_at(k0, r0);
      form_at(k0 + 1, rp);
      const PertBg bp = pert_at(a.t.pz, (size_t)k0 * g.nr + igc);
      auto get = [&](int s, int f) { return s == 0 ? e2[f] : s == 1 ? rm[f] : s == 2 ? r0[f] : rp[f]; };
      if (!face(DZ(), get, nullptr, bp, act && k0 == 0, fzlo)) {
        Face32 q;
#pragma unroll
        for (int f = 0; f < NG; ++f) { q.A[f] = e2[f]; q.B[f] = rm[f]; q.C[f] = r0[f]; q.D[f] = rp[f]; }
        general(2, q, k0 - 1, igc, act && k0 == 0, fzlo);
      }
      if (a.second && k0 == 0 && act) ledger -= rt[RT_AZ] * (double)fzlo[4];
#pragma unroll
      for (int f = 0; f < NG; ++f) s_rm[f][tid] = rm[f];
    } else {
      form_at(0, r0);
#pragma unroll
      for (int f = 0; f < NG; ++f) { rp[f] = 0.0f; fzlo[f] = 0.0f; }
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) s_pl[k0 & 1][f][ti + 2][tj + 2] = r0[f];
    if (halo_t) {
      halo_fetch(k0, R);
      halo_store(k0, R);
    }
  }
  const double dt = a.dt_idx >= 0 ? a.c.dtlog[a.dt_idx] : 0.0;

  // One barrier per plane: behind the one that ends plane k the update of plane k - 1 and, in
  // the other half of the LDS arrays, the faces of plane k.
  const double* row = s_row[ti];
  Raw base;
  double rds[ND > 0 ? ND : 1];
  float vds[ND > 0 ? ND : 1][3], dz[NG];
  for (int kk = k0;; ++kk) {
    __syncthreads();
    // the column's cell kk+2 and the next plane's halo and tables
    const bool more = kk + 1 < k1;
    Raw nraw, hraw;
    double tab_next = 0.0;
    col_fetch(vin, kk + 2, nraw);
    if (more) {
      if (halo_t) halo_fetch(kk + 1, hraw);
      tab_next = tab_load(kk + 1);
    }
    if (kk > k0) {
      const int k = kk - 1;
      // boundary outflow ledger (the stationary flow has no mass flux through these faces)
      if (a.second && act) {
        if (ig == g.nr - 1) ledger += row[RW_AR1] * (double)s_fr[k & 1][4][ti + 1][tj];
        if (ig == 0) ledger -= row[RW_AR0] * (double)s_fr[k & 1][4][0][tj];
        if (!twod && k == g.nz - 1) ledger += row[RW_AZ] * (double)fzlo[4];
      }
      // ---- divergence -sum_s A_s F.n_s (Sect. 2.2), sources (App. B), drag (Sect. 2.9): the
      //      source change S(E) - S(E0), every term formed from the perturbations W' (the
      //      stationary flow has no radial or vertical velocity)
      float r0[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) r0[f] = s_pl[k & 1][f][ti + 2][tj + 2];
      const double* upd = &s_upd[k & 3][ti * 9];
      const PertBg& fc = bg_at(&s_face[k & 3][ti * PFD]);
      const float rhop = r0[4], up = r0[0], vp = r0[1], wp = r0[2], pp = r0[3];
      const float v0 = fc.cell.v, rho = (float)(fc.cell.rho + (double)rhop);
      const float ir = (float)row[RW_INVRC], fgr = (float)upd[5], fgz = (float)upd[6];
      const float dmv2 = rhop * fc.cell.vsq + rho * vp * (2.0f * v0 + vp);
      float S[NG];
      S[0] = (dmv2 + pp) * ir + rhop * fgr;
      S[1] = -(rho * up * (v0 + vp)) * ir;
      S[2] = rhop * fgz;
      S[3] = rho * (up * fgr + wp * fgz);
      S[4] = 0.0f;
      if (drag) {
        const double rg = upd[7] + (double)rhop;
        const double u = (double)up, v = upd[8] + (double)vp, w2 = (double)wp;
        const double pq = (EXT && g.drag_law) ? a.t.wc[((size_t)k * g.nr + igc) * WB_N + WB_P] + (double)pp : 0.0;
        double dx = 0.0, dy = 0.0, dzz = 0.0;
#pragma unroll
        for (int s2 = 0; s2 < ND; ++s2) {
          // the FP32 layout stores the dust velocities as deviations from the stationary
          // flow's, as the gas W' is: the velocity difference is formed from the deviations
          const double rd = rds[s2];
          const bool full = rd > 0.0;
          const double dud = full ? (double)vds[s2][0] - (double)up : -u;
          const double dvd = full ? (double)vds[s2][1] - (double)vp : -v;
          const double dwd = full ? (double)vds[s2][2] - (double)wp : -w2;
          const double its = inv_tstop<EXT>(g, s2, row[RW_OMK], rg, pq);
          dx += rd * dud * its;
          dy += rd * dvd * its;
          dzz += rd * dwd * its;
        }
        S[0] += (float)dx;
        S[1] += (float)dy;
        S[2] += (float)dzz;
        S[3] += (float)(u * dx + v * dy + w2 * dzz);
      }
      // indirect gravity (Sect. 2.10): minus the star's acceleration by the disc
      if (EXT && g.indirect) {
        const double A = a.t.indab[0], B = a.t.indab[1];
        const double cs = a.t.trig[jl], sn = a.t.trig[g.nth + jl];
        const double acr = -g.GM * (A * cs + B * sn), act_ = -g.GM * (B * cs - A * sn);
        const double rg = upd[7] + (double)rhop;
        S[0] += (float)(rg * acr);
        S[1] += (float)(rg * act_);
        S[3] += (float)(rg * (double)up * acr + rg * (upd[8] + (double)vp) * act_);
      }
      // boundary damping zones (Sect. 2.4): the gas deviation relaxes to the stationary flow
      if (EXT && g.damp) {
        const double kd = a.t.damp[(size_t)k * g.nr + igc];
        Raw e;
        col_fetch(vin, k, e);
#pragma unroll
        for (int f = 0; f < NG; ++f) S[f] -= (float)(kd * (double)e.e[f]);
      }
      // (every face read first, in one batch)
      const float *r_hi = &s_fr[k & 1][0][ti + 1][tj], *r_lo = &s_fr[k & 1][0][ti][tj];
      const float* t_lo = tj ? &s_ft[0][tid - 1] : &s_fe[k & 1][0][ti];
      const int t_st = tj ? NTM : TM;
      const float ar0 = (float)row[RW_AR0], ar1 = (float)row[RW_AR1], ath = (float)row[RW_ATH], vol = (float)row[RW_V];
      float Gt[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) {
        const float dr = ar1 * r_hi[f * (TM + 1) * TJ] - ar0 * r_lo[f * (TM + 1) * TJ];
        const float dth = ath * (s_ft[f][tid] - t_lo[f * t_st]);
        Gt[f] = fma(S[f], vol, -((dr + dth) + dz[f]));
      }
      if (a.mode == MODE_OPER) {
        if (act) {
#pragma unroll
          for (int f = 0; f < NG; ++f)
            at_row((float*)a.out + (size_t)f * g.N + (size_t)k * plane + row0, jl) = Gt[f];
        }
      } else if (act) {
        // all loads before any store (the second stage updates in place)
        const float cdt = (float)(a.coef * dt * row[RW_INVV]);
        float nv[NG];
        double qn[NG];
#pragma unroll
        for (int f = 0; f < NG; ++f) qn[f] = upd[f];
#pragma unroll
        for (int f = 0; f < NG; ++f) {
          nv[f] = fma(cdt, Gt[f], base.e[f]);
          qn[f] += (double)nv[f];
          at_row((float*)a.out + (size_t)f * g.N + (size_t)k * plane + row0, jl) = nv[f];
        }
        // positivity of the new gas state; CFL of the new state (second stage)
        const double in2 = 1.0 / qn[4];
        const double un = qn[0] * in2, vn = qn[1] * in2, wn = qn[2] * in2;
        const double pn = (g.gamma - 1.0) * (qn[3] - 0.5 * (qn[0] * un + qn[1] * vn + qn[2] * wn));
        if (!(qn[4] > 0.0 && pn > 0.0)) {
          atomicOr(&a.c.ctrl->status, FL_NEG);
          atomicMin(&a.c.ctrl->first_bad, (unsigned long long)((size_t)k * plane + (size_t)ig * g.nth + jg));
          atomicCAS(&a.c.ctrl->bad_step, -1, a.step);
        } else if (a.second) {
          const double spd = sqrt(un * un + vn * vn + wn * wn) + sqrt(g.gamma * pn * in2);
          smax = fmax(smax, spd);
          if (EXT && g.drag_law) {
#pragma unroll
            for (int s2 = 0; s2 < ND; ++s2)
              tsmin = fmin(tsmin, 1.0 / inv_tstop<EXT>(g, s2, row[RW_OMK], qn[4], pn));
          }
        }
      }
      if (kk < k1) {
#pragma unroll
        for (int f = 0; f < NG; ++f) s_rm[f][tid] = r0[f];
      }
    }
    if (kk == k1) break;
    wave_order();
    const int k = kk;
    float (*pl)[TM + 4][HW] = s_pl[k & 1];
    const PertBg& face_c = bg_at(&s_face[k & 3][ti * PFD]);
    const PertBg& face_r = bg_at(&s_face[k & 3][(TM + ti + 1) * PFD]);
    const PertBg& face_z = bg_at(&s_face[k & 3][(2 * TM + 1 + ti) * PFD]);
    unsigned bad = 0;
    // ---- theta face j+1/2
    {
      auto get = [&](int c, int f) { return pl[f][ti + 2][tj + 1 + c]; };
      float F[NG];
      if (!face(DT(), get, nullptr, face_c, act, F)) bad |= 1;
#pragma unroll
      for (int f = 0; f < NG; ++f) s_ft[f][tid] = F[f];
    }
    // ---- r face i+1/2
    {
      auto get = [&](int c, int f) { return pl[f][ti + 1 + c][tj + 2]; };
      float F[NG];
      if (!face(DR(), get, s_wt[ti + 1], face_r, act, F)) bad |= 2;
#pragma unroll
      for (int f = 0; f < NG; ++f) s_fr[k & 1][f][ti + 1][tj] = F[f];
    }
    // ---- lower-edge faces of the tile: r face i0-1/2 (threads 0..63) and theta face
    //      j0-1/2 of each row (threads 64..71)
    if (tid < TJ) {
      auto get = [&](int c, int f) { return pl[f][c][tid + 2]; };
      float F[NG];
      // (the upper face of the tile below, which owns it, except at the inner boundary)
      if (!face(DR(), get, s_wt[0], bg_at(&s_face[k & 3][TM * PFD]),
                i0 == 0 && jg < g.nth, F))
        bad |= 4;
#pragma unroll
      for (int f = 0; f < NG; ++f) s_fr[k & 1][f][0][tid] = F[f];
    } else if (tid < TJ + TM) {
      const int row = tid - TJ;
      auto get = [&](int c, int f) { return pl[f][row + 2][c]; };
      float F[NG];
      if (!face(DT(), get, nullptr, bg_at(&s_face[k & 3][row * PFD]), false, F))
        bad |= 4;
#pragma unroll
      for (int f = 0; f < NG; ++f) s_fe[k & 1][f][row] = F[f];
    }
    // the next plane's halo and tables
    if (more) {
      if (halo_t) halo_store(k + 1, hraw);
      tab_store(k + 1, tab_next);
    }
    // the update's base of this cell and the dust its drag needs (raw stored values)
    if (a.mode == MODE_UPDATE && act) col_fetch((const float*)a.base, k, base);
    if (drag) {
      const size_t r = (size_t)k * plane + row0;
#pragma unroll
      for (int s2 = 0; s2 < ND; ++s2) {
        rds[s2] = at_row((const double*)a.in + p32_f64_base(g) + (size_t)s2 * g.N + r, jl);
#pragma unroll
        for (int c = 0; c < 3; ++c) vds[s2][c] = at_row(vin + (size_t)(5 + 3 * s2 + c) * g.N + r, jl);
      }
    }
    // ---- z face k+1/2
    float rn[NG], fzhi[NG];
    if (!twod) {
      col_form(k + 2, nraw, cen(k + 2, ti + 2), rn);
      auto get = [&](int c, int f) {
        return c == 0 ? s_rm[f][tid] : c == 1 ? pl[f][ti + 2][tj + 2] : c == 2 ? rp[f] : rn[f];
      };
      if (!face(DZ(), get, nullptr, face_z, act, fzhi)) bad |= 8;
    } else {
#pragma unroll
      for (int f = 0; f < NG; ++f) { rn[f] = 0.0f; fzhi[f] = 0.0f; }
    }
    // ---- the faces the short form did not take (rare), one call for all kinds: own theta and
    //      r face, tile edge, z face
    if (__builtin_expect(!wave_none(bad != 0), 0)) {
#pragma nounroll
      for (int kind = 0; kind < 4; ++kind) {
        if (!(bad >> kind & 1)) continue;
        const bool edge_r = kind == 2 && tid < TJ, along_th = kind == 0 || (kind == 2 && !edge_r);
        const int rr = kind == 0 ? ti + 2 : kind == 1 ? ti + 1 : edge_r ? 0 : tid - TJ + 2;
        const int cc = kind == 0 ? tj + 1 : along_th ? 0 : tj + 2;
        Face32 q;
#pragma unroll
        for (int f = 0; f < NG; ++f) {
          const float* p = &pl[f][rr][cc];
          const int st = along_th ? 1 : HW;
          if (kind == 3) {
            q.A[f] = s_rm[f][tid]; q.B[f] = pl[f][ti + 2][tj + 2]; q.C[f] = rp[f]; q.D[f] = rn[f];
          } else {
            q.A[f] = p[0]; q.B[f] = p[st]; q.C[f] = p[2 * st]; q.D[f] = p[3 * st];
          }
        }
        const int i = kind == 1 ? min(ig, g.nr) : kind == 2 ? (edge_r ? i0 - 1 : min(i0 + tid - TJ, g.nr - 1)) : igc;
        float F[NG];
        general(along_th ? 1 : kind == 3 ? 2 : 0, q, k, i,
                kind == 2 ? edge_r && i0 == 0 && jg < g.nth : act, F);
#pragma unroll
        for (int f = 0; f < NG; ++f) {
          if (kind == 0) s_ft[f][tid] = F[f];
          else if (kind == 1) s_fr[k & 1][f][ti + 1][tj] = F[f];
          else if (kind == 3) fzhi[f] = F[f];
          else if (edge_r) s_fr[k & 1][f][0][tid] = F[f];
          else s_fe[k & 1][f][tid - TJ] = F[f];
        }
      }
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) {
      dz[f] = (float)row[RW_AZ] * (fzhi[f] - fzlo[f]);
      fzlo[f] = fzhi[f];
      if (more) s_pl[(k + 1) & 1][f][ti + 2][tj + 2] = rp[f];
      rp[f] = rn[f];
    }
  }

  // ---- block reductions: counters, CFL partial, boundary outflow partial
  __syncthreads();
  const int wv = tid / 64, ln = tid & 63;
  const int mi = wave_imax(maxit);
  if (ln < 8 && s_nh[wv][ln])
    atomicAdd(&a.c.ctrl->newton_hist[ln], (unsigned long long)s_nh[wv][ln]);
  if (ln == 0 && mi) atomicMax(&a.c.ctrl->maxit, mi);
  if (tid == 0) {
    if (s_cnt.fall) atomicAdd(&a.c.ctrl->nfall, (unsigned long long)s_cnt.fall);
    if (s_cnt.vac) { atomicAdd(&a.c.ctrl->nvac, (unsigned long long)s_cnt.vac); atomicOr(&a.c.ctrl->status, FL_VAC); }
    if (s_cnt.resolve) atomicAdd(&a.c.ctrl->nresolve, (unsigned long long)s_cnt.resolve);
    if (s_cnt.noconv) { atomicOr(&a.c.ctrl->status, FL_NOCONV); atomicCAS(&a.c.ctrl->bad_step, -1, a.step); }
  }
  if (a.second && a.mode == MODE_UPDATE) {
    // the CFL bound of the thread's row decreases with the speed: the largest one's
    const double m = wave_min(smax > 0.0 ? g.cfl * rt[RT_V] / (smax * rt[RT_MAXA]) : 1e300);
    const double ls = wave_sum(ledger);
    const double tm = (EXT && ND > 0) ? wave_min(tsmin) : 1e300;
    if (ln == 0) { s_red[wv][0] = m; s_red[wv][1] = ls; s_red[wv][2] = tm; }
    __syncthreads();
    if (tid == 0) {
      double mm = s_red[0][0], lsum = s_red[0][1], tmm = s_red[0][2];
      for (int w2 = 1; w2 < NTM / 64; ++w2) {
        mm = fmin(mm, s_red[w2][0]);
        lsum += s_red[w2][1];
        tmm = fmin(tmm, s_red[w2][2]);
      }
      a.c.cflp[(size_t)blockIdx.x * 5] = mm;
      a.c.outp[(size_t)blockIdx.x * 5] = lsum;
      if (EXT && g.drag_law) a.c.tsp[blockIdx.x] = tmm;
    }
  }
}

// ------------------------------------------------------------------------------------
// standalone CFL of a state (start of a call) with the positivity check

template <int ND, bool P32>
__global__ void __launch_bounds__(256) k_cfl(StageArgs a, const void* state) {
  __shared__ double s_m[4];
  __shared__ double s_t[4];
  const Geo& g = a.g;
  double dtmin = 1e300, tsmin = 1e300;
  const double gm1 = g.gamma - 1.0;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < g.N;
       c += (size_t)gridDim.x * blockDim.x) {
    const size_t ki = c / g.nth;
    const int i = (int)(ki % g.nr);
    const double* bgc = a.t.bgc + ki * 5;
    const int k = (int)(ki / g.nr);
    double q[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) q[f] = bgc[f] + ld_cell<P32>(a, state, f, k, i, c);
    const double in2 = 1.0 / q[4];
    const double u = q[0] * in2, v = q[1] * in2, w = q[2] * in2;
    const double p = gm1 * (q[3] - 0.5 * (q[0] * u + q[1] * v + q[2] * w));
    if (!(q[4] > 0.0 && p > 0.0)) {
      atomicOr(&a.c.ctrl->status, FL_NEG);
      atomicMin(&a.c.ctrl->first_bad, (unsigned long long)c);
      atomicCAS(&a.c.ctrl->bad_step, -1, a.step);
      continue;
    }
    double spd = sqrt(u * u + v * v + w * w) + sqrt(g.gamma * p * in2);
#pragma unroll
    for (int s = 0; s < ND; ++s) {
      const int o = 5 + 4 * s;
      double rd = ld_cell<P32>(a, state, o + 3, k, i, c);
      if (rd > 0.0) {
        double id = 1.0 / rd;
        double a1 = ld_cell<P32>(a, state, o, k, i, c) * id;
        double a2 = ld_cell<P32>(a, state, o + 1, k, i, c) * id;
        double a3 = ld_cell<P32>(a, state, o + 2, k, i, c) * id;
        spd = fmax(spd, sqrt(a1 * a1 + a2 * a2 + a3 * a3));
      }
    }
    const double* rt = a.t.rt + (size_t)i * RT_N;
    dtmin = fmin(dtmin, g.cfl * rt[RT_V] / (spd * rt[RT_MAXA]));
    if (g.drag_law) {
#pragma unroll
      for (int s = 0; s < ND; ++s) tsmin = fmin(tsmin, 1.0 / inv_tstop(g, s, rt[RT_OMK], q[4], p));
    }
  }
  double m = wave_min(dtmin);
  double tm = wave_min(tsmin);
  if ((threadIdx.x & 63) == 0) { s_m[threadIdx.x / 64] = m; s_t[threadIdx.x / 64] = tm; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double mm = fmin(fmin(s_m[0], s_m[1]), fmin(s_m[2], s_m[3]));
    a.c.cflp[blockIdx.x] = mm;
    if (g.drag_law) a.c.tsp[blockIdx.x] = fmin(fmin(s_t[0], s_t[1]), fmin(s_t[2], s_t[3]));
  }
}

// ------------------------------------------------------------------------------------
// the drag alone over a part of the step, exactly (split integration of the Sect. 2.9
// forces for steps that may exceed the stopping times)
//
// With the densities and the stopping times of a cell held, the total momentum of each
// velocity component is constant and the dust-gas velocity differences d_s = u_s - u_g
// (species with rho_s > 0) obey dd/dt = B d, B_ab = -eps_b / t_b - [a == b] / t_a,
// eps_b = rho_b / rho_g, so d(tau) = exp(tau B) d(0).  exp(tau B) is taken by scaling
// and squaring: X = tau B / 2^s with |X| (largest absolute row sum) <= 1/8, the Taylor
// polynomial of degree 12 in Horner form (remainder below 1e-21), then s squarings; B's
// eigenvalues are negative, so the squarings do not amplify rounding.  New velocities:
// u_g = (P - sum rho_s d_s) / (rho_g + sum rho_s), u_s = u_g + d_s; the gas energy changes
// by the gas kinetic-energy change (the pressure is unchanged).

template <int ND>
__device__ __forceinline__ void mat_mul(const double* A, const double* B, double* C) {
#pragma unroll
  for (int r = 0; r < ND; ++r)
#pragma unroll
    for (int c = 0; c < ND; ++c) {
      double acc = 0.0;
#pragma unroll
      for (int m = 0; m < ND; ++m) acc = fma(A[r * ND + m], B[m * ND + c], acc);
      C[r * ND + c] = acc;
    }
}

template <int ND, bool P32>
__global__ void __launch_bounds__(256) k_drag(StageArgs a, void* state, double frac) {
  __shared__ int s_stop;
  if (threadIdx.x == 0) s_stop = __atomic_load_n(&a.c.ctrl->status, __ATOMIC_RELAXED);
  __syncthreads();
  if (s_stop & FL_HARD) return;
  const Geo& g = a.g;
  const double tau = frac * a.c.dtlog[a.dt_idx];
  const double gm1 = g.gamma - 1.0;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < g.N;
       c += (size_t)gridDim.x * blockDim.x) {
    const size_t ki = c / g.nth;
    const int i = (int)(ki % g.nr);
    const int k = (int)(ki / g.nr);
    const double* bgc = a.t.bgc + ki * 5;
    double q[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) q[f] = bgc[f] + ld_cell<P32>(a, state, f, k, i, c);
    const double rho = q[4], ir = 1.0 / rho;
    double ug[3] = {q[0] * ir, q[1] * ir, q[2] * ir};
    const double p = gm1 * (q[3] - 0.5 * (q[0] * ug[0] + q[1] * ug[1] + q[2] * ug[2]));
    const double omk = a.t.rt[(size_t)i * RT_N + RT_OMK];
    const double v0 = a.t.wc[ki * WB_N + WB_V];
    double rd[ND], ia[ND], ud[ND][3];
    double mtot = rho;
    bool any = false;
#pragma unroll
    for (int s = 0; s < ND; ++s) {
      const int o = 5 + 4 * s;
      rd[s] = ld_cell<P32>(a, state, o + 3, k, i, c);
      const bool on = rd[s] > 0.0;
      any = any || on;
      if constexpr (P32) {
        const float* vel = (const float*)state + (size_t)(5 + 3 * s) * g.N + c;
        ud[s][0] = (double)vel[0];
        ud[s][1] = v0 + (double)vel[g.N];
        ud[s][2] = (double)vel[2 * g.N];
      } else {
        const double id = on ? 1.0 / rd[s] : 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) ud[s][d] = ((const double*)state)[(size_t)(o + d) * g.N + c] * id;
      }
      ia[s] = on ? inv_tstop<true>(g, s, omk, rho, p) : 0.0;
      if (on) mtot += rd[s];
      else rd[s] = 0.0;
    }
    if (!any) continue;
    // exp(tau B)
    double X[ND * ND], M[ND * ND], T[ND * ND];
    double nrm = 0.0;
#pragma unroll
    for (int r = 0; r < ND; ++r) {
      double row = 0.0;
#pragma unroll
      for (int b = 0; b < ND; ++b) {
        X[r * ND + b] = -(rd[b] * ir) * ia[b] - (r == b ? ia[r] : 0.0);
        row += fabs(X[r * ND + b]);
      }
      nrm = fmax(nrm, row * tau);
    }
    int sq = 0;
    while (nrm > 0.125 && sq < 1100) { nrm *= 0.5; ++sq; }  // bounded for a non-finite norm
    const double sc = ldexp(tau, -sq);
#pragma unroll
    for (int e = 0; e < ND * ND; ++e) X[e] *= sc;
    // Horner: M = I + X/12, then M = I + (X/k) M for k = 11 .. 1
#pragma unroll
    for (int e = 0; e < ND * ND; ++e) M[e] = X[e] * (1.0 / 12.0) + ((e / ND) == (e % ND) ? 1.0 : 0.0);
#pragma unroll
    for (int kk = 11; kk >= 1; --kk) {
      mat_mul<ND>(X, M, T);
      const double ik = 1.0 / (double)kk;
#pragma unroll
      for (int e = 0; e < ND * ND; ++e) M[e] = fma(T[e], ik, (e / ND) == (e % ND) ? 1.0 : 0.0);
    }
    for (int r = 0; r < sq; ++r) {
      mat_mul<ND>(M, M, T);
#pragma unroll
      for (int e = 0; e < ND * ND; ++e) M[e] = T[e];
    }
    // relax each component
    double dke = 0.0;
    const double imt = 1.0 / mtot;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double P = q[d], d0[ND];
#pragma unroll
      for (int s = 0; s < ND; ++s) {
        P += rd[s] * ud[s][d];
        d0[s] = rd[s] > 0.0 ? ud[s][d] - ug[d] : 0.0;
      }
      double pd = 0.0, d1[ND];
#pragma unroll
      for (int s = 0; s < ND; ++s) {
        double acc = 0.0;
#pragma unroll
        for (int b = 0; b < ND; ++b) acc = fma(M[s * ND + b], d0[b], acc);
        d1[s] = acc;
        pd += rd[s] * acc;
      }
      const double ug1 = (P - pd) * imt;
      dke += 0.5 * rho * (ug1 * ug1 - ug[d] * ug[d]);
      st_cell<P32>(a, state, d, k, i, c, rho * ug1 - bgc[d]);
#pragma unroll
      for (int s = 0; s < ND; ++s) {
        if (!(rd[s] > 0.0)) continue;
        if constexpr (P32) {
          const double u1 = ug1 + d1[s] - (d == 1 ? v0 : 0.0);
          ((float*)state)[(size_t)(5 + 3 * s + d) * g.N + c] = (float)u1;
        } else {
          ((double*)state)[(size_t)(5 + 4 * s + d) * g.N + c] = rd[s] * (ug1 + d1[s]);
        }
      }
    }
    st_cell<P32>(a, state, 3, k, i, c, q[3] + dke - bgc[3]);
  }
}

// final reduction after a step: next dt (CFL), stiffness check, boundary outflow ledger
__global__ void __launch_bounds__(256) k_reduce(StageArgs a, int nparts, int nparts_dust, int dt_next,
                                                int want_dt, int want_ledger) {
  __shared__ double s_m[4];
  __shared__ double s_ts[4];
  __shared__ double s_l[4][5];
  __shared__ int s_stop;
  if (threadIdx.x == 0) s_stop = __atomic_load_n(&a.c.ctrl->status, __ATOMIC_RELAXED);
  __syncthreads();
  if (s_stop & FL_HARD) return;
  double m = 1e300, tsm = 1e300;
  double l[5] = {0, 0, 0, 0, 0};
  const bool dyn_ts = a.g.drag_law && a.g.nd > 0;
  // fixed partition and order: deterministic sums
  // stage partials: [block][5] (gas, dust species); standalone CFL: [nparts]
  const int stride = want_ledger ? 5 : 1;
  for (int b = threadIdx.x; b < nparts; b += blockDim.x) {
    if (dyn_ts) tsm = fmin(tsm, a.c.tsp[b]);
    if (want_dt) m = fmin(m, a.c.cflp[(size_t)b * stride]);
    if (want_ledger) l[0] += a.c.outp[(size_t)b * 5];
  }
  if (want_ledger)
    for (int b = threadIdx.x; b < nparts_dust; b += blockDim.x)
#pragma unroll
      for (int s = 1; s < 5; ++s)
        if (s <= a.g.nd) {
          if (want_dt) m = fmin(m, a.c.cflp[(size_t)b * 5 + s]);
          l[s] += a.c.outp[(size_t)b * 5 + s];
        }
  m = wave_min(m);
  tsm = wave_min(tsm);
#pragma unroll
  for (int s = 0; s < 5; ++s) l[s] = wave_sum(l[s]);
  if ((threadIdx.x & 63) == 0) {
    s_m[threadIdx.x / 64] = m;
    s_ts[threadIdx.x / 64] = tsm;
#pragma unroll
    for (int s = 0; s < 5; ++s) s_l[threadIdx.x / 64][s] = l[s];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (want_dt) {
      double mm = fmin(fmin(s_m[0], s_m[1]), fmin(s_m[2], s_m[3]));
      a.c.dtlog[dt_next] = mm;
    }
    if (want_ledger)
#pragma unroll
      for (int s = 0; s < 5; ++s)
        a.c.ctrl->outflow[s] = ((s_l[0][s] + s_l[1][s]) + (s_l[2][s] + s_l[3][s]));
    double dtn = a.c.dtlog[dt_next];
    // stiffness: dt against the smallest stopping time (constant law: from the tables;
    // law 1: over the cells of the state the step starts from)
    const double tsmin = dyn_ts ? fmin(fmin(s_ts[0], s_ts[1]), fmin(s_ts[2], s_ts[3]))
                                : a.c.ctrl->min_ts;
    if (a.g.nd > 0 && !a.g.drag_exact && dtn >= tsmin) {
      atomicOr(&a.c.ctrl->status, FL_STIFF);
      // dt_next 0: the first step of the call (a.step); else the step after a.step
      atomicCAS(&a.c.ctrl->bad_step, -1, dt_next == 0 ? a.step : a.step + 1);
    }
  }
}

// ------------------------------------------------------------------------------------
// tables and initial state (device side of the initialisation)

struct EqPoint {
  double rho, P, v;
};

// Stationary flow (App. A): rho0 = rho_mid(r) exp[(GM/c^2)(1/s - 1/r)], P0 = c^2 rho0 with
// the isothermal c^2 = h0^2 GM r^beta_T, and the azimuthal velocity from the radial
// balance, v^2 = GM/r + c^2 (beta_T + beta_rho) + beta_T GM (1/r - 1/s) (the analytic
// pressure gradient folded in).
__device__ EqPoint eq_point(const rb_config& c, double r, double z) {
  EqPoint e;
  const double c2 = c.h0 * c.h0 * c.GM * pow(r, c.beta_T);
  const double s = sqrt(r * r + z * z);
  const double invs = 1.0 / s, invr = 1.0 / r;
  e.rho = c.rho_mid0 * pow(r, c.beta_rho) * exp(c.GM / c2 * (invs - invr));
  e.P = c2 * e.rho;
  e.v = sqrt(c.GM * invr + c2 * (c.beta_T + c.beta_rho) + c.beta_T * c.GM * (invr - invs));
  return e;
}

__device__ void gas_cons(double g, double rho, double u, double v, double P, double* q) {
  q[0] = rho * u;
  q[1] = rho * v;
  q[2] = 0.0;
  q[3] = P / (g - 1.0) + 0.5 * rho * (u * u + v * v);
  q[4] = rho;
}

// Primitive variables of a conservative gas state q as a WB_N table entry: velocity,
// pressure, density, sound speed, E + P, 1/rho.  Zero for the Sod annulus (its split has
// no stationary reference).
__device__ void prim_entry(const rb_config& c, const double* q, double* o) {
  if (c.init_kind != RB_INIT_DISC) {
    for (int s = 0; s < WB_N; ++s) o[s] = 0.0;
    return;
  }
  const double rho = q[4];
  o[WB_U] = q[0] / rho;
  o[WB_V] = q[1] / rho;
  o[WB_W] = q[2] / rho;
  o[WB_P] = (c.gamma - 1.0) * (q[3] - 0.5 * (q[0] * o[WB_U] + q[1] * o[WB_V] + q[2] * o[WB_W]));
  o[WB_RHO] = rho;
  o[WB_C] = sqrt(c.gamma * o[WB_P] / rho);
  o[WB_H] = q[3] + o[WB_P];
  o[WB_IRHO] = 1.0 / rho;
}

// PertBg entry of the FP32-perturbation form from a WB_N entry.
__device__ void pert_entry(const double* b, double* out) {
  *(PertBg*)out = {{b[WB_RHO], (float)b[WB_V], (float)(b[WB_V] * b[WB_V])},
                   b[WB_P], (float)b[WB_C], (float)b[WB_H], (float)(b[WB_RHO] * b[WB_V]), 0.0f};
}

// Reconstructed variables of a ghost cell whose full state is q (nf fields): the gas
// deviation W(q) - W0 (zero on a disc, whose ghosts hold the stationary flow; the
// state's own primitives for the Sod annulus), and each dust fluid's velocity (zero
// where it is empty) and density.
__device__ void ghost_recon(const rb_config& c, int nf, const double* q, double* o) {
  if (c.init_kind == RB_INIT_DISC) {
    for (int f = 0; f < 5; ++f) o[f] = 0.0;
  } else {
    const double rho = q[4];
    const double u = q[0] / rho, v = q[1] / rho, w = q[2] / rho;
    o[0] = u; o[1] = v; o[2] = w;
    o[3] = (c.gamma - 1.0) * (q[3] - 0.5 * (q[0] * u + q[1] * v + q[2] * w));
    o[4] = rho;
  }
  for (int b = 5; b < nf; b += 4) {
    const double rd = q[b + 3];
    for (int m = 0; m < 3; ++m) o[b + m] = rd > 0.0 ? q[b + m] / rd : 0.0;
    o[b + 3] = rd;
  }
}

// initial dust layer of species s: eps (H/H_d) rho_mid(r) exp(-z^2 / 2 H_d^2)
__device__ double dust_layer(const rb_config& c, int s, double r, double z) {
  const double c2 = c.h0 * c.h0 * c.GM * pow(r, c.beta_T);
  const double H = sqrt(c2) / sqrt(c.GM / (r * r * r));
  const double Hd = c.hd_over_h[s] * H;
  return c.eps_dust[s] / c.hd_over_h[s] * c.rho_mid0 * pow(r, c.beta_rho) *
         exp(-(z * z) / (2.0 * Hd * Hd));
}

// full stationary state (gas + dust layer moving with the gas) at (r, z); Sod: the
// initial state at radius r
__device__ void background_full(const InitArgs& a, double r, double z, double* q) {
  const rb_config& c = a.cfg;
  if (c.init_kind == RB_INIT_SOD) {
    const double* s = r < c.sod_r0 ? c.sod_left : c.sod_right;
    gas_cons(c.gamma, s[0], s[2], 0.0, s[1], q);
    return;
  }
  EqPoint e = eq_point(c, r, z);
  gas_cons(c.gamma, e.rho, 0.0, e.v, e.P, q);
  for (int s = 0; s < c.n_dust; ++s) {
    double rd = dust_layer(c, s, r, z);
    q[5 + 4 * s + 0] = 0.0;
    q[5 + 4 * s + 1] = rd * e.v;
    q[5 + 4 * s + 2] = 0.0;
    q[5 + 4 * s + 3] = rd;
  }
}

__device__ __forceinline__ double face_r(const rb_config& c, int i) {
  if (c.log_r) return c.r_in * pow(c.r_out / c.r_in, (double)i / c.nr);
  return c.r_in + i * ((c.r_out - c.r_in) / c.nr);
}
__device__ __forceinline__ double cell_r(const rb_config& c, int i) {
  return 0.5 * (face_r(c, i) + face_r(c, i + 1));
}

// radial tables: one block
__global__ void __launch_bounds__(256) k_tables_r(InitArgs a) {
  const rb_config& c = a.cfg;
  const Layout& L = a.L;
  double* w = a.work;
  const int nr = c.nr;
  const bool twod = c.nz == 1;
  const double dth = 2.0 * M_PI / c.ntheta;
  const double dz = twod ? 1.0 : 2.0 * c.z_half / c.nz;
  for (int i = threadIdx.x; i < nr + 4; i += blockDim.x) w[L.rcell + i] = cell_r(c, i - 2);
  for (int i = threadIdx.x; i <= nr; i += blockDim.x) w[L.rface + i] = face_r(c, i);
  for (int k = threadIdx.x; k < c.nz; k += blockDim.x)
    w[L.zc + k] = twod ? 0.0 : (k + 0.5 - 0.5 * c.nz) * dz;
  for (int j = threadIdx.x; j < c.ntheta; j += blockDim.x) {
    const double th = (j + 0.5) * dth;
    w[L.trig + j] = cos(th);
    w[L.trig + c.ntheta + j] = sin(th);
  }
  for (int i = threadIdx.x; i <= nr; i += blockDim.x) w[L.ar + i] = face_r(c, i) * dth * dz;
  for (int i = threadIdx.x; i < nr; i += blockDim.x) {
    double rm = face_r(c, i), rp = face_r(c, i + 1);
    double* rt = w + L.rt + (size_t)i * RT_N;
    double area = 0.5 * (rp * rp - rm * rm);
    rt[RT_V] = area * dth * dz;
    rt[RT_INVV] = 1.0 / rt[RT_V];
    rt[RT_ATH] = (rp - rm) * dz;
    rt[RT_AZ] = area * dth;
    double rc = 0.5 * (rm + rp);
    rt[RT_RC] = rc;
    rt[RT_INVRC] = 1.0 / rc;
    rt[RT_OMK] = sqrt(c.GM / (rc * rc * rc));
    double amax = fmax(fmax(rm * dth * dz, rp * dth * dz), rt[RT_ATH]);
    if (!twod) amax = fmax(amax, rt[RT_AZ]);
    rt[RT_MAXA] = amax;
  }
  // parabola weights and limiter bounds along r for cells -1..nr (Sect. 2.7)
  for (int cI = threadIdx.x; cI < nr + 2; cI += blockDim.x) {
    int cc = cI - 1;
    double xm = cell_r(c, cc - 1), x0 = cell_r(c, cc), xp = cell_r(c, cc + 1);
    double hm = x0 - xm, hp = xp - x0, sum = hm + hp;
    double* co = w + L.rco + (size_t)cI * RC_N;
    double d = face_r(c, cc + 1) - x0;
    co[RC_WPP] = (d * d + hm * d) / (hp * sum);
    co[RC_WPM] = (hp * d - d * d) / (hm * sum);
    co[RC_LPM] = 2.0 * d / hm;
    co[RC_LPP] = 2.0 * d / hp;
    d = face_r(c, cc) - x0;
    co[RC_WMP] = (d * d + hm * d) / (hp * sum);
    co[RC_WMM] = (hp * d - d * d) / (hm * sum);
    co[RC_LMM] = 2.0 * d / hm;
    co[RC_LMP] = 2.0 * d / hp;
    if (a.g.p32)
      for (int q = 0; q < RC_N; ++q) ((float*)(w + L.rcf))[(size_t)cI * RC_N + q] = (float)co[q];
  }
  if (threadIdx.x == 0) {
    Ctrl* ct = reinterpret_cast<Ctrl*>(w + L.ctrl);
    double mts = 1e300;
    for (int s = 0; s < c.n_dust && c.drag_law == 0; ++s)
      for (int i = 0; i < nr; ++i) {
        double rc = cell_r(c, i);
        mts = fmin(mts, c.stokes[s] / sqrt(c.GM / (rc * rc * rc)));
      }
    ct->min_ts = mts;
  }
}

// 2D tables over (k, i) including two ghost layers in each direction
__global__ void __launch_bounds__(256) k_tables_2d(InitArgs a) {
  const rb_config& c = a.cfg;
  const Layout& L = a.L;
  double* w = a.work;
  const int nr = c.nr, nz = c.nz, nf = a.g.nf;
  const bool twod = nz == 1;
  const double dz = twod ? 1.0 : 2.0 * c.z_half / nz;
  const int W = nr + 4, H = nz + 4;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < W * H; t += gridDim.x * blockDim.x) {
    const int ii = t % W - 2, kk = t / W - 2;
    const double zc = twod ? 0.0 : (kk + 0.5 - 0.5 * nz) * dz;
    double q[MAXF];
    const bool kin = kk >= 0 && kk < nz, iin = ii >= 0 && ii < nr;
    if (kin && iin) {
      // indirect-gravity weight V r / (r^2 + z^2)^(3/2) of the cell
      const double rm = face_r(c, ii), rp = face_r(c, ii + 1), rc = cell_r(c, ii);
      const double V = 0.5 * (rp * rp - rm * rm) * (2.0 * M_PI / c.ntheta) * dz;
      const double s2 = rc * rc + zc * zc;
      w[L.indw + (size_t)kk * nr + ii] = V * rc / (s2 * sqrt(s2));
      // boundary damping zones: rate R / tau, R the squared fraction of the way from the
      // zone edge to the boundary, tau = damp_tau orbital periods
      double rate = 0.0;
      if (c.bc_r == 1) {
        const double e_in = c.damp_r_in * c.r_in, e_out = c.damp_r_out * c.r_out;
        if (rc < e_in) {
          const double x = (e_in - rc) / (e_in - c.r_in);
          rate += x * x * sqrt(c.GM / (c.r_in * c.r_in * c.r_in)) / (2.0 * M_PI * c.damp_tau);
        }
        if (rc > e_out) {
          const double x = (rc - e_out) / (c.r_out - e_out);
          rate += x * x * sqrt(c.GM / (c.r_out * c.r_out * c.r_out)) / (2.0 * M_PI * c.damp_tau);
        }
      }
      if (c.bc_z == 2 && !twod) {
        const double e_z = c.damp_z * c.z_half, az = fabs(zc);
        if (az > e_z) {
          const double x = (az - e_z) / (c.z_half - e_z);
          rate += x * x * sqrt(c.GM / (rc * rc * rc)) / (2.0 * M_PI * c.damp_tau);
        }
      }
      w[L.damp + (size_t)kk * nr + ii] = rate;
    }
    if (kin && iin) {
      const double r = cell_r(c, ii);
      background_full(a, r, zc, q);
      for (int f = 0; f < 5; ++f) w[L.bgc + ((size_t)kk * nr + ii) * 5 + f] =
          c.init_kind == RB_INIT_DISC ? q[f] : 0.0;
      double* o = w + L.wc + ((size_t)kk * nr + ii) * WB_N;
      prim_entry(c, q, o);
      if (a.g.p32) pert_entry(o, w + L.pc + ((size_t)kk * nr + ii) * PF_D);
      double s3 = pow(r * r + zc * zc, 1.5);
      w[L.grav + ((size_t)kk * nr + ii) * 2 + 0] = -c.GM * r / s3;
      w[L.grav + ((size_t)kk * nr + ii) * 2 + 1] = -c.GM * zc / s3;
    }
    if (kin && ii >= 0 && ii <= nr) {
      background_full(a, face_r(c, ii), zc, q);
      for (int f = 0; f < 5; ++f) w[L.bgr + ((size_t)kk * (nr + 1) + ii) * 5 + f] =
          c.init_kind == RB_INIT_DISC ? q[f] : 0.0;
      double* o = w + L.wr + ((size_t)kk * (nr + 1) + ii) * WB_N;
      prim_entry(c, q, o);
      if (a.g.p32) pert_entry(o, w + L.pr + ((size_t)kk * (nr + 1) + ii) * PF_D);
    }
    if (!twod && iin && kk >= 0 && kk <= nz) {
      background_full(a, cell_r(c, ii), (kk - 0.5 * nz) * dz, q);
      for (int f = 0; f < 5; ++f) w[L.bgz + ((size_t)kk * nr + ii) * 5 + f] =
          c.init_kind == RB_INIT_DISC ? q[f] : 0.0;
      double* o = w + L.wz + ((size_t)kk * nr + ii) * WB_N;
      prim_entry(c, q, o);
      if (a.g.p32) pert_entry(o, w + L.pz + ((size_t)kk * nr + ii) * PF_D);
    }
    // ghost cells: reconstructed variables (gas W', dust primitives) and the stationary
    // flow's primitives
    if (kin && !iin && ii >= -2 && ii <= nr + 1) {
      const int side = ii < 0 ? 0 : 1, layer = ii < 0 ? -1 - ii : ii - nr;
      background_full(a, cell_r(c, ii), zc, q);
      ghost_recon(c, nf, q, w + L.ghr + ((size_t)(side * 2 + layer) * nz + kk) * nf);
      prim_entry(c, q, w + L.ghrw + ((size_t)(side * 2 + layer) * nz + kk) * WB_N);
    }
    if (!twod && iin && !kin && kk >= -2 && kk <= nz + 1) {
      const int side = kk < 0 ? 0 : 1, layer = kk < 0 ? -1 - kk : kk - nz;
      background_full(a, cell_r(c, ii), zc, q);
      ghost_recon(c, nf, q, w + L.ghz + ((size_t)(side * 2 + layer) * nr + ii) * nf);
      prim_entry(c, q, w + L.ghzw + ((size_t)(side * 2 + layer) * nr + ii) * WB_N);
      // outflow ghosts: stationary density of the ghost over that of the boundary cell
      const double rho_g = q[4];
      background_full(a, cell_r(c, ii), (side == 0 ? 0.5 - 0.5 * nz : nz - 0.5 - 0.5 * nz) * dz, q);
      w[L.ozr + (size_t)(side * 2 + layer) * nr + ii] = rho_g / q[4];
    }
  }
}

// store of the initial state: FP64, or the FP32 layout (dust velocity components given
// directly through dust_vel, stored as deviations from the stationary flow's velocity)
__device__ __forceinline__ void store_init(const InitArgs& a, int f, int k, int i, size_t cl,
                                           double v, double dust_vel = 0.0) {
  const Geo& g = a.g;
  if (g.p32) {
    if (f < 5) { ((float*)a.state)[(size_t)f * g.N + cl] = (float)v; return; }
    const int sp = (f - 5) >> 2, c = (f - 5) & 3;
    if (c == 3) { ((double*)a.state)[p32_f64_base(g) + (size_t)sp * g.N + cl] = v; return; }
    const double u0 = c == 1 ? a.work[a.L.wc + ((size_t)k * g.nr + i) * WB_N + WB_V] : 0.0;
    ((float*)a.state)[(size_t)(5 + 3 * sp + c) * g.N + cl] = (float)(dust_vel - u0);
  } else {
    ((double*)a.state)[(size_t)f * g.N + cl] = v;
  }
}

// Initial state: Sod annulus, or the disc with the column Gaussian vortex (streamfunction
// psi = psi0 exp(-X^2/2 sr^2 - Y^2/2 sa^2), X = r - r_v, Y = r_v wrap(theta - theta_v),
// centre vorticity 2 Ro Omega_K(r_v) with Ro = -amplitude), density noise
// rho0 (1 + a xi) at unchanged pressure, the same on each dust layer from its own noise
// field, dust moving with the gas.  Stored as E' (gas) and whole variables (dust).
__global__ void __launch_bounds__(256) k_init_state(InitArgs a) {
  const rb_config& c = a.cfg;
  const Geo& g = a.g;
  const int nr = c.nr, nth = c.ntheta, nz = c.nz;
  const bool twod = nz == 1;
  const double dz = twod ? 1.0 : 2.0 * c.z_half / nz;
  const double dth = 2.0 * M_PI / nth;
  for (size_t cl = (size_t)blockIdx.x * blockDim.x + threadIdx.x; cl < g.N;
       cl += (size_t)gridDim.x * blockDim.x) {
    const int j = (int)(cl % nth);
    const int i = (int)((cl / nth) % nr);
    const int k = (int)(cl / ((size_t)nth * nr));
    const double r = cell_r(c, i);
    const double z = twod ? 0.0 : (k + 0.5 - 0.5 * nz) * dz;
    double q[MAXF];
    if (c.init_kind == RB_INIT_SOD) {
      background_full(a, r, z, q);
      for (int f = 0; f < 5; ++f) store_init(a, f, k, i, cl, q[f]);
      continue;
    }
    EqPoint e = eq_point(c, r, z);
    double q0[5];
    gas_cons(c.gamma, e.rho, 0.0, e.v, e.P, q0);
    const double A = a.amp ? a.amp[cl] : c.vortex_amp;
    const double rv = c.vortex_r0, sr = c.vortex_sig_r, sa = c.vortex_sig_a;
    const double X = r - rv;
    double d = (j + 0.5) * dth - c.vortex_th0;
    d -= 2.0 * M_PI * floor((d + M_PI) / (2.0 * M_PI));
    const double Y = rv * d;
    const double Om = sqrt(c.GM / (rv * rv * rv));
    const double psi = -2.0 * Om / (1.0 / (sr * sr) + 1.0 / (sa * sa)) *
                       exp(-X * X / (2.0 * sr * sr) - Y * Y / (2.0 * sa * sa));
    // Rossby-wave-instability seed (Sect. 4.3): density bump B at unchanged temperature,
    // rotation from the radial balance with the bump's pressure gradient
    // (v^2 = v0^2 + r c_iso^2 B'/B, c_iso^2 = P0/rho0), m-mode radial velocity
    double B = 1.0, vr = 0.0, vt = e.v;
    if (c.rwi_delta != 0.0 || c.rwi_eps != 0.0) {
      const double x = r - c.rwi_r0, w2 = c.rwi_dr * c.rwi_dr;
      const double gx = exp(-0.5 * x * x / w2);
      B = 1.0 + c.rwi_delta * gx;
      vt = sqrt(e.v * e.v - r * (e.P / e.rho) * (c.rwi_delta * gx * x / w2) / B);
      vr = c.rwi_eps * e.v * sin(c.rwi_m * ((j + 0.5) * dth)) * gx;
    }
    const double u = A * (-psi * rv * Y / (r * sa * sa)) + vr;
    const double v = vt + A * (psi * X / (sr * sr));
    const double xi = a.noise ? a.noise[cl] : 0.0;
    const double rho = e.rho * B * (1.0 + c.noise_amp * xi);
    gas_cons(c.gamma, rho, u, v, e.P * B, q);
    for (int f = 0; f < 5; ++f) store_init(a, f, k, i, cl, q[f] - q0[f]);
    for (int s = 0; s < c.n_dust; ++s) {
      const double xd = a.noise ? a.noise[(size_t)(1 + s) * g.N + cl] : 0.0;
      const double rd = dust_layer(c, s, r, z) * (1.0 + c.noise_amp * xd);
      const int o = 5 + 4 * s;
      store_init(a, o + 0, k, i, cl, rd * u, u);
      store_init(a, o + 1, k, i, cl, rd * v, v);
      store_init(a, o + 2, k, i, cl, 0.0, 0.0);
      store_init(a, o + 3, k, i, cl, rd);
    }
  }
}

// Derivative of the initial state with respect to the per-cell vortex amplitude A,
// contracted with a state cotangent lam: u = A u_hat, v = v0 + A v_hat, so
// d(rho u, rho v, 0, E, rho)/dA = (rho u_hat, rho v_hat, 0, rho (u u_hat + v v_hat), 0)
// and d(rho_d u, rho_d v, 0, rho_d)/dA = (rho_d u_hat, rho_d v_hat, 0, 0).
__global__ void __launch_bounds__(256) k_amp_grad(InitArgs a, const double* lam, double* out) {
  const rb_config& c = a.cfg;
  const Geo& g = a.g;
  const int nr = c.nr, nth = c.ntheta, nz = c.nz;
  const bool twod = nz == 1;
  const double dz = twod ? 1.0 : 2.0 * c.z_half / nz;
  const double dth = 2.0 * M_PI / nth;
  for (size_t cl = (size_t)blockIdx.x * blockDim.x + threadIdx.x; cl < g.N;
       cl += (size_t)gridDim.x * blockDim.x) {
    const int j = (int)(cl % nth);
    const int i = (int)((cl / nth) % nr);
    const int k = (int)(cl / ((size_t)nth * nr));
    const double r = cell_r(c, i);
    const double z = twod ? 0.0 : (k + 0.5 - 0.5 * nz) * dz;
    EqPoint e = eq_point(c, r, z);
    const double A = a.amp ? a.amp[cl] : c.vortex_amp;
    const double rv = c.vortex_r0, sr = c.vortex_sig_r, sa = c.vortex_sig_a;
    const double X = r - rv;
    double d = (j + 0.5) * dth - c.vortex_th0;
    d -= 2.0 * M_PI * floor((d + M_PI) / (2.0 * M_PI));
    const double Y = rv * d;
    const double Om = sqrt(c.GM / (rv * rv * rv));
    const double psi = -2.0 * Om / (1.0 / (sr * sr) + 1.0 / (sa * sa)) *
                       exp(-X * X / (2.0 * sr * sr) - Y * Y / (2.0 * sa * sa));
    const double uh = -psi * rv * Y / (r * sa * sa);
    const double vh = psi * X / (sr * sr);
    const double u = A * uh;
    const double v = e.v + A * vh;
    const double xi = a.noise ? a.noise[cl] : 0.0;
    const double rho = e.rho * (1.0 + c.noise_amp * xi);
    double acc = lam[0 * g.N + cl] * rho * uh + lam[1 * g.N + cl] * rho * vh +
                 lam[3 * g.N + cl] * rho * (u * uh + v * vh);
    for (int s = 0; s < c.n_dust; ++s) {
      const double xd = a.noise ? a.noise[(size_t)(1 + s) * g.N + cl] : 0.0;
      const double rd = dust_layer(c, s, r, z) * (1.0 + c.noise_amp * xd);
      const int o = 5 + 4 * s;
      acc += lam[(size_t)(o + 0) * g.N + cl] * rd * uh + lam[(size_t)(o + 1) * g.N + cl] * rd * vh;
    }
    out[cl] = acc;
  }
}

// ------------------------------------------------------------------------------------
// conversions and reductions

// a fresh control block (no flags, no bad cell), for calls whose control block is not
// the context's
__global__ void k_ctrl_init(Ctrl* c) {
  if (threadIdx.x == 0) {
    c->status = 0;
    c->bad_step = -1;
    c->maxit = 0;
    c->first_bad = ~0ull;
    c->nfall = 0;
    c->nvac = 0;
    c->nresolve = 0;
    for (int b = 0; b < 8; ++b) c->newton_hist[b] = 0;
    c->nnegd = 0;
    c->min_ts = 1e300;
  }
}

// the reduced CFL step to the caller's slot, or zero when the state had a cell with a
// non-positive density or pressure
__global__ void k_cfl_out(const Ctrl* c, const double* dt, double* out) {
  if (threadIdx.x == 0) out[0] = (c->status & FL_NEG) ? 0.0 : dt[0];
}

__global__ void k_fill(double* p, size_t n, double v) {
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
       q += (size_t)gridDim.x * blockDim.x)
    p[q] = v;
}

// field f of the state -> full FP64 values (gas: E0 + E'; dust: momenta, densities)
template <bool P32>
__global__ void k_to_full(StageArgs a, const void* state, double* out, int f) {
  const Geo& g = a.g;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < g.N;
       c += (size_t)gridDim.x * blockDim.x) {
    const size_t ki = c / g.nth;
    double v = ld_cell<P32>(a, state, f, (int)(ki / g.nr), (int)(ki % g.nr), c);
    if (f < 5) v += a.t.bgc[ki * 5 + f];
    out[c] = v;
  }
}
template <bool P32>
__global__ void k_from_full(StageArgs a, const double* in, void* state, int f) {
  const Geo& g = a.g;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < g.N;
       c += (size_t)gridDim.x * blockDim.x) {
    const size_t ki = c / g.nth;
    double v = in[c];
    if (f < 5) v -= a.t.bgc[ki * 5 + f];
    st_cell<P32>(a, state, f, (int)(ki / g.nr), (int)(ki % g.nr), c, v);
  }
}

// mass of field f (density slot): per-block partial sums of rho V over fixed chunks,
// each summed by a fixed tree (deterministic, FP64)
template <bool P32>
__global__ void __launch_bounds__(256) k_mass(StageArgs a, const void* state, double* part, int f) {
  __shared__ double s_s[4];
  const Geo& g = a.g;
  const size_t chunk = (g.N + gridDim.x - 1) / gridDim.x;
  const size_t c0 = (size_t)blockIdx.x * chunk, c1 = min(g.N, c0 + chunk);
  double acc = 0.0;
  for (size_t c = c0 + threadIdx.x; c < c1; c += blockDim.x) {
    const size_t ki = c / g.nth;
    const int i = (int)(ki % g.nr);
    double v = ld_cell<P32>(a, state, f, (int)(ki / g.nr), i, c);
    if (f < 5) v += a.t.bgc[ki * 5 + f];
    acc += v * a.t.rt[(size_t)i * RT_N + RT_V];
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) s_s[threadIdx.x / 64] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (s_s[0] + s_s[1]) + (s_s[2] + s_s[3]);
}

// Indirect-gravity sums A = sum m w cos(theta), B = sum m w sin(theta) over the cells,
// m = gas + dust density, w = V r / (r^2 + z^2)^(3/2): per-block partials over fixed
// chunks, then one block adds them in a fixed order (deterministic, FP64).
template <bool P32>
__global__ void __launch_bounds__(256) k_indirect(StageArgs a, const void* state, double* part) {
  __shared__ double s_s[2][4];
  const Geo& g = a.g;
  const size_t chunk = (g.N + gridDim.x - 1) / gridDim.x;
  const size_t c0 = (size_t)blockIdx.x * chunk, c1 = min(g.N, c0 + chunk);
  double sa = 0.0, sb = 0.0;
  for (size_t c = c0 + threadIdx.x; c < c1; c += blockDim.x) {
    const size_t ki = c / g.nth;
    const int j = (int)(c % g.nth), i = (int)(ki % g.nr), k = (int)(ki / g.nr);
    double m = a.t.bgc[ki * 5 + 4] + ld_cell<P32>(a, state, 4, k, i, c);
    for (int s = 0; s < g.nd; ++s) m += ld_cell<P32>(a, state, 5 + 4 * s + 3, k, i, c);
    const double mw = m * a.t.indw[ki];
    sa += mw * a.t.trig[j];
    sb += mw * a.t.trig[g.nth + j];
  }
  sa = wave_sum(sa);
  sb = wave_sum(sb);
  if ((threadIdx.x & 63) == 0) { s_s[0][threadIdx.x / 64] = sa; s_s[1][threadIdx.x / 64] = sb; }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = (s_s[0][0] + s_s[0][1]) + (s_s[0][2] + s_s[0][3]);
    part[2 * blockIdx.x + 1] = (s_s[1][0] + s_s[1][1]) + (s_s[1][2] + s_s[1][3]);
  }
}

__global__ void __launch_bounds__(256) k_indirect_final(const double* part, int n, double* ab) {
  __shared__ double s_s[2][4];
  double sa = 0.0, sb = 0.0;
  for (int b = threadIdx.x; b < n; b += blockDim.x) { sa += part[2 * b]; sb += part[2 * b + 1]; }
  sa = wave_sum(sa);
  sb = wave_sum(sb);
  if ((threadIdx.x & 63) == 0) { s_s[0][threadIdx.x / 64] = sa; s_s[1][threadIdx.x / 64] = sb; }
  __syncthreads();
  if (threadIdx.x == 0) {
    ab[0] = (s_s[0][0] + s_s[0][1]) + (s_s[0][2] + s_s[0][3]);
    ab[1] = (s_s[1][0] + s_s[1][1]) + (s_s[1][2] + s_s[1][3]);
  }
}

__global__ void __launch_bounds__(256) k_sum(const double* part, int n, double* out) {
  __shared__ double s_s[4];
  double acc = 0.0;
  for (int b = threadIdx.x; b < n; b += blockDim.x) acc += part[b];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) s_s[threadIdx.x / 64] = acc;
  __syncthreads();
  if (threadIdx.x == 0) *out = (s_s[0] + s_s[1]) + (s_s[2] + s_s[3]);
}

// ------------------------------------------------------------------------------------
// launchers

hipError_t launch_tables(const InitArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_tables_r, dim3(1), dim3(256), 0, s, a);
  const int cells = (a.cfg.nr + 4) * (a.cfg.nz + 4);
  const int blocks = (cells + 255) / 256;
  hipLaunchKernelGGL(k_tables_2d, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_init_state(const InitArgs& a, hipStream_t s) {
  const int blocks = (int)std::min<size_t>((a.g.N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_init_state, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

// the optional physics (indirect gravity, drag law 1) and boundary options (damping zones,
// outflow ghosts) run in their own instantiation; the base one compiles them out
static bool uses_ext(const Geo& g) { return g.indirect || g.damp || g.bc_z == 1 || g.drag_law; }

template <int ND, bool EXT>
static void gas_ext(const StageArgs& a, int blocks, hipStream_t s) {
  if (a.g.p32)
    hipLaunchKernelGGL((k_gas32<ND, EXT>), dim3(blocks), dim3(NTM), 0, s, a);
  else if (a.g.gamma == 1.4)
    hipLaunchKernelGGL((k_gas<ND, true, EXT>), dim3(blocks), dim3(NTM), 0, s, a);
  else
    hipLaunchKernelGGL((k_gas<ND, false, EXT>), dim3(blocks), dim3(NTM), 0, s, a);
}
template <int ND>
static void gas_nd(const StageArgs& a, int blocks, hipStream_t s) {
  if (uses_ext(a.g)) gas_ext<ND, true>(a, blocks, s);
  else gas_ext<ND, false>(a, blocks, s);
}

hipError_t launch_stage_group(const StageArgs& a, const Layout& L, int group, hipStream_t s) {
  if (group > 0) {
    const dim3 blocks(L.nblocks_dust), threads(NTM);
    const bool ext = uses_ext(a.g);
    if (a.g.p32 && ext) hipLaunchKernelGGL((k_dust<true, true>), blocks, threads, 0, s, a, group - 1);
    else if (a.g.p32) hipLaunchKernelGGL((k_dust<true, false>), blocks, threads, 0, s, a, group - 1);
    else if (ext) hipLaunchKernelGGL((k_dust<false, true>), blocks, threads, 0, s, a, group - 1);
    else hipLaunchKernelGGL((k_dust<false, false>), blocks, threads, 0, s, a, group - 1);
    return hipGetLastError();
  }
  switch (a.g.nd) {
    case 0: gas_nd<0>(a, L.nblocks, s); break;
    case 1: gas_nd<1>(a, L.nblocks, s); break;
    case 2: gas_nd<2>(a, L.nblocks, s); break;
    case 3: gas_nd<3>(a, L.nblocks, s); break;
    case 4: gas_nd<4>(a, L.nblocks, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_stage(const StageArgs& a, const Layout& L, hipStream_t s) {
  hipError_t e = launch_stage_group(a, L, 0, s);
  if (e != hipSuccess || a.gas_only) return e;
  for (int sp = 0; sp < a.g.nd; ++sp) {
    e = launch_stage_group(a, L, 1 + sp, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int ND>
static void cfl_nd(const StageArgs& a, const void* state, int blocks, hipStream_t s) {
  if (a.g.p32) hipLaunchKernelGGL((k_cfl<ND, true>), dim3(blocks), dim3(256), 0, s, a, state);
  else hipLaunchKernelGGL((k_cfl<ND, false>), dim3(blocks), dim3(256), 0, s, a, state);
}

hipError_t launch_cfl(const StageArgs& a, const void* state, int blocks, int dt_idx,
                      hipStream_t s) {
  (void)dt_idx;
  switch (a.g.nd) {
    case 0: cfl_nd<0>(a, state, blocks, s); break;
    case 1: cfl_nd<1>(a, state, blocks, s); break;
    case 2: cfl_nd<2>(a, state, blocks, s); break;
    case 3: cfl_nd<3>(a, state, blocks, s); break;
    case 4: cfl_nd<4>(a, state, blocks, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int ND>
static void drag_nd(const StageArgs& a, void* state, double frac, int blocks, hipStream_t s) {
  if (a.g.p32) hipLaunchKernelGGL((k_drag<ND, true>), dim3(blocks), dim3(256), 0, s, a, state, frac);
  else hipLaunchKernelGGL((k_drag<ND, false>), dim3(blocks), dim3(256), 0, s, a, state, frac);
}

hipError_t launch_drag(const StageArgs& a, void* state, double frac, int blocks, hipStream_t s) {
  switch (a.g.nd) {
    case 1: drag_nd<1>(a, state, frac, blocks, s); break;
    case 2: drag_nd<2>(a, state, frac, blocks, s); break;
    case 3: drag_nd<3>(a, state, frac, blocks, s); break;
    case 4: drag_nd<4>(a, state, frac, blocks, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_reduce(const StageArgs& a, int nparts, int nparts_dust, int dt_idx_next,
                         int want_dt, int want_ledger, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(256), 0, s, a, nparts, nparts_dust, dt_idx_next,
                     want_dt, want_ledger);
  return hipGetLastError();
}

hipError_t launch_ctrl_init(Ctrl* c, hipStream_t s) {
  hipLaunchKernelGGL(k_ctrl_init, dim3(1), dim3(64), 0, s, c);
  return hipGetLastError();
}

hipError_t launch_cfl_out(const Ctrl* c, const double* dt, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_cfl_out, dim3(1), dim3(64), 0, s, c, dt, out);
  return hipGetLastError();
}

hipError_t launch_fill(double* p, size_t n, double v, hipStream_t s) {
  const int blocks = (int)std::min<size_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(k_fill, dim3(std::max(blocks, 1)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_to_full(const StageArgs& a, const void* state, double* out, int f,
                          hipStream_t s) {
  const int blocks = (int)std::min<size_t>((a.g.N + 255) / 256, 65536);
  if (a.g.p32) hipLaunchKernelGGL(k_to_full<true>, dim3(blocks), dim3(256), 0, s, a, state, out, f);
  else hipLaunchKernelGGL(k_to_full<false>, dim3(blocks), dim3(256), 0, s, a, state, out, f);
  return hipGetLastError();
}

hipError_t launch_from_full(const StageArgs& a, const double* in, void* state, int f,
                            hipStream_t s) {
  const int blocks = (int)std::min<size_t>((a.g.N + 255) / 256, 65536);
  if (a.g.p32) hipLaunchKernelGGL(k_from_full<true>, dim3(blocks), dim3(256), 0, s, a, in, state, f);
  else hipLaunchKernelGGL(k_from_full<false>, dim3(blocks), dim3(256), 0, s, a, in, state, f);
  return hipGetLastError();
}

hipError_t launch_mass(const StageArgs& a, const void* state, double* partials, int f,
                       int blocks, hipStream_t s) {
  if (a.g.p32) hipLaunchKernelGGL(k_mass<true>, dim3(blocks), dim3(256), 0, s, a, state, partials, f);
  else hipLaunchKernelGGL(k_mass<false>, dim3(blocks), dim3(256), 0, s, a, state, partials, f);
  return hipGetLastError();
}

hipError_t launch_amp_grad(const InitArgs& a, const double* lam, double* out, hipStream_t s) {
  const int blocks = (int)std::min<size_t>((a.g.N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_amp_grad, dim3(blocks), dim3(256), 0, s, a, lam, out);
  return hipGetLastError();
}

hipError_t launch_indirect(const StageArgs& a, const void* state, double* partials, int blocks,
                           double* ab, hipStream_t s) {
  if (a.g.p32) hipLaunchKernelGGL(k_indirect<true>, dim3(blocks), dim3(256), 0, s, a, state, partials);
  else hipLaunchKernelGGL(k_indirect<false>, dim3(blocks), dim3(256), 0, s, a, state, partials);
  hipLaunchKernelGGL(k_indirect_final, dim3(1), dim3(256), 0, s, partials, blocks, ab);
  return hipGetLastError();
}

hipError_t launch_sum(const double* partials, int n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, s, partials, n, out);
  return hipGetLastError();
}

}  // namespace rb
