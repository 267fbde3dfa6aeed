// Discrete adjoint of the RK2 stage operator on gfx950 (FP64).
//
// A stage is E_out = base + c dt V^-1 (G(E) - R0).  Given a cotangent lambda of E_out,
// the kernels here form J_G(E)^T w with w = c dt V^-1 lambda: the reverse of every
// face flux -- the exact Riemann solution differentiated on the wave pattern the
// primal solve took (star pressure by implicit differentiation of the pressure-function
// equation, Sect. 2.6), the limited parabolic reconstruction on the limiter branch taken
// (Sect. 2.7), the positivity fallback on the side it was taken -- scattered back to the
// four cells of each face stencil, plus the cell-local reverse of the geometric and
// gravity sources and of the gas-dust drag (Sect. 2.9, App. B).  The primal face
// solves are recomputed with the forward solver itself (its short form where that applies,
// else its recording variant), so the branch decisions are the forward run's, but for ties:
// a theta face's states, formed with r's weights, may differ from its in the last bit.
//
// k_adj_plane follows the forward stage kernel's tiles: a workgroup owns a 64 (theta) x
// 8 (r) tile and a chunk of z planes.  Each plane is staged in LDS with a three-cell halo
// (a cell receives contributions from the faces 3/2 cells away); the contributions of
// the theta and r faces to the tile's cells are accumulated in LDS in a fixed order, one
// phase per stencil position, so results are deterministic.  k_adj_z then marches every
// column upwards in registers and adds the z faces' contributions, each cell's in the
// order of its faces.
#include <algorithm>

#include "rb_device.h"

namespace rb {

// ------------------------------------------------------------------------------------
// reverse of the building blocks

// Derivative (cm, cp) of a limited increment with respect to the backward and forward
// differences of its cell, on the branch the limiter took: in the signed variables of
// face_pair (any: the arguments are positive) the parabola's x where it is the least, else
// the backward difference's y or the forward one's z.
__device__ __forceinline__ void dlim(bool any, double x, double y, double z, double wm, double wp,
                                     double lm, double lp, double& cm, double& cp) {
  const bool par = any && x <= fmin(y, z), bwd = any && !par && y <= z, fwd = any && !par && !bwd;
  cm = par ? wm : bwd ? lm : 0.0;
  cp = par ? wp : fwd ? lp : 0.0;
}

// The reverse of one field of face_pair: cotangents qL, qR of the limited states -> the
// stencil cells' values; a state that fell back (fbL, fbR) is its cell's own.
// ADD: added to oA .. oD, else stored.
template <int DIR, bool ADD>
__device__ __forceinline__ void pair_rev(double A, double B, double C, double D, const double* coB,
                                         const double* coC, bool fbL, bool fbR, double qL,
                                         double qR, double& oA, double& oB, double& oC, double& oD) {
  const double d2 = C - B, s = copysign(1.0, d2), a = fabs(d2);
  const double b1 = s * (B - A), b3 = s * (D - C);
  double um, up, lm, lp;
  if constexpr (DIR == 0) {
    dlim(!fbL && a > 0.0 && b1 > 0.0, fma(coB[RC_WPP], a, coB[RC_WPM] * b1), coB[RC_LPM] * b1,
         coB[RC_LPP] * a, coB[RC_WPM], coB[RC_WPP], coB[RC_LPM], coB[RC_LPP], um, up);
    dlim(!fbR && a > 0.0 && b3 > 0.0, fma(-coC[RC_WMP], b3, -coC[RC_WMM] * a), -coC[RC_LMM] * a,
         -coC[RC_LMP] * b3, coC[RC_WMM], coC[RC_WMP], coC[RC_LMM], coC[RC_LMP], lm, lp);
  } else {
    dlim(!fbL && a > 0.0 && b1 > 0.0, fma(3.0, a, b1) * 0.125, b1, a, 0.125, 0.375, 1.0, 1.0, um, up);
    dlim(!fbR && a > 0.0 && b3 > 0.0, fma(3.0, a, b3) * 0.125, a, b3, -0.375, -0.125, -1.0, -1.0, lm, lp);
  }
  const double vA = -um * qL, vB = fma(1.0 + um - up, qL, -lm * qR);
  const double vC = fma(up, qL, (1.0 + lm - lp) * qR), vD = lp * qR;
  if constexpr (ADD) {
    oA += vA; oB += vB; oC += vC; oD += vD;
  } else {
    oA = vA; oB = vB; oC = vC; oD = vD;
  }
}

// One side's pressure function at p and its partial derivatives: df/dp, and df/drho_K,
// df/dp_K at fixed p (shock: f = (p - p_K) sqrt(A/(p + B)); rarefaction:
// f = 2 c_K/(g-1) ((p/p_K)^((g-1)/2g) - 1)).
struct PD {
  double f, df, fr, fp;
};
template <bool G75>
__device__ __forceinline__ PD pfun_pd(double p, double rK, double pK, double cK, const GasC& c) {
  PD o;
  if (p > pK) {
    const double ipb = 1.0 / (p + c.kshock * pK);
    const double q = sqrt(c.a2 / rK * ipb);
    o.f = (p - pK) * q;
    o.df = q * (1.0 - 0.5 * (p - pK) * ipb);
    o.fr = -0.5 * o.f / rK;
    o.fp = -q - 0.5 * o.f * c.kshock * ipb;
  } else {
    Pow3<G75> w(p / pK, c);
    o.f = c.g2m1 * cK * (w.p17 - 1.0);
    o.df = w.pm67 / (rK * cK);
    o.fr = -0.5 * o.f / rK;
    o.fp = 0.5 * o.f / pK - cK * w.p17 / (c.g * pK);
  }
  return o;
}

// Reverse of F(W) for the sampled primitive state W = (rho, un, t1, t2, p); flb in the
// order mass, normal momentum, two tangential momenta, energy.  Output: W cotangent.
__device__ __forceinline__ void flux_rev(const GasC& c, const GasRec& w, const double flb[5],
                                         double Wb[5]) {
  const double m = w.rho * w.un;
  const double ke = 0.5 * (w.un * w.un + w.t1 * w.t1 + w.t2 * w.t2);
  const double en = w.p * c.inv_gm1 + w.rho * ke;
  const double mb = flb[0] + flb[1] * w.un + flb[2] * w.t1 + flb[3] * w.t2;
  const double enb = flb[4] * w.un;
  Wb[0] = enb * ke + mb * w.un;
  Wb[1] = flb[1] * m + flb[4] * (en + w.p) + enb * w.rho * w.un + mb * w.rho;
  Wb[2] = flb[2] * m + enb * w.rho * w.t1;
  Wb[3] = flb[3] * m + enb * w.rho * w.t2;
  Wb[4] = flb[1] + flb[4] * w.un + enb * c.inv_gm1;
}

// Reverse of the Riemann solution at x/t = 0 on the recorded wave pattern: W cotangent
// -> cotangents of the primitive face states WL, WR (rho, un, t1, t2, p).  The star
// state depends on the face states directly and through p*, u*:
//   f_L(p*) + f_R(p*) + u_R - u_L = 0,  u* = (u_L + u_R)/2 + (f_R(p*) - f_L(p*))/2.
template <bool G75>
__device__ void riemann_rev(const GasC& c, const double* WL, const double* WR, const GasRec& rec,
                            const double* Wb, double* WLb, double* WRb) {
#pragma unroll
  for (int q = 0; q < 5; ++q) { WLb[q] = 0.0; WRb[q] = 0.0; }
  const int br = rec.branch;
  if (br == GR_LEFT) {
#pragma unroll
    for (int q = 0; q < 5; ++q) WLb[q] = Wb[q];
    return;
  }
  if (br == GR_RIGHT) {
#pragma unroll
    for (int q = 0; q < 5; ++q) WRb[q] = Wb[q];
    return;
  }
  if (br == GR_VACUUM) return;
  if (br == GR_FAN_L || br == GR_FAN_R) {
    // inside a fan: c_c = 2/(g+1) (c_K +- (g-1)/2 u_K), rho = rho_K (c_c/c_K)^(2/(g-1)),
    // p = p_K (c_c/c_K)^(2g/(g-1)), un = +-c_c
    const bool left = br == GR_FAN_L;
    const double* W = left ? WL : WR;
    double* Wk = left ? WLb : WRb;
    const double sg = left ? 1.0 : -1.0;
    const double rK = W[0], uK = W[1], pK = W[4];
    const double cK = sqrt(c.g * pK / rK);
    const double cc = c.a2 * (cK + sg * c.half_gm1 * uK);
    const double ratio = cc / cK;
    const double e1 = c.g2m1, e2 = 2.0 * c.g / (c.g - 1.0);
    const double r1 = pow(ratio, e1 - 1.0), r2 = pow(ratio, e2 - 1.0);
    const double ratb = Wb[0] * rK * e1 * r1 + Wb[4] * pK * e2 * r2;
    Wk[0] += Wb[0] * r1 * ratio;
    Wk[4] += Wb[4] * r2 * ratio;
    const double ccb = sg * Wb[1] + ratb / cK;
    const double cKb = -ratb * cc / (cK * cK) + c.a2 * ccb;
    Wk[1] += sg * c.a2 * c.half_gm1 * ccb;
    Wk[4] += cKb * cK / (2.0 * pK);
    Wk[0] -= cKb * cK / (2.0 * rK);
    Wk[2] += Wb[2];
    Wk[3] += Wb[3];
    return;
  }
  // star states
  const bool left = br == GR_STAR_L_SHOCK || br == GR_STAR_L_RARE;
  const double* W = left ? WL : WR;
  double* Wk = left ? WLb : WRb;
  const double ps = rec.ps;
  double psb = Wb[4];
  const double usb = Wb[1];
  Wk[2] += Wb[2];
  Wk[3] += Wb[3];
  const double rK = W[0], pK = W[4];
  if (br == GR_STAR_L_SHOCK || br == GR_STAR_R_SHOCK) {
    // rho* = rho_K (q + k)/(k q + 1), q = p*/p_K, k = (g-1)/(g+1)
    const double q = ps / pK, k = c.kshock, den = k * q + 1.0;
    Wk[0] += Wb[0] * (q + k) / den;
    const double qb = Wb[0] * rK * (1.0 - k * k) / (den * den);
    psb += qb / pK;
    Wk[4] -= qb * q / pK;
  } else {
    // rho* = rho_K (p*/p_K)^(1/g)
    const double rho = rec.rho;
    Wk[0] += Wb[0] * rho / rK;
    psb += Wb[0] * rho / (c.g * ps);
    Wk[4] -= Wb[0] * rho / (c.g * pK);
  }
  const double cL = sqrt(c.g * WL[4] / WL[0]), cR = sqrt(c.g * WR[4] / WR[0]);
  const PD L = pfun_pd<G75>(ps, WL[0], WL[4], cL, c);
  const PD R = pfun_pd<G75>(ps, WR[0], WR[4], cR, c);
  // u*
  WLb[1] += 0.5 * usb;
  WRb[1] += 0.5 * usb;
  psb += 0.5 * usb * (R.df - L.df);
  WRb[0] += 0.5 * usb * R.fr;
  WRb[4] += 0.5 * usb * R.fp;
  WLb[0] -= 0.5 * usb * L.fr;
  WLb[4] -= 0.5 * usb * L.fp;
  // p*: dp* = -(dPhi) / (f_L' + f_R')
  const double s = psb / (L.df + R.df);
  WLb[1] += s;
  WRb[1] -= s;
  WLb[0] -= s * L.fr;
  WLb[4] -= s * L.fp;
  WRb[0] -= s * R.fr;
  WRb[4] -= s * R.fp;
}

// Cotangent of a cell's reconstructed variables -> cotangent of its conservative
// variables.  Gas: W = (u, v, w, P, rho) of E = (rho u, rho v, rho w, E, rho) at the full
// state (the stationary flow b plus the cell's W'), u = m / rho,
// P = (g - 1)(E - |m|^2 / (2 rho)).
__device__ __forceinline__ void gas_cot_to_cons(const double* w, const double* b, double gm1,
                                                const double* wb, double* eb) {
  const double rho = b[WB_RHO] + w[4];
  const double ir = 1.0 / rho;
  const double u[3] = {b[WB_U] + w[0], b[WB_V] + w[1], b[WB_W] + w[2]};
  const double pb = gm1 * wb[3];
  double dot = 0.0, u2 = 0.0;
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    eb[m] = wb[m] * ir - pb * u[m];
    dot += wb[m] * u[m];
    u2 += u[m] * u[m];
  }
  eb[3] = pb;
  eb[4] = wb[4] - dot * ir + 0.5 * pb * u2;
}
// Dust: W = (u, v, w, rho_d) of (rho_d u, rho_d v, rho_d w, rho_d); the velocity of an
// empty cell is held at zero.
__device__ __forceinline__ void dust_cot_to_cons(const double* w, const double* wb, double* eb) {
  const double rd = w[3];
  if (rd > 0.0) {
    const double ir = 1.0 / rd;
    eb[0] = wb[0] * ir;
    eb[1] = wb[1] * ir;
    eb[2] = wb[2] * ir;
    eb[3] = wb[3] - (wb[0] * w[0] + wb[1] * w[1] + wb[2] * w[2]) * ir;
  } else {
    eb[0] = 0.0; eb[1] = 0.0; eb[2] = 0.0;
    eb[3] = wb[3];
  }
}

// Reverse of a gas face by the short form (gamma = 7/5; states, cotangents in field slots):
// the star state and the pressure functions by gas_face64's polynomials, their slopes by the
// same polynomials' derivatives, and the partial derivatives of f = sqrt(p_K / rho_K) h(p/p_K)
// from f and f' alone: df/drho_K = -f / (2 rho_K), df/dp_K = f / (2 p_K) - (p / p_K) f'.
// Returns false, the cotangents unset, where the short form does not apply.
template <int DIR>
__device__ __forceinline__ bool gas_weak_rev(const GasC& c, const double* qL, const double* qR,
                                             const double* Fb, double* qLb, double* qRb) {
  constexpr int N = Dirs<DIR>::n, T1 = Dirs<DIR>::t1, T2 = Dirs<DIR>::t2;
  const double rL = qL[4], rR = qR[4], pL = qL[3], pR = qR[3], uL = qL[N], uR = qR[N];
  const double irL = frcp(rL), irR = frcp(rR);
  const double c2L = c.g * pL * irL, c2R = c.g * pR * irR;
  const bool weak = rL > 0.0 && pL > 0.0 && rR > 0.0 && pR > 0.0 && uL * uL < 0.81 * c2L &&
                    uR * uR < 0.81 * c2R;
  const double rsL = frsq(c2L), rsR = frsq(c2R);
  const double cL = c2L * rsL, cR = c2R * rsR, du = uR - uL;
  const double ipL = frcp(pL), ipR = frcp(pR);
  const double gL = (5.0 / 7.0) * cL, gR = (5.0 / 7.0) * cR;
  const WeakStar w = weak_star(c, pL, pR, ipL, ipR, gL, gR, irL * rsL, irR * rsR, du,
                               0.5 * (pL + pR) - 0.125 * du * (rL + rR) * (cL + cR), weak);
  const double ps = w.ps, xL = (ps - pL) * ipL, xR = (ps - pR) * ipR;
  const bool narrow = w.xm <= 1.0 / 512.0;
  double GL, GR, dGL, dGR;
  if (narrow) {
    const ctab t = weak_table(WK_G);
    GL = weak_poly_d<4>(t, xL, 1.0, dGL);
    GR = weak_poly_d<4>(t, xR, 1.0, dGR);
  } else {
    const ctab t = weak_table(WKW_G);
    GL = weak_poly_d<8>(t, xL, 1.0, dGL);
    GR = weak_poly_d<8>(t, xR, 1.0, dGR);
  }
  const double fL = gL * xL * GL, fR = gR * xR * GR;
  const double dfL = gL * ipL * fma(xL, dGL, GL), dfR = gR * ipR * fma(xR, dGR, GR);
  const double us = 0.5 * (uL + uR) + 0.5 * (fR - fL);
  if (!(weak && w.conv && us * us < 0.81 * fmin(c2L, c2R))) return false;
  const bool left = us >= 0.0;
  const double rK = left ? rL : rR, ipK = left ? ipL : ipR, x = left ? xL : xR;
  double R, dR;
  if (narrow) R = weak_poly_d<4>(weak_table(WK_R), x, 5.0 / 7.0, dR);
  else R = weak_poly_d<8>(weak_table(WKW_R), x, 5.0 / 7.0, dR);
  const double ratio = fma(x, R, 1.0), drs = rK * fma(x, dR, R) * ipK;  // rho* / rho_K, drho*/dp*
  GasRec rec;
  rec.rho = fma(rK * x, R, rK);
  rec.un = us;
  rec.t1 = left ? qL[T1] : qR[T1];
  rec.t2 = left ? qL[T2] : qR[T2];
  rec.p = ps;
  const double flb[5] = {Fb[4], Fb[N], Fb[T1], Fb[T2], Fb[3]};
  double Wb[5];
  flux_rev(c, rec, flb, Wb);
  // (as riemann_rev: through rho*, u* and p*)
  const double hub = 0.5 * Wb[1], rb = Wb[0] * ratio, pb = -Wb[0] * drs * (1.0 + x);
  const double s = (Wb[4] + Wb[0] * drs + hub * (dfR - dfL)) * frcp(dfL + dfR);
  const double aL = -(hub + s), aR = hub - s;  // cotangents of f_L, f_R at fixed p*
  qLb[4] = aL * (-0.5 * fL * irL) + (left ? rb : 0.0);
  qRb[4] = aR * (-0.5 * fR * irR) + (left ? 0.0 : rb);
  qLb[3] = aL * (0.5 * fL * ipL - (1.0 + xL) * dfL) + (left ? pb : 0.0);
  qRb[3] = aR * (0.5 * fR * ipR - (1.0 + xR) * dfR) + (left ? 0.0 : pb);
  qLb[N] = hub + s;
  qRb[N] = hub - s;
  qLb[T1] = left ? Wb[2] : 0.0;
  qLb[T2] = left ? Wb[3] : 0.0;
  qRb[T1] = left ? 0.0 : Wb[2];
  qRb[T2] = left ? 0.0 : Wb[3];
  return true;
}

// Reverse of one gas face: Fb (field order) is the cotangent of the face flux; the
// contributions to the reconstructed variables W' of the stencil cells A, B | C, D are
// stored in cA .. cD, or (ADD) added to them.  cell(c, f): W' of a cell, after again() read anew (held across
// the solve the cells would cost 40 registers); bf(f): the stationary flow at the face;
// bB(f), bC(f): at the centres of B and C.
template <int DIR, bool ADD, bool G75, class Cell, class Bf, class Bc>
__device__ __forceinline__ void gas_face_vjp(const GasC& c, const RecC& rc, Cell cell, const double* coB,
                                             const double* coC, Bf bf, Bc bB, Bc bC,
                                             const double* Fb, double* cA,
                                             double* cB, double* cC, double* cD) {
  constexpr int N = Dirs<DIR>::n, T1 = Dirs<DIR>::t1, T2 = Dirs<DIR>::t2;
  double qL[5], qR[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    face_pair<DIR>(rc, cell(0, f), cell(1, f), cell(2, f), cell(3, f), coB, coC, qL[f], qR[f]);
    const double w0 = bf(f);
    qL[f] = w0 + qL[f];
    qR[f] = w0 + qR[f];
  }
  double qLb[5], qRb[5];
  bool fbL = false, fbR = false, done = false;
  if constexpr (G75) done = gas_weak_rev<DIR>(c, qL, qR, Fb, qLb, qRb);
  if (!done) {
    fbL = !(qL[4] > 0.0 && qL[3] > 0.0);
    fbR = !(qR[4] > 0.0 && qR[3] > 0.0);
    if (fbL) {
#pragma unroll
      for (int f = 0; f < 5; ++f) qL[f] = bB(f) + cell(1, f);
    }
    if (fbR) {
#pragma unroll
      for (int f = 0; f < 5; ++f) qR[f] = bC(f) + cell(2, f);
    }
    double WLb[5], WRb[5];
    {
      double fl[5];
      TStat st = {0, 0, 0, 0, 0, 0, 0};
      GasRec rec;
      gas_riemann<G75, true>(c, qL[4], frcp(qL[4]), qL[N], qL[T1], qL[T2], qL[3], qR[4], frcp(qR[4]),
                             qR[N], qR[T1], qR[T2], qR[3], fl, st, &rec);
      const double flb[5] = {Fb[4], Fb[N], Fb[T1], Fb[T2], Fb[3]};
      double Wb[5];
      flux_rev(c, rec, flb, Wb);
      const double WL[5] = {qL[4], qL[N], qL[T1], qL[T2], qL[3]};
      const double WR[5] = {qR[4], qR[N], qR[T1], qR[T2], qR[3]};
      riemann_rev<G75>(c, WL, WR, rec, Wb, WLb, WRb);
    }
    // face-frame cotangents (rho, un, t1, t2, p) -> field slots (u, v, w, P, rho)
    qLb[4] = WLb[0]; qLb[N] = WLb[1]; qLb[T1] = WLb[2]; qLb[T2] = WLb[3]; qLb[3] = WLb[4];
    qRb[4] = WRb[0]; qRb[N] = WRb[1]; qRb[T1] = WRb[2]; qRb[T2] = WRb[3]; qRb[3] = WRb[4];
  }
  // left face state -> cells A, B, C (or B alone after a fallback); right -> B, C, D
  cell.again();
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    pair_rev<DIR, ADD>(cell(0, f), cell(1, f), cell(2, f), cell(3, f), coB, coC, fbL, fbR, qLb[f],
                       qRb[f], cA[f], cB[f], cC[f], cD[f]);
  }
}

// Reverse of one dust face (velocity and density reconstructed whole; a negative face
// density falls back to the cell value).  Contributions to the cells' reconstructed
// variables.
template <int DIR, bool ADD, class Cell>
__device__ __forceinline__ void dust_face_vjp(const RecC& rc, Cell cell, const double* coB, const double* coC,
                                              const double* Fb, double* cA,
                                             double* cB, double* cC, double* cD) {
  constexpr int N = Dirs<DIR>::n, T1 = Dirs<DIR>::t1, T2 = Dirs<DIR>::t2;
  double qL[4], qR[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    face_pair<DIR>(rc, cell(0, f), cell(1, f), cell(2, f), cell(3, f), coB, coC, qL[f], qR[f]);
  }
  const bool fbL = qL[3] < 0.0, fbR = qR[3] < 0.0;
  if (fbL) {
#pragma unroll
    for (int f = 0; f < 4; ++f) qL[f] = cell(1, f);
  }
  if (fbR) {
#pragma unroll
    for (int f = 0; f < 4; ++f) qR[f] = cell(2, f);
  }
  double fl[4];
  int side;
  dust_riemann<true>(qL[3], qL[N], qL[T1], qL[T2], qR[3], qR[N], qR[T1], qR[T2], fl, &side);
  const double flb[4] = {Fb[3], Fb[N], Fb[T1], Fb[T2]};
  double qLb[4] = {0.0, 0.0, 0.0, 0.0}, qRb[4] = {0.0, 0.0, 0.0, 0.0};
  // one side's flux (r u, r u^2, r u a, r u b) in its face state (r, u, a, b); zero for an
  // empty side (its velocity is held at zero)
  auto side_rev = [&](const double* q, double wgt, double* qb) {
    const double r = q[3];
    if (!(r > 0.0)) return;
    const double u = q[N], ta = q[T1], tb = q[T2];
    qb[3] += wgt * (flb[0] * u + flb[1] * u * u + flb[2] * u * ta + flb[3] * u * tb);
    qb[N] += wgt * (flb[0] * r + 2.0 * flb[1] * r * u + flb[2] * r * ta + flb[3] * r * tb);
    qb[T1] += wgt * flb[2] * r * u;
    qb[T2] += wgt * flb[3] * r * u;
  };
  if (side == -1) side_rev(qL, 1.0, qLb);
  else if (side == 1) side_rev(qR, 1.0, qRb);
  else if (side == 0) {
    side_rev(qL, 0.5, qLb);
    side_rev(qR, 0.5, qRb);
  }
  cell.again();
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    pair_rev<DIR, ADD>(cell(0, f), cell(1, f), cell(2, f), cell(3, f), coB, coC, fbL, fbR, qLb[f],
                       qRb[f], cA[f], cB[f], cC[f], cD[f]);
  }
}

// ------------------------------------------------------------------------------------
// the adjoint stage kernels: the theta and r faces and the cell-local sources of a tile
// of planes (k_adj_plane, LDS-staged), then the z faces of every column (k_adj_z,
// registers only, adding into the output of the first).  Two kernels keep each one's
// register footprint within the file (one kernel holding both spilled to scratch).

// group-independent set-up shared by both kernels
template <bool GAS>
struct AdjCtx {
  static constexpr int NG = GAS ? 5 : 4;
  const AdjArgs& A;
  const StageArgs& a;
  const Geo& g;
  GasC gc;
  int F0;
  __device__ AdjCtx(const AdjArgs& A_, int species)
      : A(A_), a(A_.s), g(A_.s.g), gc(gas_consts(A_.s.g.gamma, A_.s.g.newton_max)), F0(GAS ? 0 : 5 + 4 * species) {}
  __device__ int jwrap(int j) const {
    j %= g.nth;
    return j < 0 ? j + g.nth : j;
  }
  // w of every field of a cell (zero outside the grid), all loads requested together
  __device__ void wc_all(int k, int i, int j, double* out) const {
    const bool in = !(k < 0 || k >= g.nz || i < 0 || i >= g.nr);
    const size_t c = in ? ((size_t)k * g.nr + i) * g.nth + j : 0;
    const double v = in ? a.t.rt[(size_t)i * RT_N + RT_INVV] : 0.0;
    double x[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) x[f] = A.cot[(size_t)(F0 + f) * g.N + c];
#pragma unroll
    for (int f = 0; f < NG; ++f) out[f] = in ? A.cw * v * x[f] : 0.0;
  }
  // the difference w(k1, i1, j1) - w(k0, i0, j0) of every field, times s, with all loads
  // requested before any arithmetic (loads under per-field conditions each waited)
  __device__ void wc_diff(int k1, int i1, int j1, int k0, int i0, int j0, double s,
                          double* out) const {
    const bool in1 = !(k1 < 0 || k1 >= g.nz || i1 < 0 || i1 >= g.nr);
    const bool in0 = !(k0 < 0 || k0 >= g.nz || i0 < 0 || i0 >= g.nr);
    const size_t c1 = in1 ? ((size_t)k1 * g.nr + i1) * g.nth + j1 : 0;
    const size_t c0 = in0 ? ((size_t)k0 * g.nr + i0) * g.nth + j0 : 0;
    const double v1 = in1 ? a.t.rt[(size_t)i1 * RT_N + RT_INVV] : 0.0;
    const double v0 = in0 ? a.t.rt[(size_t)i0 * RT_N + RT_INVV] : 0.0;
    double x1[NG], x0[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) {
      x1[f] = A.cot[(size_t)(F0 + f) * g.N + c1];
      x0[f] = A.cot[(size_t)(F0 + f) * g.N + c0];
    }
#pragma unroll
    for (int f = 0; f < NG; ++f)
      out[f] = s * ((in1 ? A.cw * v1 * x1[f] : 0.0) - (in0 ? A.cw * v0 * x0[f] : 0.0));
  }
};

template <int D, bool ADD, bool GAS, bool G75, class Cell, class Bf, class Bc>
__device__ __forceinline__ void face_vjp(const GasC& gc, const RecC& rc, Cell cell, const double* coB,
                                         const double* coC, Bf bf, Bc bB, Bc bC,
                                         const double* Fb, double* cA,
                                             double* cB, double* cC, double* cD) {
  if constexpr (GAS) gas_face_vjp<D, ADD, G75>(gc, rc, cell, coB, coC, bf, bB, bC, Fb, cA, cB, cC, cD);
  else dust_face_vjp<D, ADD>(rc, cell, coB, coC, Fb, cA, cB, cC, cD);
}

// cotangent of a cell's reconstructed variables w (stationary flow b) -> conservative
template <bool GAS>
__device__ __forceinline__ void cot_to_cons(const double* w, const double* b, double gm1,
                                            const double* wb, double* eb) {
  if constexpr (GAS) gas_cot_to_cons(w, b, gm1, wb, eb);
  else dust_cot_to_cons(w, wb, eb);
}

// In-plane faces and sources.  Bound by instruction issue (4000 -> 2700 lane-instructions per
// cell of the gas) and, for a quarter of the time, by the loads of a plane and its halo.  The
// general reverse of a face runs the recording solver, twenty divisions and every branch of
// the wave pattern; a face of weak waves takes gas_weak_rev.  One copy of the face serves the
// theta faces, the r faces and the tile's edge: four copies spilled 72 registers.  128 x 256 x
// 32 cells, one dust species: gas 300 -> 183 us per launch, dust 158 -> 120.  Tiles of four rows
// with two workgroups on a CU, which overlap the loads of one with the faces of the other,
// gave 201 and 120: the halo and the edge faces weigh more.
template <bool GAS, int ND, bool G75>
__global__ void __launch_bounds__(NT, 2) k_adj_plane(AdjArgs A, int species) {
  using C = AdjCtx<GAS>;
  constexpr int NG = C::NG;
  constexpr int H = 3;
  constexpr int W = TJ + 2 * H, PL = (TI + 2 * H) * W, PT = TI * TJ;
  __shared__ double s_e[NG * PL];
  // w = cw V^-1 lambda of the staged cells (zero outside the grid), staged with the plane
  // so that the faces read no global memory
  __shared__ double s_w[NG * PL];
  // the cells' totals from the theta and the r faces
  __shared__ double s_acc[2 * NG * PT];
  // faces by slot: theta faces of row r in slot r, r faces above tile row rb in TI + 2 + rb:
  // the face area and, per plane, the stationary flow there
  constexpr int NS = 2 * TI + 3;
  __shared__ double s_fa[NS], s_bf[GAS ? NS : 1][5];
  // parabola weights of the cells of tile rows -2 .. TI + 1, and of a theta stencil
  __shared__ double s_co[TI + 5][RC_N];
  __shared__ double s_red[NT / 64];

  const C X(A, species);
  const StageArgs& a = X.a;
  const Geo& g = X.g;
  const int F0 = X.F0;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int tjb = tile % a.ntj;
  const int tib = (tile / a.ntj) % a.nti;
  const int kcb = tile / (a.ntj * a.nti);
  // the row index is wavefront-uniform (one 64-lane wavefront per row of a 1D workgroup):
  // per-row tables go to scalar registers
  const int tid = threadIdx.x, tj = tid & (TJ - 1);
  const int ti = __builtin_amdgcn_readfirstlane(tid / TJ);
  const int j0 = tjb * TJ, i0 = tib * TI;
  const int k0 = kcb * A.tk, k1 = min(g.nz, k0 + A.tk);
  const int jg = j0 + tj;
  const int ig = i0 + ti;
  const bool act = jg < g.nth && ig < g.nr;
  const bool colok = jg < g.nth;
  const int igc = min(ig, g.nr - 1);
  const double* E = (const double*)a.in;
  const double* cot = A.cot;
  const size_t N = g.N;
  const double cw = A.cw;
  const double* rt = a.t.rt + (size_t)igc * RT_N;
  const double invrc = rt[RT_INVRC], omk = rt[RT_OMK];
  static_assert((TI + 5) * RC_N + NS <= NT && 5 * NS <= NT && 3 * (TI + TJ) <= NT,
                "one table entry, one edge face per thread");
  if (tid < (TI + 4) * RC_N) {
    s_co[tid / RC_N][tid % RC_N] = rco_ptr(a, min(i0 + tid / RC_N - 2, g.nr))[tid % RC_N];
  } else if (tid < (TI + 5) * RC_N) {
    // (RC_WPM .. RC_LMP on equal spacing)
    const int e = tid % RC_N;
    s_co[TI + 4][e] = e == RC_WPM   ? 0.125
                      : e == RC_WPP ? 0.375
                      : e == RC_WMM ? -0.375
                      : e == RC_WMP ? -0.125
                      : e < RC_WMM  ? 1.0
                                    : -1.0;
  } else if (tid < (TI + 5) * RC_N + NS) {
    const int q = tid - (TI + 5) * RC_N;
    s_fa[q] = q < TI ? a.t.rt[(size_t)min(i0 + q, g.nr - 1) * RT_N + RT_ATH]
                     : a.t.ar[min(max(i0 + q - TI - 1, 0), g.nr)];
  }

  const RecC recc;
  double stb = 0.0;  // Stokes-number partial (dust)
  for (int k = k0; k < k1; ++k) {
    // (the last plane's cells have been read)
    if (k > k0) __syncthreads();
    // ---- stage the plane with a three-cell halo; clear the tile accumulators
    {
      // all cells' loads issued before the stores
      constexpr int PER = (PL + NT - 1) / NT;
      double v[PER][NG], c[PER][NG];
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int h = min(tid + q * NT, PL - 1);
        X.wc_all(k, i0 + h / W - H, X.jwrap(j0 + h % W - H), c[q]);
      }
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int h = min(tid + q * NT, PL - 1);
        load_recon<NG>(a, E, F0, k, i0 + h / W - H, X.jwrap(j0 + h % W - H), v[q]);
      }
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int h = tid + q * NT;
        if (h < PL) {
#pragma unroll
          for (int f = 0; f < NG; ++f) {
            s_e[f * PL + h] = v[q][f];
            s_w[f * PL + h] = c[q][f];
          }
        }
      }
      if (GAS && tid >= NT - NS * 5) {
        const int q = (tid - (NT - NS * 5)) / 5, f = (tid - (NT - NS * 5)) % 5;
        const double* b = q < TI ? a.t.wc + ((size_t)k * g.nr + min(i0 + q, g.nr - 1)) * WB_N
                                 : a.t.wr + ((size_t)k * (g.nr + 1) + min(max(i0 + q - TI - 1, 0), g.nr)) * WB_N;
        s_bf[q][f] = b[f];
      }
    }
#pragma unroll
    for (int f = 0; f < 2 * NG; ++f) s_acc[f * PT + tid] = 0.0;
    __syncthreads();

    // ---- the faces within 3/2 cells of the tile, one copy of the face for all: the thread's
    //      own theta face j+1/2; its own r face i+1/2; the others (theta faces at tile columns
    //      -3/2, -1/2, 64+1/2 of each row by the first 3 TI threads, r faces at tile rows -3/2,
    //      -1/2, TI+1/2 of each column by the next 3 TJ).  A face in its own frame is a DIR = 0
    //      face: the velocity along theta swaps slots with the radial one, and the equal
    //      spacing's weights stand for the table's.  Four ordered scatter phases each
#pragma nounroll
    for (int pass = 0; pass < 3; ++pass) {
      bool theta = pass == 0, ok = pass < 2 && ig < g.nr && (theta || colok);
      int line = theta ? ti : tj, pos = theta ? tj : ti;  // tile row / column; lower cell
      if (pass == 2) {
        const int e = tid - 3 * TI, q = e < 0 ? tid % 3 : e / TJ;
        theta = e < 0;
        line = theta ? tid / 3 : e % TJ;
        pos = q == 0 ? -2 : q == 1 ? -1 : theta ? TJ : TI;
        ok = theta ? i0 + line < g.nr
                   : e < 3 * TJ && i0 + pos + 1 >= 0 && i0 + pos < g.nr && j0 + line < g.nth;
      }
      double o[4][NG];
      const int s0 = theta ? 1 : 0, s1 = theta ? 0 : 1;  // slots of the normal and first tangent
      if (ok) {
        const int st = theta ? 1 : W, at = theta ? (line + H) * W + pos + H : (pos + H) * W + line + H;
        const int slot = theta ? line : TI + 2 + pos;
        auto off = [&](int f) { return at + (f == 0 ? s0 * PL : f == 1 ? s1 * PL : f * PL); };
        // (the base index of the second reads is one the optimiser cannot see through)
        struct Cells {
          const double* e;
          int at, o0, o1, st;
          __device__ double operator()(int c, int f) const {
            return e[at + (f == 0 ? o0 : f == 1 ? o1 : f * PL) + (c - 1) * st];
          }
          __device__ void again() { asm volatile("" : "+v"(at)); }
        };
        const Cells cell = {s_e, at, s0 * PL, s1 * PL, st};
        double Fb[NG];
#pragma unroll
        for (int f = 0; f < NG; ++f) Fb[f] = s_fa[slot] * (s_w[off(f) + st] - s_w[off(f)]);
        auto bf = [&](int f) { return s_bf[GAS ? slot : 0][f == 0 ? s0 : f == 1 ? s1 : f]; };
        struct Centre {
          const double* b;
          int s0, s1;
          __device__ double operator()(int f) const { return b[f == 0 ? s0 : f == 1 ? s1 : f]; }
        };
        const int ib = theta ? i0 + line : i0 + pos;
        const Centre bB = {theta ? a.t.wc + ((size_t)k * g.nr + ib) * WB_N : bg_ptr(a, k, ib), s0, s1};
        const Centre bC = {theta ? bB.b : bg_ptr(a, k, ib + 1), s0, s1};
        const int co = theta ? TI + 4 : pos + 2;
        face_vjp<0, false, GAS, G75>(X.gc, recc, cell, s_co[co], s_co[theta ? co : co + 1], bf, bB, bC, Fb,
                              o[0], o[1], o[2], o[3]);
      }
      double* acc = s_acc + (theta ? 0 : NG * PT);
#pragma unroll
      for (int ph = 0; ph < 4; ++ph) {
        const int t = pos - 1 + ph;  // target cell along the face normal
        if (ok && t >= 0 && t < (theta ? TJ : TI)) {
          const int at = theta ? line * TJ + t : t * TJ + line;
#pragma unroll
          for (int f = 0; f < NG; ++f) acc[(f == 0 ? s0 : f == 1 ? s1 : f) * PT + at] += o[ph][f];
        }
        __syncthreads();
      }
    }
    // ---- in-plane total of the thread's cell, the reverse of its sources, the bases
    if (!act) continue;
    double cur[NG];
    {
      // in-plane faces' cotangent of the cell's reconstructed variables -> conservative
      double wb[NG], w[NG];
#pragma unroll
      for (int f = 0; f < NG; ++f) {
        wb[f] = s_acc[f * PT + tid] + s_acc[(NG + f) * PT + tid];
        w[f] = s_e[f * PL + (ti + H) * W + tj + H];
      }
      cot_to_cons<GAS>(w, a.t.wc + ((size_t)k * g.nr + ig) * WB_N, X.gc.gm1, wb, cur);
    }
    const size_t cell = ((size_t)k * g.nr + ig) * g.nth + jg;
    const double gr = a.t.grav[((size_t)k * g.nr + ig) * 2 + 0];
    const double gz = a.t.grav[((size_t)k * g.nr + ig) * 2 + 1];
    const double* bgc = a.t.bgc + ((size_t)k * g.nr + ig) * 5;
    double q[5], sg[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      q[f] = bgc[f] + E[(size_t)f * N + cell];
      sg[f] = cw * cot[(size_t)f * N + cell];
    }
    const double ir = 1.0 / q[4];
    const double U[3] = {q[0] * ir, q[1] * ir, q[2] * ir};
    if constexpr (GAS) {
      const double gm1 = X.gc.gm1;
      const double u = U[0], v = U[1], w = U[2];
      // S_r = (m_th v + p)/r + rho g_r, S_th = -m_r v / r, S_z = rho g_z,
      // S_E = m_r g_r + m_z g_z
      cur[0] += sg[0] * (-gm1 * u * invrc) + sg[1] * (-v * invrc) + sg[3] * gr;
      cur[1] += sg[0] * ((2.0 - gm1) * v * invrc) + sg[1] * (-u * invrc);
      cur[2] += sg[0] * (-gm1 * w * invrc) + sg[3] * gz;
      cur[3] += sg[0] * gm1 * invrc;
      cur[4] += sg[0] * ((-v * v + 0.5 * gm1 * (u * u + v * v + w * w)) * invrc + gr) +
                sg[1] * (u * v * invrc) + sg[2] * gz;
      // drag D_s = rho_d (v_d - v) Omega_K / St on the gas (+) and the dust (-), and
      // v . D in the gas energy
      double Ub[3] = {0.0, 0.0, 0.0}, Dt[3] = {0.0, 0.0, 0.0};
      // every species' variables and cotangents requested together (loads made
      // conditional on the density would each wait for it)
      double ev[ND > 0 ? ND : 1][4], cv[ND > 0 ? ND : 1][3];
#pragma unroll
      for (int s = 0; s < ND; ++s)
#pragma unroll
        for (int c2 = 0; c2 < 4; ++c2) {
          ev[s][c2] = E[(size_t)(5 + 4 * s + c2) * N + cell];
          if (c2 < 3) cv[s][c2] = cot[(size_t)(5 + 4 * s + c2) * N + cell];
        }
#pragma unroll
      for (int s = 0; s < ND; ++s) {
        const double rdn = ev[s][3];
        double vd[3] = {0.0, 0.0, 0.0};
        if (rdn > 0.0) {
          const double id = 1.0 / rdn;
#pragma unroll
          for (int c2 = 0; c2 < 3; ++c2) vd[c2] = ev[s][c2] * id;
        }
        const double its = omk * g.inv_st[s];
#pragma unroll
        for (int c2 = 0; c2 < 3; ++c2) {
          Dt[c2] += rdn * (vd[c2] - U[c2]) * its;
          const double Db = sg[c2] + sg[3] * U[c2] - cw * cv[s][c2];
          Ub[c2] -= its * rdn * Db;
        }
      }
      double dot = 0.0;
#pragma unroll
      for (int c2 = 0; c2 < 3; ++c2) {
        Ub[c2] += sg[3] * Dt[c2];
        cur[c2] += Ub[c2] * ir;
        dot += Ub[c2] * U[c2];
      }
      cur[4] -= dot * ir;
    } else {
      const double m[3] = {E[(size_t)F0 * N + cell], E[(size_t)(F0 + 1) * N + cell],
                           E[(size_t)(F0 + 2) * N + cell]};
      const double rdn = E[(size_t)(F0 + 3) * N + cell];
      double sd[4];
#pragma unroll
      for (int f = 0; f < 4; ++f) sd[f] = cw * cot[(size_t)(F0 + f) * N + cell];
      double vd[3] = {0.0, 0.0, 0.0};
      if (rdn > 0.0) {
        const double id = 1.0 / rdn;
        vd[0] = m[0] * id; vd[1] = m[1] * id; vd[2] = m[2] * id;
        // S_r = m_th v_d / r + rho_d g_r, S_th = -m_r v_d / r
        cur[1] += sd[0] * 2.0 * vd[1] * invrc - sd[1] * vd[0] * invrc;
        cur[0] += -sd[1] * vd[1] * invrc;
        cur[3] += sd[0] * (-vd[1] * vd[1] * invrc) + sd[1] * (vd[0] * vd[1] * invrc);
      }
      cur[3] += sd[0] * gr + sd[2] * gz;
      const double its = omk * g.inv_st[species];
      const double st = 1.0 / g.inv_st[species];
      double dotU = 0.0, dotD = 0.0;
#pragma unroll
      for (int c2 = 0; c2 < 3; ++c2) {
        const double Ds = rdn * (vd[c2] - U[c2]) * its;
        const double Db = sg[c2] + sg[3] * U[c2] - sd[c2];
        if (rdn > 0.0) cur[c2] += its * Db;
        dotU += Db * U[c2];
        dotD += Db * Ds;
      }
      cur[3] -= its * dotU;
      stb -= dotD / st;
    }
    // all loads before any store (out may be one of the bases), each base's fields
    // requested together
    double v[NG], b1[NG], b2[NG];
    if (A.base1) {
#pragma unroll
      for (int f = 0; f < NG; ++f) b1[f] = A.base1[(size_t)(F0 + f) * N + cell];
    }
    if (A.base2) {
#pragma unroll
      for (int f = 0; f < NG; ++f) b2[f] = A.base2[(size_t)(F0 + f) * N + cell];
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) {
      v[f] = cur[f];
      if (A.base1) v[f] += b1[f];
      if (A.base2) v[f] += b2[f];
    }
#pragma unroll
    for (int f = 0; f < NG; ++f) A.out[(size_t)(F0 + f) * N + cell] = v[f];
  }
  // ---- Stokes-number partial of the block (dust)
  if constexpr (!GAS) {
    const double ws = wave_sum(stb);
    if ((tid & 63) == 0) s_red[tid / 64] = ws;
    __syncthreads();
    if (tid == 0) {
      double acc = 0.0;
      for (int w = 0; w < NT / 64; ++w) acc += s_red[w];
      A.stpart[blockIdx.x] = acc;
    }
  }
}

// z faces: one thread per column and chunk of planes, marching up; adds the four stencil
// contributions of every z face to the output written by k_adj_plane (each cell
// completed in order: its faces k-3/2 .. k+3/2, lower first).  One copy of the face, with
// k_adj_plane's short form: gas 134 -> 80 us per launch on 128 x 256 x 32, dust 44 -> 34.
template <bool GAS, int ND, bool G75>
__global__ void __launch_bounds__(256, 2) k_adj_z(AdjArgs A, int species, int tkz) {
  using C = AdjCtx<GAS>;
  constexpr int NG = C::NG;
  const C X(A, species);
  const StageArgs& a = X.a;
  const Geo& g = X.g;
  const int F0 = X.F0;
  const size_t ncol = (size_t)g.nr * g.nth;
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t col = t % ncol;
  const int kc = (int)(t / ncol);
  const int k0 = kc * tkz;
  if (k0 >= g.nz) return;
  const int k1 = min(g.nz, k0 + tkz);
  const int ig = (int)(col / g.nth), jg = (int)(col % g.nth);
  const double* E = (const double*)a.in;
  const double Az = a.t.rt[(size_t)ig * RT_N + RT_AZ];

  const RecC recc;
  double ra[NG], rb[NG], rc[NG], rd[NG];  // cells kf-1 .. kf+2 of the face kf+1/2
  auto load = [&](double* dst, int k) { load_recon<NG>(a, E, F0, k, ig, jg, dst); };
  struct ZCells {
    const double *a, *b, *c, *d;
    __device__ double operator()(int q, int f) const { return q == 0 ? a[f] : q == 1 ? b[f] : q == 2 ? c[f] : d[f]; }
    __device__ void again() {}
  };
  const ZCells zcell = {ra, rb, rc, rd};
  struct At {
    const double* b;
    __device__ double operator()(int f) const { return b[f]; }
  };
  // adds the face's contributions into oA..oD
  auto zface = [&](int kf, double* oA, double* oB, double* oC, double* oD) {
    double Fb[NG];
    X.wc_diff(kf + 1, ig, jg, kf, ig, jg, Az, Fb);
    const double* bf = a.t.wz + ((size_t)(kf + 1) * g.nr + ig) * WB_N;
    const double *bB = bg_ptr(a, kf, ig), *bC = bg_ptr(a, kf + 1, ig);
    face_vjp<2, true, GAS, G75>(X.gc, recc, zcell, nullptr, nullptr, [&](int f) { return bf[f]; },
                          At{bB}, At{bC}, Fb, oA, oB, oC, oD);
  };
  auto real = [&](int kf) { return kf >= -1 && kf <= g.nz - 1; };
  // adds the z faces' cotangent v of cell k's reconstructed variables (w: the cell's W')
  // to the cell's conservative cotangent
  auto add_out = [&](int k, const double* w, const double* v) {
    const size_t cell = ((size_t)k * g.nr + ig) * g.nth + jg;
    double ec[NG];
    cot_to_cons<GAS>(w, a.t.wc + ((size_t)k * g.nr + ig) * WB_N, X.gc.gm1, v, ec);
    double o[NG];
#pragma unroll
    for (int f = 0; f < NG; ++f) o[f] = A.out[(size_t)(F0 + f) * g.N + cell] + ec[f];
#pragma unroll
    for (int f = 0; f < NG; ++f) A.out[(size_t)(F0 + f) * g.N + cell] = o[f];
  };

  // za, zb, zc, zd: totals of the cells k-1, k, k+1, k+2 of the face k+1/2 being processed; the
  // first two faces (k0-3/2, k0-1/2) reach into the chunk from below, and what they and the
  // next give to cells below k0 is dropped
  double za[NG], zb[NG], zc[NG], zd[NG];
#pragma unroll
  for (int f = 0; f < NG; ++f) { za[f] = 0.0; zb[f] = 0.0; zc[f] = 0.0; zd[f] = 0.0; }
  const int kf0 = k0 - 2;
  load(rb, kf0 - 1); load(rc, kf0); load(rd, kf0 + 1);
  if constexpr (GAS) {
    for (int k = kf0; k <= k1; ++k) {
#pragma unroll
      for (int f = 0; f < NG; ++f) { ra[f] = rb[f]; rb[f] = rc[f]; rc[f] = rd[f]; }
      load(rd, k + 2);
      // face k+1/2 (cells k-1, k, k+1, k+2)
      if (real(k)) zface(k, za, zb, zc, zd);
      if (k - 1 >= k0) add_out(k - 1, ra, za);
#pragma unroll
      for (int f = 0; f < NG; ++f) { za[f] = zb[f]; zb[f] = zc[f]; zc[f] = zd[f]; zd[f] = 0.0; }
    }
  } else {
    // dust (registers to spare): the next plane's loads are requested one plane ahead and
    // used raw a plane later — the column's next cell, the cotangent of the next face's
    // upper cell and the output cell of the next step — so that no plane waits for memory
    const double vinv = a.t.rt[(size_t)ig * RT_N + RT_INVV];
    // w of a cell of the column from its cotangent (zero outside the grid)
    auto wcell = [&](int k, const double* x, double* w) {
      const bool in = k >= 0 && k < g.nz;
#pragma unroll
      for (int f = 0; f < NG; ++f) w[f] = in ? A.cw * vinv * x[f] : 0.0;
    };
    // a field group of cell k of the column (k clamped into the grid: a cell outside it is
    // never used)
    auto col_fetch = [&](const double* src, int k, double* x) {
      const size_t c = ((size_t)min(max(k, 0), g.nz - 1) * g.nr + ig) * g.nth + jg;
#pragma unroll
      for (int f = 0; f < NG; ++f) x[f] = src[(size_t)(F0 + f) * g.N + c];
    };
    double wlo[NG], xr[NG], orw[NG];
    {
      double x[NG];
      col_fetch(A.cot, kf0, x);
      wcell(kf0, x, wlo);
    }
    col_fetch(A.cot, kf0 + 1, xr);
    DustRaw nraw;
    dust_fetch(a, E, F0, kf0 + 2, ig, jg, nraw);
#pragma unroll
    for (int f = 0; f < NG; ++f) orw[f] = 0.0;
    for (int k = kf0; k <= k1; ++k) {
#pragma unroll
      for (int f = 0; f < NG; ++f) { ra[f] = rb[f]; rb[f] = rc[f]; rc[f] = rd[f]; }
      dust_finish(nraw, rd);  // cell k+2
      double whi[NG], ocur[NG];
      wcell(k + 1, xr, whi);
#pragma unroll
      for (int f = 0; f < NG; ++f) ocur[f] = orw[f];  // the output of cell k-1
      if (k + 1 <= k1) {
        dust_fetch(a, E, F0, k + 3, ig, jg, nraw);
        col_fetch(A.cot, k + 2, xr);
        col_fetch(A.out, max(k, k0), orw);
      }
      // face k+1/2 (cells k-1, k, k+1, k+2)
      if (real(k)) {
        double Fb[NG];
#pragma unroll
        for (int f = 0; f < NG; ++f) Fb[f] = Az * (whi[f] - wlo[f]);
        face_vjp<2, true, GAS, G75>(X.gc, recc, zcell, nullptr, nullptr, At{nullptr}, At{nullptr}, At{nullptr},
                              Fb, za, zb, zc, zd);
      }
      if (k - 1 >= k0) {
        const size_t cell = ((size_t)(k - 1) * g.nr + ig) * g.nth + jg;
        double ec[NG];
        cot_to_cons<GAS>(ra, nullptr, X.gc.gm1, za, ec);
#pragma unroll
        for (int f = 0; f < NG; ++f) A.out[(size_t)(F0 + f) * g.N + cell] = ocur[f] + ec[f];
      }
#pragma unroll
      for (int f = 0; f < NG; ++f) {
        wlo[f] = whi[f];
        za[f] = zb[f]; zb[f] = zc[f]; zc[f] = zd[f]; zd[f] = 0.0;
      }
    }
  }
}

// acc[0] += sum of parts[0 .. n) in a fixed order
__global__ void __launch_bounds__(256) k_st_accum(const double* parts, int n, double* acc) {
  __shared__ double s_s[4];
  double v = 0.0;
  for (int b = threadIdx.x; b < n; b += blockDim.x) v += parts[b];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) s_s[threadIdx.x / 64] = v;
  __syncthreads();
  if (threadIdx.x == 0) acc[0] += (s_s[0] + s_s[1]) + (s_s[2] + s_s[3]);
}

// ------------------------------------------------------------------------------------
// launchers

template <int ND>
static void adj_nd(const AdjArgs& a, int blocks, int zblocks, int tkz, int group, hipStream_t s) {
  if (group == 0) {
    if (a.s.g.gamma == 1.4) {
      hipLaunchKernelGGL((k_adj_plane<true, ND, true>), dim3(blocks), dim3(NT), 0, s, a, 0);
      if (!a.s.g.twod)
        hipLaunchKernelGGL((k_adj_z<true, ND, true>), dim3(zblocks), dim3(256), 0, s, a, 0, tkz);
    } else {
      hipLaunchKernelGGL((k_adj_plane<true, ND, false>), dim3(blocks), dim3(NT), 0, s, a, 0);
      if (!a.s.g.twod)
        hipLaunchKernelGGL((k_adj_z<true, ND, false>), dim3(zblocks), dim3(256), 0, s, a, 0, tkz);
    }
  } else {
    if constexpr (ND > 0) {
      hipLaunchKernelGGL((k_adj_plane<false, ND, true>), dim3(blocks), dim3(NT), 0, s, a, group - 1);
      if (!a.s.g.twod)
        hipLaunchKernelGGL((k_adj_z<false, ND, true>), dim3(zblocks), dim3(256), 0, s, a, group - 1,
                           tkz);
    }
  }
}

hipError_t launch_adj_group(const AdjArgs& a, int blocks, int group, hipStream_t s) {
  // z kernel: whole columns when they alone give 2048 wavefronts (8 per SIMD), else
  // chunks of 8 planes (each chunk re-solves the 3 faces below its first plane)
  const size_t ncol = (size_t)a.s.g.nr * a.s.g.nth;
  const int tkz = ncol / 64 >= 2048 ? a.s.g.nz : std::min(8, a.s.g.nz);
  const size_t nthreads = ncol * (size_t)((a.s.g.nz + tkz - 1) / tkz);
  const int zblocks = (int)((nthreads + 255) / 256);
  switch (a.s.g.nd) {
    case 0: adj_nd<0>(a, blocks, zblocks, tkz, group, s); break;
    case 1: adj_nd<1>(a, blocks, zblocks, tkz, group, s); break;
    case 2: adj_nd<2>(a, blocks, zblocks, tkz, group, s); break;
    case 3: adj_nd<3>(a, blocks, zblocks, tkz, group, s); break;
    default: adj_nd<4>(a, blocks, zblocks, tkz, group, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_st_accum(const double* parts, int nblocks, double* acc, hipStream_t s) {
  hipLaunchKernelGGL(k_st_accum, dim3(1), dim3(256), 0, s, parts, nblocks, acc);
  return hipGetLastError();
}

}  // namespace rb
