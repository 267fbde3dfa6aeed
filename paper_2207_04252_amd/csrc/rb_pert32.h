// FP32 perturbation form of the gas face flux (included by rb_device.h).
//
// The face background W0 (the stationary flow at the face, FP64) is the same on both
// sides, so the Riemann problem between W0 + W'_L and W0 + W'_R (the reconstructed
// primitive deviations) is solved for the perturbations: q = p* - p0 by Newton in FP32,
// every pressure-function term written without cancellation ((1+x)^(1/7) - 1 =
// x / sum_{k<7} y^k), the sampled state as a perturbation, and the flux returned as
// dF = F(W0 + W') - F(W0).  The empty-run
// residual is then never formed: G(E) - G(E0) = S' V - sum A dF.  Strong perturbations,
// a transonic fan or a Newton failure fall back to the FP64 solver.
#pragma once

namespace rb {

// FP32 reciprocal and square root from the hardware instructions (within an ulp or two;
// the perturbation form's accuracy target is 1e-5 relative)
__device__ __forceinline__ float rcp32(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float sqrt32(float x) { return __builtin_amdgcn_sqrtf(x); }

// stationary-flow primitives at a face in the face frame (FP64)
struct BgW {
  double rho, un, t1, t2, p, c, h;  // h = E + p per volume
};

// perturbation of a primitive face state
struct PW {
  float rho, un, t1, t2, p;
};

// flux perturbation of a primitive perturbation about the face background
__device__ __forceinline__ void flux_pert(const BgW& b, const PW& w, float inv_gm1, float out[5]) {
  const float un0 = (float)b.un, t10 = (float)b.t1, t20 = (float)b.t2;
  const float rho = (float)(b.rho + (double)w.rho);
  const float dmass = w.rho * un0 + rho * w.un;
  const float mflux = (float)(b.rho * b.un) + dmass;
  const float u0sq = (float)(b.un * b.un + b.t1 * b.t1 + b.t2 * b.t2);
  const float dot = un0 * w.un + t10 * w.t1 + t20 * w.t2;
  const float usq = w.un * w.un + w.t1 * w.t1 + w.t2 * w.t2;
  const float dke = 0.5f * w.rho * u0sq + rho * dot + 0.5f * rho * usq;
  const float dh = w.p * inv_gm1 + dke + w.p;
  const float h = (float)b.h + dh;
  out[0] = dmass;
  out[1] = dmass * un0 + mflux * w.un + w.p;
  out[2] = dmass * t10 + mflux * w.t1;
  out[3] = dmass * t20 + mflux * w.t2;
  out[4] = dh * un0 + h * w.un;
}

// one side of the perturbation Riemann problem
struct SideP {
  float pp;       // p'_K
  float p;        // p_K = p0 + p'_K
  float rho, c, A, B, irc, ip;
  float u;        // full normal velocity u0 + u'_K
  float up;       // u'_K
};

__device__ __forceinline__ SideP make_side_p(const BgW& b, const PW& w, const GasC& g) {
  SideP s;
  s.pp = w.p;
  s.p = (float)(b.p + (double)w.p);
  s.rho = (float)(b.rho + (double)w.rho);
  s.c = sqrt32((float)g.g * s.p * rcp32(s.rho));
  s.A = (float)g.a2 * rcp32(s.rho);
  s.B = (float)g.kshock * s.p;
  s.irc = rcp32(s.rho * s.c);
  s.ip = rcp32(s.p);
  s.up = w.un;
  s.u = (float)b.un + w.un;
  return s;
}

// y = (1 + x)^(1/7) (FP32 hardware log2/exp2, one Newton step) and (1 + x)^(1/7) - 1
// written as x / sum_{k<7} y^k (no cancellation for small x)
__device__ __forceinline__ void root7p(float x, float& y, float& ym1) {
  const float a = 1.0f + x;
  y = __builtin_amdgcn_exp2f(0.142857142857f * __builtin_amdgcn_logf(a));
  float y2 = y * y, y3 = y2 * y, y6 = y3 * y3;
  y = y - (y6 * y - a) * rcp32(7.0f * y6);
  y2 = y * y;
  y3 = y2 * y;
  const float s = 1.0f + y + y2 + y3 + y3 * y + y3 * y2 + y3 * y3;
  ym1 = x * rcp32(s);
}

// pressure function of one side at p* = p0 + q (gamma = 7/5): value and derivative
__device__ __forceinline__ void pfun_p(float q, const SideP& K, float& f, float& df) {
  const float d = q - K.pp;  // p* - p_K
  if (d > 0.0f) {
    const float ps = K.p + d;
    const float ipb = rcp32(ps + K.B);
    const float qs = sqrt32(K.A * ipb);
    f = d * qs;
    df = qs * (1.0f - 0.5f * d * ipb);
  } else {
    float y, ym1;
    root7p(d * K.ip, y, ym1);
    f = 5.0f * K.c * ym1;
    const float y2 = y * y, y3 = y2 * y, y6 = y3 * y3;
    df = rcp32(y6) * K.irc;
  }
}

// The star state of the perturbation Riemann problem at x/t = 0 behind the wave on its side
// (un0, p0: normal velocity and pressure of the background); last: Newton iterations.  Returns
// false when the FP64 solver must be used instead.
__device__ __forceinline__ bool star_pert(float un0, float p0, const PW& WL, const PW& WR,
                                          const SideP& L, const SideP& R, const GasC& g, PW& W,
                                          int& last) {
  const float du = WR.un - WL.un;
  // Newton on q = p* - p0 from the primitive-variable guess
  float q = 0.5f * (WL.p + WR.p) - 0.125f * du * (L.rho + R.rho) * (L.c + R.c);
  const float qfloor = 1e-8f * fminf(L.p, R.p) - p0;
  q = fmaxf(q, qfloor);
  float fL = 0.f, dL = 1.f, fR = 0.f, dR = 1.f, dq = 0.f;
  bool conv = false;
  int it = 0;
  while (it < 20) {
    ++it;
    pfun_p(q, L, fL, dL);
    pfun_p(q, R, fR, dR);
    float qn = q - (fL + fR + du) * rcp32(dL + dR);
    qn = fmaxf(qn, 1e-8f * (p0 + q) - p0);
    dq = qn - q;
    q = qn;
    if (fabsf(dq) <= 1e-6f * fabsf(q) + 1e-9f * p0) { conv = true; break; }
  }
  last = it;
  if (!conv) return false;
  const float us = 0.5f * (WL.un + WR.un) + 0.5f * ((fR + dR * dq) - (fL + dL * dq));
  const float usfull = un0 + us;
  const float kk = (float)g.kshock;
  if (0.0f <= usfull) {
    if (q > WL.p) {
      const float x = (q - WL.p) * L.ip;
      const float sL = L.u - L.c * sqrt32((float)g.gp1_2g * (1.0f + x) + (float)g.gm1_2g);
      if (0.0f <= sL) { W = WL; return true; }
      const float rm1 = x * (1.0f - kk) * rcp32(kk * (1.0f + x) + 1.0f);
      W.rho = WL.rho + L.rho * rm1;
    } else {
      if (0.0f <= L.u - L.c) { W = WL; return true; }
      float y, ym1;
      root7p((q - WL.p) * L.ip, y, ym1);
      if (!(0.0f > usfull - L.c * y)) return false;  // transonic fan: FP64
      const float y5m1 = ym1 * (1.0f + y + y * y + y * y * y + y * y * y * y);
      W.rho = WL.rho + L.rho * y5m1;
    }
    W.un = us; W.p = q; W.t1 = WL.t1; W.t2 = WL.t2;
    return true;
  }
  if (q > WR.p) {
    const float x = (q - WR.p) * R.ip;
    const float sR = R.u + R.c * sqrt32((float)g.gp1_2g * (1.0f + x) + (float)g.gm1_2g);
    if (0.0f >= sR) { W = WR; return true; }
    const float rm1 = x * (1.0f - kk) * rcp32(kk * (1.0f + x) + 1.0f);
    W.rho = WR.rho + R.rho * rm1;
  } else {
    if (0.0f >= R.u + R.c) { W = WR; return true; }
    float y, ym1;
    root7p((q - WR.p) * R.ip, y, ym1);
    if (!(0.0f <= usfull + R.c * y)) return false;
    const float y5m1 = ym1 * (1.0f + y + y * y + y * y * y + y * y * y * y);
    W.rho = WR.rho + R.rho * y5m1;
  }
  W.un = us; W.p = q; W.t1 = WR.t1; W.t2 = WR.t2;
  return true;
}

// Perturbation exact Riemann problem (gamma = 7/5) at x/t = 0.  Returns false when the
// FP64 solver must be used instead.
__device__ __forceinline__ bool riemann_pert(const BgW& b, const PW& WL, const PW& WR, const GasC& g,
                                             PW& W, TStat& st) {
  st.last = 0;
  // strong perturbations are left to the FP64 solver
  const float p0 = (float)b.p, r0 = (float)b.rho, c0 = (float)b.c;
  if (!(fabsf(WL.p) < 0.1f * p0 && fabsf(WR.p) < 0.1f * p0 && fabsf(WL.rho) < 0.1f * r0 &&
        fabsf(WR.rho) < 0.1f * r0 && fabsf(WL.un) < 0.1f * c0 && fabsf(WR.un) < 0.1f * c0))
    return false;
  const SideP L = make_side_p(b, WL, g);
  const SideP R = make_side_p(b, WR, g);
  const float du = WR.un - WL.un;
  // supersonic faces: the left (right) state is the solution when f(p_hi) >= 0 and the
  // contact moves the same way (same argument as the FP64 solver, with margins)
  if (L.u >= L.c) {
    const float m = L.u * rcp32(L.c);
    const float phi = L.p * (m * m - (float)g.gm1_2g) * (float)g.inv_gp1_2g;
    float fL, dL, fR, dR;
    pfun_p(phi - p0, L, fL, dL);
    pfun_p(phi - p0, R, fR, dR);
    if (fL + fR + du >= 1e-3f * fL && L.u - fL >= 1e-3f * L.u) {
      W = WL;
      return true;
    }
  } else if (R.u <= -R.c) {
    const float m = -R.u * rcp32(R.c);
    const float phi = R.p * (m * m - (float)g.gm1_2g) * (float)g.inv_gp1_2g;
    float fL, dL, fR, dR;
    pfun_p(phi - p0, L, fL, dL);
    pfun_p(phi - p0, R, fR, dR);
    if (fL + fR + du >= 1e-3f * fR && R.u + fR <= 1e-3f * R.u) {
      W = WR;
      return true;
    }
  }
  const bool ok = star_pert((float)b.un, p0, WL, WR, L, R, g, W, st.last);
  st.maxit = max(st.maxit, st.last);
  return ok;
}

// Flux perturbation about a background that flows along theta only (F in field slots), DIR the
// normal: flux_pert's own roundings without its products with zero velocities.
template <int DIR>
__device__ __forceinline__ void flux_pert_az(const PertBg& b, const PW& w, float* F) {
#pragma clang fp contract(off)
  const float v0 = b.cell.v, rho = (float)(b.cell.rho + (double)w.rho);
  const float vp = DIR == 0 ? w.t1 : DIR == 1 ? w.un : w.t2;  // velocity along theta
  const float usq = fmaf(w.t2, w.t2, fmaf(w.un, w.un, w.t1 * w.t1));
  const float dke = fmaf(0.5f * rho, usq, fmaf(0.5f * w.rho, b.cell.vsq, rho * (v0 * vp)));
  const float dh = fmaf(w.p, 2.5f, dke) + w.p;
  const float h = b.h + dh;
  if constexpr (DIR == 1) {
    const float dmass = fmaf(w.rho, v0, rho * w.un), mflux = b.rhov + dmass;
    F[4] = dmass;
    F[1] = fmaf(dmass, v0, mflux * w.un) + w.p;
    F[0] = mflux * w.t1;
    F[2] = mflux * w.t2;
    F[3] = fmaf(dh, v0, h * w.un);
  } else {
    const float dmass = rho * w.un;
    F[4] = dmass;
    F[DIR] = dmass * w.un + w.p;
    F[1] = fmaf(dmass, v0, dmass * vp);
    F[2 - DIR] = dmass * (DIR == 0 ? w.t2 : w.t1);
    F[3] = h * w.un;
  }
}

// The short form of a face, for weak perturbations about a flow without radial and vertical
// velocity (gamma = 7/5; qL, qR: the face states W' in field slots, b: the face's background).
// Its results are the general form's to the last bit.  The state's FP64 part depends on that:
// the dust density, accumulated in FP64, follows the gas velocity through the drag, so that a
// change of rounding in a face moves it by up to 1e-6 in single cells of split exact drag.
// Returns false where it does not apply: a perturbation above a tenth of the background (the
// general form leaves those to FP64), a star state that the general form leaves to FP64,
// azimuthal flow below Mach 2, or densities in units with which riemann_pert's products leave
// the FP32 range.
//
// Azimuthal faces: with the flow above Mach 2 and the perturbations below a tenth, u_L is above
// 1.7 c_L, so the pressure p_hi of a standing left shock is above 3.2 p_L, more than p_R; f_L
// there is above 0.9 c_L, more than u_L - u_R, and f_R is positive, so riemann_pert's proof that
// the left state is the solution holds for every such face: no solve.
// Radial and vertical faces: the background has no normal flow, so they are subsonic and need
// the star state only.
template <int DIR>
__device__ __forceinline__ bool gas_face32(const PertBg& b, const float* qL, const float* qR,
                                           float* F, int& last) {
  constexpr int N = Dirs<DIR>::n, T1 = Dirs<DIR>::t1, T2 = Dirs<DIR>::t2;
  const float r0 = (float)b.cell.rho, p0 = (float)b.p, c0 = b.c;
  const float unit = r0 * p0;
  bool ok = fabsf(qL[3]) < 0.1f * p0 && fabsf(qR[3]) < 0.1f * p0 && fabsf(qL[4]) < 0.1f * r0 &&
            fabsf(qR[4]) < 0.1f * r0 && fabsf(qL[N]) < 0.1f * c0 && fabsf(qR[N]) < 0.1f * c0 &&
            unit > 1e-30f && unit < 1e30f;
  last = 0;
  const PW WL = {qL[4], qL[N], qL[T1], qL[T2], qL[3]};
  if constexpr (DIR == 1) {
    ok = ok && b.cell.v >= 2.0f * c0;
    flux_pert_az<DIR>(b, WL, F);
  } else {
    const PW WR = {qR[4], qR[N], qR[T1], qR[T2], qR[3]};
    const GasC g = gas_consts(1.4);
    PW W = WL;
    if (ok) {
      const BgW bg = {b.cell.rho, 0.0, 0.0, 0.0, b.p, 0.0, 0.0};
      ok = star_pert(0.0f, p0, WL, WR, make_side_p(bg, WL, g), make_side_p(bg, WR, g), g, W, last);
    }
    flux_pert_az<DIR>(b, W, F);
  }
  return ok;
}

}  // namespace rb
