// Device-side building blocks shared by the forward stage kernels and the adjoint
// kernels: reconstruction, exact gas and pressureless dust Riemann solvers, face
// fluxes, state access with ghost cells, wave reductions, tile order.
#pragma once

#include <math.h>

#include <type_traits>

#include "rb_internal.h"

namespace rb {

// ------------------------------------------------------------------------------------
// small helpers

// Read-only tables by scalar loads: constant address space, for indexes that are the same in
// every lane of a wavefront.  Only tables that no kernel writes while the reading one runs.
using ctab = const __attribute__((address_space(4))) double*;
__device__ __forceinline__ ctab to_ctab(const double* p) { return (ctab)(uintptr_t)p; }

// A PertBg entry of a table, likewise.
__device__ __forceinline__ PertBg pert_at(const double* table, size_t entry) {
  const ctab t = to_ctab(table) + entry * PF_D;
  double d[PF_D];
#pragma unroll
  for (int q = 0; q < PF_D; ++q) d[q] = t[q];
  PertBg b;
  __builtin_memcpy(&b, d, sizeof b);
  return b;
}

// Minmod of three in FP32: minmod(a, b) is the median of a, b and 0, and minmod of three is
// minmod(x, minmod(y, z)): two hardware medians, each returning one of its arguments.
__device__ __forceinline__ float minmod3(float x, float y, float z) {
  return __builtin_amdgcn_fmed3f(x, __builtin_amdgcn_fmed3f(y, z, 0.0f), 0.0f);
}

// Uniform direction (index coordinates): the three-point parabola gives the upper-face
// increment (dm + 3 dp)/8 and the lower-face increment -(3 dm + dp)/8, limited by the
// one-sided differences (Sect. 2.7).  Written so that mirrored data give exactly
// opposite increments.
__device__ __forceinline__ float inc_up_u(float em, float e0, float ep) {
  const float dm = e0 - em, dp = ep - e0;
  return minmod3(fma(3.0f, dp, dm) * 0.125f, dm, dp);
}
__device__ __forceinline__ float inc_lo_u(float em, float e0, float ep) {
  const float dm = e0 - em, dp = ep - e0;
  return minmod3(-(fma(3.0f, dm, dp) * 0.125f), -dm, -dp);
}
// Non-uniform r: precomputed parabola weights and limiter bounds of the cell.
__device__ __forceinline__ float inc_up_c(float em, float e0, float ep, const float* co) {
  const float dm = e0 - em, dp = ep - e0;
  return minmod3(fma(co[RC_WPP], dp, co[RC_WPM] * dm), co[RC_LPM] * dm, co[RC_LPP] * dp);
}
__device__ __forceinline__ float inc_lo_c(float em, float e0, float ep, const float* co) {
  const float dm = e0 - em, dp = ep - e0;
  return minmod3(fma(co[RC_WMP], dp, co[RC_WMM] * dm), co[RC_LMM] * dm, co[RC_LMP] * dp);
}

// Constants of the pair reconstruction, in scalar registers: written as literals they cost a
// register copy per multiply-add and a slower exponent shift.
struct RecC {
  double three, eighth;
  __device__ __forceinline__ RecC() : three(3.0), eighth(0.125) {
    asm("" : "+s"(three), "+s"(eighth));
  }
};

// Both limited states of the face between cells B and C in FP64 (the same values as B plus
// inc_up and C plus inc_lo).  With d1 = B - A, d2 = C - B, d3 = D - C and s the sign of d2,
// the three arguments of either limiter share a sign exactly when s d1 (or s d3) is not
// negative -- the parabola's weights are positive, so its increment then has that sign too
// -- and the limited magnitude is max(0, min of the three) in the signed variables; s
// returns in the final multiply-add.  The stage kernels are bound by instruction issue and
// the chains between barriers: 19 instructions a field (23 along r) against 26 for the two
// limiters taken apart.  With dust_face's one-way path below, the step of the three-dust
// disc 512 x 1024 x 128 in the FP32-perturbation form went from 25.0 to 22.1 ms (dust launch
// 2.40 -> 1.92 ms), the one-dust disc 256 x 512 x 64 in FP64 from 2.34 to 2.24 ms.
template <int DIR, class Co>
__device__ __forceinline__ void face_pair(const RecC& rc, double A, double B, double C, double D,
                                          Co coB, Co coC, double& L, double& R) {
  const double d1 = B - A, d2 = C - B, d3 = D - C;
  const double s = copysign(1.0, d2), a = fabs(d2);
  const double b1 = s * d1, b3 = s * d3;
  double up, lo;
  if constexpr (DIR == 0) {
    up = fmin(fmin(fma(coB[RC_WPP], a, coB[RC_WPM] * b1), coB[RC_LPP] * a), coB[RC_LPM] * b1);
    lo = fmin(fmin(fma(-coC[RC_WMP], b3, -coC[RC_WMM] * a), -coC[RC_LMM] * a), -coC[RC_LMP] * b3);
  } else {
    up = fmin(fmin(fma(rc.three, a, b1) * rc.eighth, a), b1);
    lo = fmin(fmin(fma(rc.three, a, b3) * rc.eighth, a), b3);
  }
  L = fma(s, fmax(up, 0.0), B);
  R = fma(-s, fmax(lo, 0.0), C);
}

// true when the condition holds in no active lane of the wavefront (a scalar test)
__device__ __forceinline__ bool wave_none(bool c) { return __builtin_amdgcn_ballot_w64(c) == 0; }

// Orders what the lanes of a wavefront read of each other's LDS entries before against what
// they write after.  The hardware keeps one wavefront's LDS accesses in order; this keeps the
// compiler, which reasons about one lane, from moving them (no instruction).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// x^(-1/7) for x > 0: FP32 hardware log2/exp2 seed (relative error ~1e-7 for x in the
// clamped range), then Newton on z^-7 = x written as z <- z + (z/7)(1 - x z^7), whose error
// goes e -> 4 e^2: two steps reach FP64 rounding (4 (4e-14)^2 ~ 1e-26); x = 1 is a fixed
// point.
__device__ __forceinline__ double inv_root7(double x) {
  if (x == 1.0) return 1.0;
  float xf = fminf(fmaxf((float)x, 1e-30f), 1e30f);
  double z = (double)__builtin_amdgcn_exp2f(-0.142857142857142857f * __builtin_amdgcn_logf(xf));
  const double k7 = 1.0 / 7.0;
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    double z2 = z * z;
    double z3 = z2 * z;
    double z7 = z3 * z3 * z;
    z = fma(z * k7, fma(-x, z7, 1.0), z);
  }
  return z;
}

// 1/x for normal positive or negative x: hardware estimate and two Newton steps
// (within an ulp of the correctly rounded quotient).
__device__ __forceinline__ double frcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// 1/sqrt(x) for normal positive x: hardware estimate and two Newton steps
// r <- r (3/2 - x r^2 / 2) (error e -> 3/2 e^2; within an ulp or two of the rounded value).
__device__ __forceinline__ double frsq(double x) {
  double r = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  r = r * fma(-h * r, r, 1.5);
  r = r * fma(-h * r, r, 1.5);
  return r;
}

struct GasC {
  double g, gm1, inv_gm1, g2m1, gm1_2g, gp1_2g, kshock, a2, half_gm1, inv_g, inv_gp1_2g, inv_a2;
  int max_iter;  // Newton iteration cap
};

__device__ __forceinline__ GasC gas_consts(double g, int max_iter = 50) {
  GasC c;
  c.max_iter = max_iter;
  c.g = g;
  c.gm1 = g - 1.0;
  c.inv_gm1 = 1.0 / (g - 1.0);
  c.g2m1 = 2.0 / (g - 1.0);
  c.gm1_2g = (g - 1.0) / (2.0 * g);
  c.gp1_2g = (g + 1.0) / (2.0 * g);
  c.kshock = (g - 1.0) / (g + 1.0);
  c.a2 = 2.0 / (g + 1.0);
  c.half_gm1 = 0.5 * (g - 1.0);
  c.inv_g = 1.0 / g;
  c.inv_gp1_2g = (2.0 * g) / (g + 1.0);
  c.inv_a2 = 0.5 * (g + 1.0);
  return c;
}

// Powers of x = p/p_K needed by the exact solver: x^((g-1)/2g), x^(-(g+1)/2g), x^(1/g).
// With g = 7/5 they are x^(1/7), x^(-6/7), x^(5/7), all from one x^(-1/7).
template <bool G75> struct Pow3 {
  double p17, pm67, p57;
  __device__ __forceinline__ Pow3(double x, const GasC& c) {
    if (G75) {
      double z = inv_root7(x);
      double z2 = z * z;
      double z6 = z2 * z2 * z2;
      p17 = x * z6;
      pm67 = z6;
      p57 = x * z2;
    } else {
      p17 = pow(x, c.gm1_2g);
      pm67 = pow(x, -c.gp1_2g);
      p57 = pow(x, 1.0 / c.g);
    }
  }
};

template <bool G75>
__device__ __forceinline__ double ipow_fan_rho(double ratio, const GasC& c) {
  if (G75) { double r2 = ratio * ratio; return r2 * r2 * ratio; }
  return pow(ratio, c.g2m1);
}
template <bool G75>
__device__ __forceinline__ double ipow_fan_p(double ratio, const GasC& c) {
  if (G75) { double r2 = ratio * ratio; double r3 = r2 * ratio; return r3 * r3 * ratio; }
  return pow(ratio, 2.0 * c.g / (c.g - 1.0));
}

// One side of the pressure function of the exact solver (Sect. 2.6) and its derivative.
// Per-side constants of the pressure function: A = 2/((g+1) rho), B = (g-1)/(g+1) p,
// 1/p and 1/(rho c).
struct Side {
  double r, u, p, c, A, B, ip, irc, iA;
};

// c and 1/c of the side come in as c2 * rs and rs, rs = 1/sqrt(c2)
__device__ __forceinline__ Side make_side(double r, double ir, double u, double p, double c,
                                          double rs, const GasC& g) {
  Side s;
  s.r = r; s.u = u; s.p = p; s.c = c;
  s.A = g.a2 * ir;
  s.B = g.kshock * p;
  s.ip = frcp(p);
  s.irc = ir * rs;
  s.iA = r * g.inv_a2;
  return s;
}

template <bool G75>
__device__ __forceinline__ void pfun(double p, const Side& K, const GasC& c, double& f,
                                     double& df) {
  if (p > K.p) {
    // q = sqrt(A / (p + B)) = 1/sqrt((p + B)/A) and 1/(p + B) = q^2 / A
    const double q = frsq((p + K.B) * K.iA);
    const double ipb = q * q * K.iA;
    f = (p - K.p) * q;
    df = q * (1.0 - 0.5 * (p - K.p) * ipb);
  } else {
    Pow3<G75> w(p * K.ip, c);
    f = c.g2m1 * K.c * (w.p17 - 1.0);
    df = w.pm67 * K.irc;
  }
}

struct TStat {
  int fall, vac, maxit, noconv, resolve;
  int last;  // Newton iterations of the latest gas solve (0: none was needed)
  int negd;  // dust densities that came out negative
};

// Wave pattern taken by the exact gas solver at x/t = 0 (kept by the adjoint, which
// differentiates the branch the primal solve took).
enum : int {
  GR_LEFT = 0,      // the left state
  GR_RIGHT,         // the right state
  GR_FAN_L,         // inside the left rarefaction fan
  GR_FAN_R,         // inside the right rarefaction fan
  GR_VACUUM,        // inside a vacuum region
  GR_STAR_L_SHOCK,  // left star state behind a shock
  GR_STAR_L_RARE,   // left star state behind a rarefaction
  GR_STAR_R_SHOCK,
  GR_STAR_R_RARE
};
struct GasRec {
  int branch;
  double ps, us;                 // star pressure and velocity (star branches)
  double rho, un, t1, t2, p;     // the sampled state
};

// Exact Riemann problem of the ideal gas sampled at x/t = 0 (Sect. 2.6): Newton on p*
// from the primitive-variable guess (relative change <= 1e-12, at most c.max_iter),
// star velocity, then the wave pattern at x/t = 0; tangential velocities come from the
// side of the contact.  Output: mass, normal momentum, two tangential momenta, energy.
template <bool G75, bool REC = false>
__device__ void gas_riemann(const GasC& c, double rL, double irL, double uL, double aL, double bL,
                            double pL, double rR, double irR, double uR, double aR, double bR,
                            double pR, double fl[5], TStat& st, GasRec* rec = nullptr) {
  const double du = uR - uL;
  const double c2L = c.g * pL * irL, c2R = c.g * pR * irR;
  // Supersonic faces.  With u_L >= c_L, let p_hi be the star pressure at which a left
  // shock would stand still, p_hi = (rho_L u_L^2 / g - (g-1)/(2g) p_L) (2g)/(g+1).  If
  // p_hi >= p_R then f_R(p_hi) >= 0, and f_L(p_hi) + du >= 0 gives f(p_hi) >= 0, so
  // p* <= p_hi (f increases): the left wave (rarefaction with head u_L - c_L >= 0, or shock
  // with speed >= 0) lies at x/t >= 0, and u* = u_L - f_L(p*) >= u_L - f_L(p_hi) >= 0: the
  // solution at x/t = 0 is the left state, which is what the full solve returns.  Both
  // tests are taken on squares (f_L(p_hi)^2 = (p_hi - p_L)^2 A_L / (p_hi + B_L)), so no
  // square root or division is needed; faces that may open a vacuum are left to the full
  // solve.  Mirror for u_R <= -c_R.
  {
    const double g2 = c.g2m1 * c.g2m1;
    const bool novac_L = du <= 0.0 || du * du < g2 * c2L;
    const bool novac_R = du <= 0.0 || du * du < g2 * c2R;
    if (uL > 0.0 && uL * uL >= c2L && novac_L) {
      const double u2 = uL * uL;
      const double phi = (rL * u2 * c.inv_g - c.gm1_2g * pL) * c.inv_gp1_2g;
      if (phi >= pR) {
        const double D = phi - pL;
        const double D2A = D * D * (c.a2 * irL);
        const double pb = phi + c.kshock * pL;
        if ((du >= 0.0 || D2A >= du * du * pb) && u2 * pb >= D2A) {
          if constexpr (REC) {
            rec->branch = GR_LEFT;
            rec->rho = rL; rec->un = uL; rec->t1 = aL; rec->t2 = bL; rec->p = pL;
          }
          st.last = 0;
          const double m0 = rL * uL;
          const double en = pL * c.inv_gm1 + 0.5 * rL * (uL * uL + aL * aL + bL * bL);
          fl[0] = m0; fl[1] = m0 * uL + pL; fl[2] = m0 * aL; fl[3] = m0 * bL; fl[4] = (en + pL) * uL;
          return;
        }
      }
    } else if (uR < 0.0 && uR * uR >= c2R && novac_R) {
      const double u2 = uR * uR;
      const double phi = (rR * u2 * c.inv_g - c.gm1_2g * pR) * c.inv_gp1_2g;
      if (phi >= pL) {
        const double D = phi - pR;
        const double D2A = D * D * (c.a2 * irR);
        const double pb = phi + c.kshock * pR;
        if ((du >= 0.0 || D2A >= du * du * pb) && u2 * pb >= D2A) {
          if constexpr (REC) {
            rec->branch = GR_RIGHT;
            rec->rho = rR; rec->un = uR; rec->t1 = aR; rec->t2 = bR; rec->p = pR;
          }
          st.last = 0;
          const double m0 = rR * uR;
          const double en = pR * c.inv_gm1 + 0.5 * rR * (uR * uR + aR * aR + bR * bR);
          fl[0] = m0; fl[1] = m0 * uR + pR; fl[2] = m0 * aR; fl[3] = m0 * bR; fl[4] = (en + pR) * uR;
          return;
        }
      }
    }
  }
  const double rsL = frsq(c2L), rsR = frsq(c2R);
  const double cL = c2L * rsL;
  const double cR = c2R * rsR;
  double rho, un, t1, t2, p;
  if (c.g2m1 * (cL + cR) <= du) {
    // vacuum between two rarefactions
    st.vac++;
    st.last = 0;
    double sHL = uL - cL, sSL = uL + c.g2m1 * cL, sSR = uR - c.g2m1 * cR, sHR = uR + cR;
    int br;
    if (0.0 <= sHL) { rho = rL; un = uL; t1 = aL; t2 = bL; p = pL; br = GR_LEFT; }
    else if (0.0 < sSL) {
      double cc = c.a2 * (cL + c.half_gm1 * uL);
      double ratio = cc / cL;
      rho = rL * ipow_fan_rho<G75>(ratio, c); un = cc; p = pL * ipow_fan_p<G75>(ratio, c);
      t1 = aL; t2 = bL; br = GR_FAN_L;
    } else if (0.0 <= sSR) { rho = 0.0; un = 0.0; t1 = 0.0; t2 = 0.0; p = 0.0; br = GR_VACUUM; }
    else if (0.0 < sHR) {
      double cc = c.a2 * (cR - c.half_gm1 * uR);
      double ratio = cc / cR;
      rho = rR * ipow_fan_rho<G75>(ratio, c); un = -cc; p = pR * ipow_fan_p<G75>(ratio, c);
      t1 = aR; t2 = bR; br = GR_FAN_R;
    } else { rho = rR; un = uR; t1 = aR; t2 = bR; p = pR; br = GR_RIGHT; }
    if constexpr (REC) rec->branch = br;
  } else {
    const Side L = make_side(rL, irL, uL, pL, cL, rsL, c);
    const Side R = make_side(rR, irR, uR, pR, cR, rsR, c);
    double ppv = 0.5 * (pL + pR) - 0.125 * du * (rL + rR) * (cL + cR);
    double ps = fmax(ppv, 1e-8 * fmin(pL, pR));
    int it = 0;
    bool conv = false;
    double fL = 0.0, dL = 1.0, fR = 0.0, dR = 1.0, dp = 0.0;
    while (it < c.max_iter) {
      ++it;
      pfun<G75>(ps, L, c, fL, dL);
      pfun<G75>(ps, R, c, fR, dR);
      double pn = ps - (fL + fR + du) / (dL + dR);
      if (pn < 1e-8 * ps) pn = 1e-8 * ps;
      dp = pn - ps;
      // relative change 2|dp|/(p_new + p_old) <= 1e-12, written without a division
      bool done = 2.0 * fabs(dp) <= 1e-12 * (pn + ps);
      ps = pn;
      if (done) { conv = true; break; }
    }
    st.maxit = max(st.maxit, it);
    st.last = it;
    if (!conv) st.noconv = 1;
    // star velocity at the converged p*: the last iterate's f and f' extrapolated over
    // the final (<= 1e-12 relative) Newton update; the neglected term is O(dp^2)
    double us = 0.5 * (uL + uR) + 0.5 * ((fR + dR * dp) - (fL + dL * dp));
    p = ps;
    int br;
    if (0.0 <= us) {
      t1 = aL; t2 = bL;
      if (ps > pL) {
        double q = ps * L.ip;
        double sL = uL - cL * sqrt(c.gp1_2g * q + c.gm1_2g);
        if (0.0 <= sL) { rho = rL; un = uL; p = pL; br = GR_LEFT; }
        else { rho = rL * (q + c.kshock) * frcp(c.kshock * q + 1.0); un = us; br = GR_STAR_L_SHOCK; }
      } else {
        double sHL = uL - cL;
        if (0.0 <= sHL) { rho = rL; un = uL; p = pL; br = GR_LEFT; }
        else {
          Pow3<G75> w(ps * L.ip, c);
          double sTL = us - cL * w.p17;
          if (0.0 > sTL) { rho = rL * w.p57; un = us; br = GR_STAR_L_RARE; }
          else {
            double cc = c.a2 * (cL + c.half_gm1 * uL);
            double ratio = cc / cL;
            rho = rL * ipow_fan_rho<G75>(ratio, c); un = cc; p = pL * ipow_fan_p<G75>(ratio, c);
            br = GR_FAN_L;
          }
        }
      }
    } else {
      t1 = aR; t2 = bR;
      if (ps > pR) {
        double q = ps * R.ip;
        double sR = uR + cR * sqrt(c.gp1_2g * q + c.gm1_2g);
        if (0.0 >= sR) { rho = rR; un = uR; p = pR; br = GR_RIGHT; }
        else { rho = rR * (q + c.kshock) * frcp(c.kshock * q + 1.0); un = us; br = GR_STAR_R_SHOCK; }
      } else {
        double sHR = uR + cR;
        if (0.0 >= sHR) { rho = rR; un = uR; p = pR; br = GR_RIGHT; }
        else {
          Pow3<G75> w(ps * R.ip, c);
          double sTR = us + cR * w.p17;
          if (0.0 <= sTR) { rho = rR * w.p57; un = us; br = GR_STAR_R_RARE; }
          else {
            double cc = c.a2 * (cR - c.half_gm1 * uR);
            double ratio = cc / cR;
            rho = rR * ipow_fan_rho<G75>(ratio, c); un = -cc; p = pR * ipow_fan_p<G75>(ratio, c);
            br = GR_FAN_R;
          }
        }
      }
    }
    if constexpr (REC) { rec->branch = br; rec->ps = ps; rec->us = us; }
  }
  if constexpr (REC) { rec->rho = rho; rec->un = un; rec->t1 = t1; rec->t2 = t2; rec->p = p; }
  double en = p * c.inv_gm1 + 0.5 * rho * (un * un + t1 * t1 + t2 * t2);
  double m = rho * un;
  fl[0] = m;
  fl[1] = m * un + p;
  fl[2] = m * t1;
  fl[3] = m * t2;
  fl[4] = (en + p) * un;
}

// Exact pressureless Riemann problem at x/t = 0 (Sect. 2.9): diverging or equal streams
// leave vacuum between them (upwind state or zero flux); converging streams form a
// delta shock of speed (sqrt(rho_L) u_L + sqrt(rho_R) u_R)/(sqrt(rho_L) + sqrt(rho_R)),
// the flux being the upwind one and the mean of both at a standing shock.  The sign
// of the shock speed is formed without contraction so that mirrored states give zero.
// With REC the side taken is stored in *rec: -1 left, +1 right, 0 mean, 2 no flux.
template <bool REC = false>
__device__ void dust_riemann(double rL, double uL, double aL, double bL, double rR, double uR,
                             double aR, double bR, double fl[4], int* rec = nullptr) {
#pragma clang fp contract(off)
  fl[0] = 0.0; fl[1] = 0.0; fl[2] = 0.0; fl[3] = 0.0;
  if constexpr (REC) *rec = 2;
  if (!(rL > 0.0)) { rL = 0.0; uL = 0.0; aL = 0.0; bL = 0.0; }
  if (!(rR > 0.0)) { rR = 0.0; uR = 0.0; aR = 0.0; bR = 0.0; }
  if (rL + rR == 0.0) return;
  int side;  // -1 left, +1 right, 0 mean
  if (uL <= uR) {
    if (uL > 0.0) side = -1;
    else if (uR < 0.0) side = 1;
    else return;
  } else {
    // delta shock: its speed has the sign of sqrt(rL) uL + sqrt(rR) uR.  With uL > uR,
    // both terms share a sign unless uL > 0 > uR, where the sign is that of
    // rL uL^2 - rR uR^2 (both sides squared, no square root); mirror-symmetric states
    // give exactly zero either way
    if (uR >= 0.0 && uL > 0.0) side = -1;
    else if (uL <= 0.0 && uR < 0.0) side = 1;
    else {
      const double d = rL * uL * uL - rR * uR * uR;
      side = d > 0.0 ? -1 : (d < 0.0 ? 1 : 0);
    }
  }
  if constexpr (REC) *rec = side;
  double mL = rL * uL, mR = rR * uR;
  if (side < 0) { fl[0] = mL; fl[1] = mL * uL; fl[2] = mL * aL; fl[3] = mL * bL; }
  else if (side > 0) { fl[0] = mR; fl[1] = mR * uR; fl[2] = mR * aR; fl[3] = mR * bR; }
  else {
    fl[0] = 0.5 * (mL + mR);
    fl[1] = 0.5 * (mL * uL + mR * uR);
    fl[2] = 0.5 * (mL * aL + mR * aR);
    fl[3] = 0.5 * (mL * bL + mR * bR);
  }
}

// normal / tangential velocity slots of direction DIR (0 r, 1 theta, 2 z)
template <int DIR> struct Dirs {
  static constexpr int n = DIR;
  static constexpr int t1 = DIR == 0 ? 1 : 0;
  static constexpr int t2 = DIR == 2 ? 1 : 2;
};

// ------------------------------------------------------------------------------------
// Face states and fluxes.  The parabola and MinMod limiter of Sect. 2.7 act on the
// primitive form of the variables: the gas velocity, pressure and density as deviations
// W' = W(E) - W(E0) from the stationary flow, each dust fluid's velocity and density
// whole.  A gas face state is W0(face) + W'(cell) + limited increment; only the flux of
// the Riemann solution, F* = F(E*), is formed from the face states (Sect. 2.6).

// The short form of an FP64 gas face (gamma = 7/5; qL, qR full face states in field slots).
// Returns false where it does not apply (the general form solves those): a non-positive
// state, a perturbation p*/p_K - 1 above 1/16, normal velocities above 0.9 c, no convergence,
// or a supersonic face on which the left state is not proved to be the solution.
//
// Supersonic to the right: gas_riemann's proof that the left state is the solution.
// Otherwise, with x = p / p_K - 1 small both branches of a side's pressure function are
// polynomials (f = 5/7 c x g(x), f' = D(x) / (rho c)), and so are both densities
// (rho* = rho_K (1 + x R(x))); with x and the velocities so bounded the state at x/t = 0 is
// the star state.  The polynomials interpolate at the Chebyshev nodes of [-X, 0] or [0, X]:
// relative error below 2.5e-17 with degree 4 for X = 1/512 and degree 8 for X = 1/16 (D:
// 5e-8 with degree 2 and 5e-11 with degree 5, enough that Newton takes the same steps).  f's
// error is then 1e-16 f, where the general form's difference of a root from 1 leaves 1e-16 c.
// A Newton step costs some 50 instructions (x below 1/512) instead of 150: the general form
// runs both branches of both sides wherever a wavefront's lanes differ.
// Each lane takes the polynomials of its own range: the two ranges' values differ in the last
// bit, and a face that two workgroups solve, beside other faces in each, has one flux.
// Their coefficients, highest degree first, rarefaction and shock in turn (D of the narrow
// range: one for both): g, D, R for X = 1/512, then for X = 1/16; the constant terms are 1, 1
// and 5/7.  Read by scalar loads where they are used: as literals they would be kept in
// registers across the march, and spilled.
enum : int { WK_G = 0, WK_D = 8, WK_R = 10, WKW_G = 18, WKW_D = 34, WKW_R = 44 };
static __constant__ double weak_coef[60] = {
    0.1467684060227819, 0.14703985203134992, -0.1895033823370895, -0.19679205462062704,
    0.26530612314052177, 0.2755102034197363, -0.42857142857125957, -0.42857142857126684,
    0.811186511, -0.8571412, 0.016479224249694835, 0.0002970904304251677,
    -0.024989489144093765, -0.00208246450518904, 0.04373177849459193, 0.014577259474031863,
    -0.10204081632651371, -0.10204081632653021, 0.09561162951996895, 0.04576086710171662,
    -0.08223027042671534, -0.06991785492880287, 0.09919333961673185, 0.0893809409570641,
    -0.11833715584013775, -0.11385591256242655, 0.14618922734393267, 0.14759468994287225,
    -0.1895043714738181, -0.19679300216171694, 0.2653061224593831, 0.27551020407704946,
    -0.4285714285714042, -0.42857142857141783, -0.8564544483957558, -0.5772585738467768,
    0.7202612672781041, 0.7307797030308907, -0.7583698246835111, -0.7869426057675021,
    0.7959131589272986, 0.8265272800629793, -0.8571428851683863, -0.8571428393645633,
    0.007149950940208943, -2.8236600908745726e-06, -0.006773265234381003,
    -1.4623212301073427e-07, 0.008869215307677137, 5.999868831947352e-06,
    -0.011729358301387537, -4.249561665451796e-05, 0.016421738814645315,
    0.00029749498580051704, -0.024989587552392552, -0.0020824656376448895, 0.04373177842638611,
    0.014577259475204975, -0.1020408163265289, -0.10204081632653056,};
__device__ __forceinline__ ctab weak_table(int at) {
  ctab t = to_ctab(weak_coef) + at;
  asm volatile("" : "+s"(t));
  return t;
}
// the polynomial of degree DEG with constant term c0 at x (x > 0: the shock's)
template <int DEG>
__device__ __forceinline__ double weak_poly(ctab t, double x, double c0) {
  double r = t[0], s = t[1];
#pragma unroll
  for (int n = 1; n < DEG; ++n) {
    r = fma(r, x, t[2 * n]);
    s = fma(s, x, t[2 * n + 1]);
  }
  return fma(x > 0.0 ? s : r, x, c0);
}

// the same with its derivative
template <int DEG>
__device__ __forceinline__ double weak_poly_d(ctab t, double x, double c0, double& dx) {
  double r = t[0], s = t[1], dr = r, ds = s;
#pragma unroll
  for (int n = 1; n < DEG; ++n) {
    r = fma(r, x, t[2 * n]);
    s = fma(s, x, t[2 * n + 1]);
    dr = fma(dr, x, r);
    ds = fma(ds, x, s);
  }
  dx = x > 0.0 ? ds : dr;
  return fma(x > 0.0 ? s : r, x, c0);
}

// The Newton iteration of the short form for the star pressure from the guess ps, where going:
// the pressure functions f and slopes d (times rho c) of both sides at the last but one
// iterate, the last step dp, the largest |x| met; conv: converged with |x| within 1/16.
struct WeakStar {
  double ps, fL, fR, dL, dR, dp, xm;
  int it;
  bool conv;
};
__device__ __forceinline__ WeakStar weak_star(const GasC& c, double pL, double pR, double ipL,
                                              double ipR, double gL, double gR, double zL,
                                              double zR, double du, double ps, bool going) {
  // (the caller computes on from here in every lane, and drops what did not converge)
  WeakStar w = {ps, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0, false};
  double xm = 0.0;
  bool conv = false;
  while (going && w.it < c.max_iter) {
    ++w.it;
    const double xL = (ps - pL) * ipL, xR = (ps - pR) * ipR;
    xm = fmax(xm, fmax(fabs(xL), fabs(xR)));
    if (xm <= 1.0 / 512.0) {
      const ctab t = weak_table(WK_G);
      w.fL = gL * xL * weak_poly<4>(t, xL, 1.0);
      w.fR = gR * xR * weak_poly<4>(t, xR, 1.0);
      w.dL = zL * fma(fma(t[WK_D], xL, t[WK_D + 1]), xL, 1.0);
      w.dR = zR * fma(fma(t[WK_D], xR, t[WK_D + 1]), xR, 1.0);
    } else {
      const ctab t = weak_table(WKW_G);
      w.fL = gL * xL * weak_poly<8>(t, xL, 1.0);
      w.fR = gR * xR * weak_poly<8>(t, xR, 1.0);
      const ctab d = weak_table(WKW_D);
      w.dL = zL * weak_poly<5>(d, xL, 1.0);
      w.dR = zR * weak_poly<5>(d, xR, 1.0);
    }
    const double pn = ps - (w.fL + w.fR + du) * frcp(w.dL + w.dR);
    w.dp = pn - ps;
    // relative change 2|dp|/(p_new + p_old) <= 1e-12, written without a division
    conv = 2.0 * fabs(w.dp) <= 1e-12 * (pn + ps);
    ps = pn;
    going = !conv && xm <= 0.0625;
  }
  w.ps = ps;
  w.xm = xm;
  w.conv = conv && xm <= 0.0625;
  return w;
}

template <int DIR>
__device__ __forceinline__ bool gas_face64(const GasC& c, const double* qL, const double* qR,
                                           double* F, int& last) {
  constexpr int N = Dirs<DIR>::n, T1 = Dirs<DIR>::t1, T2 = Dirs<DIR>::t2;
  const double rL = qL[4], rR = qR[4], pL = qL[3], pR = qR[3], uL = qL[N], uR = qR[N];
  bool ok = rL > 0.0 && pL > 0.0 && rR > 0.0 && pR > 0.0;
  const double irL = frcp(rL), irR = frcp(rR);
  const double c2L = c.g * pL * irL, c2R = c.g * pR * irR;
  const double du = uR - uL;
  double rho = rL, un = uL, p = pL, t1 = qL[T1], t2 = qL[T2];
  last = 0;
  // gas_riemann's test of a face supersonic to the right
  bool sup = uL > 0.0 && uL * uL >= c2L;
  if (!wave_none(sup)) {
    const double u2 = uL * uL;
    const double phi = (rL * u2 * c.inv_g - c.gm1_2g * pL) * c.inv_gp1_2g;
    const double d = phi - pL, d2A = d * d * (c.a2 * irL), pb = phi + c.kshock * pL;
    sup = sup && (du <= 0.0 || du * du < c.g2m1 * c.g2m1 * c2L) && phi >= pR &&
          (du >= 0.0 || d2A >= du * du * pb) && u2 * pb >= d2A;
  }
  if (!wave_none(ok && !sup)) {
    bool weak = uL * uL < 0.81 * c2L && uR * uR < 0.81 * c2R;
    const double rsL = frsq(c2L), rsR = frsq(c2R);
    const double cL = c2L * rsL, cR = c2R * rsR, zL = irL * rsL, zR = irR * rsR;
    const double ipL = frcp(pL), ipR = frcp(pR);
    const double gL = (5.0 / 7.0) * cL, gR = (5.0 / 7.0) * cR;
    double ps = 0.5 * (pL + pR) - 0.125 * du * (rL + rR) * (cL + cR);
    const WeakStar w = weak_star(c, pL, pR, ipL, ipR, gL, gR, zL, zR, du, ps, weak && ok && !sup);
    ps = w.ps;
    weak = weak && w.conv;
    // star velocity at the converged p* (as gas_riemann)
    const double us = 0.5 * (uL + uR) + 0.5 * ((w.fR + w.dR * w.dp) - (w.fL + w.dL * w.dp));
    weak = weak && us * us < 0.81 * fmin(c2L, c2R);
    const bool left = us >= 0.0;
    const double pK = left ? pL : pR, ipK = left ? ipL : ipR, rK = left ? rL : rR;
    const double x = (ps - pK) * ipK;
    double R;
    if (w.xm <= 1.0 / 512.0) R = weak_poly<4>(weak_table(WK_R), x, 5.0 / 7.0);
    else R = weak_poly<8>(weak_table(WKW_R), x, 5.0 / 7.0);
    const double rs = fma(rK * x, R, rK);
    if (!sup) {
      ok = ok && weak;
      last = w.it;
      rho = rs; un = us; p = ps;
      t1 = left ? qL[T1] : qR[T1];
      t2 = left ? qL[T2] : qR[T2];
    }
  }
  const double en = p * c.inv_gm1 + 0.5 * rho * (un * un + t1 * t1 + t2 * t2);
  const double m = rho * un;
  F[4] = m;
  F[N] = m * un + p;
  F[T1] = m * t1;
  F[T2] = m * t2;
  F[3] = (en + p) * un;
  return ok;
}

// Dust face: velocity and density reconstructed whole (no stationary reference); a face
// density below zero falls back to the cell-centre state.  Where both states of a face hold
// dust and both streams cross it the same way, the flux is the upwind state's; a wavefront of
// such faces (nearly every one: the others hold an emptied cell, a midplane or a turning
// point) takes that flux behind one scalar test instead of the fallback and the rules of
// dust_riemann, and without selects if all its lanes stream one way.
// cell(c, f): field f of the stencil cell c = 0 .. 3 (A, B | C, D), read again where the
// fallback needs it (held across the solve the cells would cost 16 registers).
template <int DIR, class Cell, class Co>
__device__ __forceinline__ void dust_face(const RecC& rc, Cell cell, Co coB, Co coC, double F[4],
                                          TStat& st) {
  double qL[4], qR[4];
#pragma unroll
  for (int f = 0; f < 4; ++f)
    face_pair<DIR>(rc, cell(0, f), cell(1, f), cell(2, f), cell(3, f), coB, coC, qL[f], qR[f]);
  constexpr int N = Dirs<DIR>::n, T1 = Dirs<DIR>::t1, T2 = Dirs<DIR>::t2;
  double fl[4];
  const double uL = qL[N], uR = qR[N];
  const bool toL = uL > 0.0 && uR >= 0.0, toR = uL <= 0.0 && uR < 0.0;
  if (wave_none(!(qL[3] > 0.0 && qR[3] > 0.0 && (toL || toR)))) {
    if (wave_none(toR)) {
      const double m = qL[3] * uL;
      fl[0] = m; fl[1] = m * uL; fl[2] = m * qL[T1]; fl[3] = m * qL[T2];
    } else {
      const double u = toL ? uL : uR;
      const double m = (toL ? qL[3] : qR[3]) * u;
      fl[0] = m; fl[1] = m * u;
      fl[2] = m * (toL ? qL[T1] : qR[T1]);
      fl[3] = m * (toL ? qL[T2] : qR[T2]);
    }
  } else {
    if (qL[3] < 0.0) {
#pragma unroll
      for (int f = 0; f < 4; ++f) qL[f] = cell(1, f);
      st.fall++;
    }
    if (qR[3] < 0.0) {
#pragma unroll
      for (int f = 0; f < 4; ++f) qR[f] = cell(2, f);
      st.fall++;
    }
    dust_riemann(qL[3], qL[N], qL[T1], qL[T2], qR[3], qR[N], qR[T1], qR[T2], fl);
  }
  F[3] = fl[0];
  F[N] = fl[1];
  F[T1] = fl[2];
  F[T2] = fl[3];
}

}  // namespace rb

#include "rb_pert32.h"

namespace rb {

// Reconstructed FP32 face states (W' of the gas, field slots) between cells B and C;
// cell(c, f) as dust_face's.
template <int DIR, class Cell>
__device__ __forceinline__ void recon32(Cell cell, const float* coB, const float* coC, float qL[5],
                                        float qR[5]) {
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    const float A = cell(0, f), B = cell(1, f), C = cell(2, f), D = cell(3, f);
    if constexpr (DIR == 0) {
      qL[f] = B + inc_up_c(A, B, C, coB);
      qR[f] = C + inc_lo_c(B, C, D, coC);
    } else {
      qL[f] = B + inc_up_u(A, B, C);
      qR[f] = C + inc_lo_u(B, C, D);
    }
  }
}

// A face of the FP32-perturbation form that the short form (gas_face32) does not take: the
// W' of its stencil cells A, B | C, D (field slots).
struct Face32 {
  float A[5], B[5], C[5], D[5];
};
struct Face32Out {
  float F[5];                        // flux change, field slots
  int last, maxit;                   // Newton iterations of the solve kept; the most of any
  unsigned fall, vac, resolve, noconv;
};
// counts of a workgroup's faces that the general form solved
struct GasCount {
  unsigned fall, vac, resolve;
  int noconv;
};

// ------------------------------------------------------------------------------------
// addressing of a wavefront's row

// Element at a lane's index from a pointer that is the same in the whole wavefront.  The
// pointer passes through a scalar register the optimiser cannot see through: otherwise it
// keeps one vector address per array across the march (about 30 registers).  It stays a
// pointer to global memory on the way: through a generic one each load would also count as an
// LDS access, and every wait for an LDS read would wait for the loads from memory with it.
template <class T>
using Global = __attribute__((address_space(1))) T;
template <class T>
__device__ __forceinline__ Global<T>& at_row(T* p, unsigned lane) {
  Global<T>* q = (Global<T>*)(uintptr_t)p;
  asm("" : "+s"(q));
  return *(Global<T>*)((uintptr_t)q + (size_t)(lane * (unsigned)sizeof(T)));
}
template <class T>
__device__ __forceinline__ Global<T>& at_plane(T* p, size_t off) {
  Global<T>* q = (Global<T>*)(uintptr_t)p;
  asm("" : "+s"(q));
  return q[off];
}

// ------------------------------------------------------------------------------------
// state access with ghost cells (Sect. 2.4): r and z ghosts come from tables, theta wraps

// FP32-perturbation storage layout: the gas deviation E' (5 fields) and each dust
// species' velocity as a deviation from the stationary flow's velocity at the cell centre
// (3 per species; that velocity is azimuthal, App. A, so only the theta component
// differs) in FP32, then the dust densities in FP64 (mass is accumulated in FP64).
// f64_base: first double of that part.  A dust momentum is read as density x (stationary
// velocity + stored deviation); it is stored as momentum / density - stationary velocity
// after the cell's new density, which must therefore be written first (zero deviation
// where the density is below 1e-300; the velocity of a cell without dust reads as zero).
__device__ __forceinline__ size_t p32_f64_base(const Geo& g) {
  return (((size_t)(5 + 3 * g.nd) * g.N + 63) / 64 * 64) / 2;
}

// interior conservative value of field f (FP64 storage: the gas deviation E' and the dust
// variables; or the FP32-perturbation layout above)
template <bool P32>
__device__ __forceinline__ double ld_cell(const StageArgs& a, const void* st, int f, int k, int i,
                                          size_t cell) {
  const Geo& g = a.g;
  if (P32) {
    if (f < 5) return (double)((const float*)st)[(size_t)f * g.N + cell];
    const int sp = (f - 5) >> 2, c = (f - 5) & 3;
    const double rd = ((const double*)st)[p32_f64_base(g) + (size_t)sp * g.N + cell];
    if (c == 3) return rd;
    const double u0 = c == 1 ? a.t.wc[((size_t)k * g.nr + i) * WB_N + WB_V] : 0.0;
    return rd * (u0 + (double)((const float*)st)[(size_t)(5 + 3 * sp + c) * g.N + cell]);
  }
  return ((const double*)st)[(size_t)f * g.N + cell];
}

template <bool P32>
__device__ __forceinline__ void st_cell(const StageArgs& a, void* st, int f, int k, int i,
                                        size_t cell, double v) {
  const Geo& g = a.g;
  if (P32) {
    if (f < 5) { ((float*)st)[(size_t)f * g.N + cell] = (float)v; return; }
    const int sp = (f - 5) >> 2, c = (f - 5) & 3;
    double* dens = (double*)st + p32_f64_base(g) + (size_t)sp * g.N + cell;
    if (c == 3) { *dens = v; return; }
    const double rd = *dens;  // the new density, written before the momenta
    const double u0 = c == 1 ? a.t.wc[((size_t)k * g.nr + i) * WB_N + WB_V] : 0.0;
    ((float*)st)[(size_t)(5 + 3 * sp + c) * g.N + cell] = rd > 1e-300 ? (float)(v * frcp(rd) - u0) : 0.0f;
  } else {
    ((double*)st)[(size_t)f * g.N + cell] = v;
  }
}

// Gas deviation W' = W(E0 + E') - W(E0) of a cell from its conservative deviation e and
// its stationary flow b (WB_N entry), free of cancellation: rho' = e_rho,
// u' = (m' - u0 rho') / rho, P' = (g - 1)(E' - dKE) with the kinetic-energy change
// dKE = rho' |u0|^2 / 2 + rho u0.u' + rho |u'|^2 / 2.  Exactly zero for e = 0; for the Sod
// annulus (b = 0) it is the state's own primitives.
__device__ __forceinline__ void cell_w(const double* e, const double* b, double gm1, double* w) {
  const double rp = e[4];
  const double rho = b[WB_RHO] + rp;
  const double ir = frcp(rho);
  const double u0 = b[WB_U], v0 = b[WB_V], w0 = b[WB_W];
  const double up = (e[0] - u0 * rp) * ir, vp = (e[1] - v0 * rp) * ir, wp = (e[2] - w0 * rp) * ir;
  const double dke = 0.5 * rp * (u0 * u0 + v0 * v0 + w0 * w0) + rho * (u0 * up + v0 * vp + w0 * wp) +
                     0.5 * rho * (up * up + vp * vp + wp * wp);
  w[0] = up; w[1] = vp; w[2] = wp;
  w[3] = gm1 * (e[3] - dke);
  w[4] = rp;
}
__device__ __forceinline__ void cell_w(const float* e, const double* b, float gm1, float* w) {
  const float rp = e[4];
  const float rho = (float)(b[WB_RHO] + (double)rp);
  const float ir = rcp32(rho);
  const float u0 = (float)b[WB_U], v0 = (float)b[WB_V], w0 = (float)b[WB_W];
  const float u0sq = (float)(b[WB_U] * b[WB_U] + b[WB_V] * b[WB_V] + b[WB_W] * b[WB_W]);
  const float up = (e[0] - u0 * rp) * ir, vp = (e[1] - v0 * rp) * ir, wp = (e[2] - w0 * rp) * ir;
  const float dke = 0.5f * rp * u0sq + rho * (u0 * up + v0 * vp + w0 * wp) +
                    0.5f * rho * (up * up + vp * vp + wp * wp);
  w[0] = up; w[1] = vp; w[2] = wp;
  w[3] = gm1 * (e[3] - dke);
  w[4] = rp;
}

// The same in FP32 about a flow along theta only: the second form's own roundings without its
// products with zero velocities.
__device__ __forceinline__ void cell_w32(const float* e, const PertCell& c, float gm1, float* w) {
  const float rp = e[4];
  const float rho = (float)(c.rho + (double)rp);
  const float ir = rcp32(rho);
  const float up = e[0] * ir, vp = (e[1] - c.v * rp) * ir, wp = e[2] * ir;
  const float dke = 0.5f * rp * c.vsq + rho * (c.v * vp) +
                    0.5f * rho * (up * up + vp * vp + wp * wp);
  w[0] = up; w[1] = vp; w[2] = wp;
  w[3] = gm1 * (e[3] - dke);
  w[4] = rp;
}

// Reconstructed variables of a group at any cell, interior or ghost, for FP64 storage and
// stationary ghosts (what the adjoint takes): the gas W', or the dust velocity (zero where the
// density is not positive) and density.  Each kind of ghost is read through a pointer of its
// own: with one pointer picked from the two tables, ROCm 7.2's compiler merged the tails and
// read the upper z ghosts of k_adj_z<gas> through the r table's base.
template <int NG>
__device__ __forceinline__ void load_recon(const StageArgs& a, const void* st, int F0, int k,
                                           int i, int j, double* out) {
  const Geo& g = a.g;
  if (k < 0 || k >= g.nz) {
    const int ii = min(max(i, 0), g.nr - 1);
    const int side = k < 0 ? 0 : 1;
    const int layer = min(k < 0 ? -1 - k : k - g.nz, 1);
    const double* gt = a.t.ghz + ((size_t)(side * 2 + layer) * g.nr + ii) * g.nf + F0;
#pragma unroll
    for (int f = 0; f < NG; ++f) out[f] = gt[f];
    return;
  } else if (i < 0 || i >= g.nr) {
    const int side = i < 0 ? 0 : 1;
    const int layer = min(i < 0 ? -1 - i : i - g.nr, 1);
    const double* gt = a.t.ghr + ((size_t)(side * 2 + layer) * g.nz + k) * g.nf + F0;
#pragma unroll
    for (int f = 0; f < NG; ++f) out[f] = gt[f];
    return;
  }
  const double* d = (const double*)st + (size_t)F0 * g.N + ((size_t)k * g.nr + i) * g.nth + j;
  if constexpr (NG == 5) {
    double e[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) e[f] = d[(size_t)f * g.N];
    cell_w(e, a.t.wc + ((size_t)k * g.nr + i) * WB_N, g.gamma - 1.0, out);
  } else {
    const double rd = d[3 * g.N];
    const double id = rd > 0.0 ? 1.0 / rd : 0.0;
    out[0] = d[0] * id;
    out[1] = d[g.N] * id;
    out[2] = d[2 * g.N] * id;
    out[3] = rd;
  }
}

// A dust cell's in two steps: dust_fetch issues the loads and does no arithmetic on what they
// return, dust_finish forms the variables (the same values as load_recon).  A wavefront waits
// for a load where its result is first used, so a fetch made a phase or a plane ahead of its
// finish keeps that wait off the critical path.  Ghost cells carry their table values in d.
struct DustRaw {
  double d[4];
  bool ghost;
};
__device__ __forceinline__ void dust_fetch(const StageArgs& a, const void* st, int F0, int k, int i,
                                           int j, DustRaw& R) {
  // the same loads on every path, from addresses chosen by selects (loads on separate
  // branches land in separate registers, and the copy that merges them waits for them)
  const Geo& g = a.g;
  const double* gt = nullptr;  // the ghost table row, if the cell is a ghost
  int kc = k;
  if (k < 0 || k >= g.nz) {
    const int ii = min(max(i, 0), g.nr - 1);
    const int side = k < 0 ? 0 : 1;
    const int layer = min(k < 0 ? -1 - k : k - g.nz, 1);
    gt = a.t.ghz + ((size_t)(side * 2 + layer) * g.nr + ii) * g.nf + F0;
    kc = k < 0 ? 0 : g.nz - 1;
  } else if (i < 0 || i >= g.nr) {
    const int side = i < 0 ? 0 : 1;
    const int layer = min(i < 0 ? -1 - i : i - g.nr, 1);
    gt = a.t.ghr + ((size_t)(side * 2 + layer) * g.nz + k) * g.nf + F0;
  }
  const int ic = min(max(i, 0), g.nr - 1);  // a valid cell for the loads a ghost ignores
  const bool gh = gt != nullptr;
  R.ghost = gh;
  const double* d = (const double*)st + (size_t)F0 * g.N + ((size_t)kc * g.nr + ic) * g.nth + j;
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const double* p = gh ? gt + f : d + (size_t)f * g.N;
    R.d[f] = *p;
  }
}
__device__ __forceinline__ void dust_finish(const DustRaw& R, double* out) {
  const double rd = R.d[3];
  const double id = rd > 0.0 ? 1.0 / rd : 0.0;
#pragma unroll
  for (int f = 0; f < 3; ++f) out[f] = R.ghost ? R.d[f] : R.d[f] * id;
  out[3] = rd;
}

// stationary-flow primitives (WB_N entry) of an interior cell or of the ghost next to the
// boundary (the face-state fallback's cell-centre state is this plus the cell's W')
__device__ __forceinline__ const double* bg_ptr(const StageArgs& a, int k, int i) {
  const Geo& g = a.g;
  if (k < 0 || k >= g.nz) {
    const int ii = min(max(i, 0), g.nr - 1);
    return a.t.ghzw + ((size_t)(k < 0 ? 0 : 2) * g.nr + ii) * WB_N;
  }
  if (i < 0 || i >= g.nr) return a.t.ghrw + ((size_t)(i < 0 ? 0 : 2) * g.nz + k) * WB_N;
  return a.t.wc + ((size_t)k * g.nr + i) * WB_N;
}

__device__ __forceinline__ const double* rco_ptr(const StageArgs& a, int i) {
  int c = min(max(i, -1), a.g.nr);
  return a.t.rco + (size_t)(c + 1) * RC_N;
}

// Any gas face in FP64: reconstructed states, positivity fallback to the cell-centre state
// W0(cell) + W'(cell), exact Riemann problem, F* in field order.  Direction dir, stencil
// cells as dust_face's, the lower one (k, i) (below row 0: i = -1).
template <bool G75, class Cell>
__device__ __forceinline__ void gas_face64_general(const StageArgs& a, const GasC& c,
                                                   const RecC& rc, int dir, int k, int i, Cell cell,
                                                   double* F, TStat& st) {
  const double* bB = bg_ptr(a, k, i);
  const double* bC = dir == 1 ? bB : (dir == 0 ? bg_ptr(a, k, i + 1) : bg_ptr(a, k + 1, i));
  const double* bf = dir == 1 ? bB
      : (dir == 0 ? a.t.wr + ((size_t)k * (a.g.nr + 1) + min(i + 1, a.g.nr)) * WB_N
                  : a.t.wz + ((size_t)(k + 1) * a.g.nr + i) * WB_N);
  double qL[5], qR[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    if (dir == 0)
      face_pair<0>(rc, cell(0, f), cell(1, f), cell(2, f), cell(3, f), rco_ptr(a, i),
                   rco_ptr(a, i + 1), qL[f], qR[f]);
    else
      face_pair<1>(rc, cell(0, f), cell(1, f), cell(2, f), cell(3, f), nullptr, nullptr, qL[f], qR[f]);
    qL[f] = bf[f] + qL[f];
    qR[f] = bf[f] + qR[f];
  }
  if (!(qL[4] > 0.0 && qL[3] > 0.0)) {
#pragma unroll
    for (int f = 0; f < 5; ++f) qL[f] = bB[f] + cell(1, f);
    st.fall++;
  }
  if (!(qR[4] > 0.0 && qR[3] > 0.0)) {
#pragma unroll
    for (int f = 0; f < 5; ++f) qR[f] = bC[f] + cell(2, f);
    st.fall++;
  }
  // (selects, not indexes: a direction in an index would put the states in memory)
  auto un = [&](const double* q) { return dir == 0 ? q[0] : dir == 1 ? q[1] : q[2]; };
  auto t1 = [&](const double* q) { return dir == 0 ? q[1] : q[0]; };
  auto t2 = [&](const double* q) { return dir == 2 ? q[1] : q[2]; };
  double fl[5];
  gas_riemann<G75>(c, qL[4], frcp(qL[4]), un(qL), t1(qL), t2(qL), qL[3], qR[4], frcp(qR[4]), un(qR),
                   t1(qR), t2(qR), qR[3], fl, st);
  F[4] = fl[0];
  F[0] = dir == 0 ? fl[1] : fl[2];
  F[1] = dir == 1 ? fl[1] : (dir == 0 ? fl[2] : fl[3]);
  F[2] = dir == 2 ? fl[1] : fl[3];
  F[3] = fl[4];
}

// The perturbation Riemann problem at the face in direction dir above cell (k, i) (below row
// 0: i = -1); faces it cannot take (strong perturbation, transonic fan, no convergence,
// non-positive face state) are re-solved in FP64 on the full states.
__device__ __forceinline__ Face32Out gas_face32_general(const StageArgs& a, int dir, int k, int i,
                                                        const Face32& q) {
  const GasC c = gas_consts(1.4, a.g.newton_max);
  // (selects, as in gas_face64_general)
  auto un = [&](const auto* v) { return dir == 0 ? v[0] : dir == 1 ? v[1] : v[2]; };
  auto t1 = [&](const auto* v) { return dir == 0 ? v[1] : v[0]; };
  auto t2 = [&](const auto* v) { return dir == 2 ? v[1] : v[2]; };
  const double* bB = bg_ptr(a, k, i);
  const double* bC = dir == 1 ? bB : (dir == 0 ? bg_ptr(a, k, i + 1) : bg_ptr(a, k + 1, i));
  const double* bf = dir == 1 ? bB
      : (dir == 0 ? a.t.wr + ((size_t)k * (a.g.nr + 1) + min(i + 1, a.g.nr)) * WB_N
                  : a.t.wz + ((size_t)(k + 1) * a.g.nr + i) * WB_N);
  float qL[5], qR[5];
  auto cell = [&](int s, int f) { return s == 0 ? q.A[f] : s == 1 ? q.B[f] : s == 2 ? q.C[f] : q.D[f]; };
  // (the weights in FP32, as the short form takes them)
  auto co = [&](int row) { return a.t.rcf + (size_t)(min(max(row, -1), a.g.nr) + 1) * RC_N; };
  if (dir == 0) recon32<0>(cell, co(i), co(i + 1), qL, qR);
  else recon32<1>(cell, (const float*)nullptr, (const float*)nullptr, qL, qR);
  TStat st = {0, 0, 0, 0, 0, 0, 0};
  const BgW b = {bf[WB_RHO], un(bf), t1(bf), t2(bf), bf[WB_P], bf[WB_C], bf[WB_H]};
  const PW L = {qL[4], un(qL), t1(qL), t2(qL), qL[3]};
  const PW R = {qR[4], un(qR), t1(qR), t2(qR), qR[3]};
  const bool okL = (b.rho + (double)L.rho > 0.0) && (b.p + (double)L.p > 0.0);
  const bool okR = (b.rho + (double)R.rho > 0.0) && (b.p + (double)R.p > 0.0);
  PW W;
  float fl[5];
  if (okL && okR && riemann_pert(b, L, R, c, W, st)) {
    flux_pert(b, W, (float)c.inv_gm1, fl);
  } else {
    st.resolve++;
    double xL[5], xR[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      xL[f] = okL ? bf[f] + (double)qL[f] : bB[f] + (double)q.B[f];
      xR[f] = okR ? bf[f] + (double)qR[f] : bC[f] + (double)q.C[f];
    }
    if (!okL) st.fall++;
    if (!okR) st.fall++;
    double f64[5];
    gas_riemann<true>(c, xL[4], frcp(xL[4]), un(xL), t1(xL), t2(xL), xL[3], xR[4], frcp(xR[4]),
                      un(xR), t1(xR), t2(xR), xR[3], f64, st);
    const double m0 = b.rho * b.un;
    fl[0] = (float)(f64[0] - m0);
    fl[1] = (float)(f64[1] - (m0 * b.un + b.p));
    fl[2] = (float)(f64[2] - m0 * b.t1);
    fl[3] = (float)(f64[3] - m0 * b.t2);
    fl[4] = (float)(f64[4] - b.h * b.un);
  }
  Face32Out o;
  o.F[4] = fl[0];
  o.F[0] = dir == 0 ? fl[1] : fl[2];
  o.F[1] = dir == 1 ? fl[1] : (dir == 0 ? fl[2] : fl[3]);
  o.F[2] = dir == 2 ? fl[1] : fl[3];
  o.F[3] = fl[4];
  o.last = st.last;
  o.maxit = st.maxit;
  o.fall = st.fall; o.vac = st.vac; o.resolve = st.resolve; o.noconv = st.noconv;
  return o;
}

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ int wave_isum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ int wave_imax(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

// Inverse dust stopping time of species s in a cell whose gas has density rho and
// pressure p (Sect. 2.9).  Law 0: Omega_K / St.  Law 1: Epstein 1/t = rho c_s / (rho_s r_p)
// with the isothermal c_s = sqrt(p / rho), i.e. sqrt(p rho) / (rho_s r_p); in the Stokes
// regime (r_p > 9 lambda / 4, lambda = mfp / rho) the Epstein rate times 9 lambda / (4 r_p).
template <bool EXT = true>
__device__ __forceinline__ double inv_tstop(const Geo& g, int s, double omk, double rho, double p) {
  if (!EXT || g.drag_law == 0) return omk * g.inv_st[s];
  const double ie = sqrt(p * rho) * g.inv_mp[s];
  const double x = g.rp94[s] * rho;
  return x <= g.mfp ? ie : ie * g.mfp / x;
}

// XCD-aware tile order: workgroup b is dispatched to XCD b % 8; give every XCD a
// contiguous range of tiles so that halo re-reads hit its own L2.
__device__ __forceinline__ int xcd_tile(int b, int nblk) {
  int q = nblk >> 3, rem = nblk & 7, x = b & 7;
  return x * q + min(x, rem) + (b >> 3);
}

}  // namespace rb
