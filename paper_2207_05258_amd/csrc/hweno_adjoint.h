// Hand-written reverse-mode derivatives (vector-Jacobian products) of the
// device math in hweno_math.h: the discrete adjoint of the semi-discrete
// operator (eqs. odeH / ode2H with the reconstruction of Section 2.1) and of
// the limiter (Section 2.2), with the Lax-Friedrichs speeds held fixed.
//
// Conventions: every *_vjp function recomputes the forward quantities it needs
// from the same inputs; it adds to the input adjoints or overwrites them, as its
// comment says.
// |x| is differentiated as sign(x) with sign(0) = 0.
#pragma once

#include "hweno_math.h"

namespace hweno {

template <typename T>
HW_HD T sgn(T x) {
  return T((x > T(0)) - (x < T(0)));
}

// reverse of the combination blend_c(): with R0, R1, R2 its candidates and r = num / den its value, the adjoints gR_l and gc_l (overwritten) for the
// adjoint g of r; returns r.  In the form of one reciprocal per indicator (e_l = 1
// + k_l) in both precisions: k_l = kappa t^2 / c_l, s_l = g_l (k_l - k_0),
//   r = ((1 + k0) R0 + s1 R1 + s2 R2) / (1 + k0 + s1 + s2).
// g1, g2: linear weights; |x| is differentiated as sign(x).
template <int KAP48, typename T>
HW_HD T blend_vjp(T R0, T R1, T R2, T c0, T c1, T c2, T g1, T g2, T g, T& gR0, T& gR1, T& gR2,
                  T& gc0, T& gc1, T& gc2) {
  const T d01 = c0 - c1, d02 = c0 - c2;
  const T st = T(sqrt_kappa<KAP48>()) * (fabs(d01) + fabs(d02));
  const T tau = st * st;
  const T i0 = fast_rcp(c0), i1 = fast_rcp(c1), i2 = fast_rcp(c2);
  const T k0 = tau * i0, k1 = tau * i1, k2 = tau * i2;
  const T m = T(1) + k0, s1 = g1 * (k1 - k0), s2 = g2 * (k2 - k0);
  const T iden = fast_rcp((m + s1) + s2);
  const T r = mad(m, R0, mad(s1, R1, s2 * R2)) * iden;
  const T gi = g * iden;
  gR0 = gi * m;
  gR1 = gi * s1;
  gR2 = gi * s2;
  const T p1 = gi * g1 * (R1 - r), p2 = gi * g2 * (R2 - r);  // adjoints of k1, k2
  const T p0 = mad(gi, R0 - r, -(p1 + p2));                   // and of k0
  // d tau / d t = 2 sqrt(kappa) st
  const T gt = T(2.0 * sqrt_kappa<KAP48>()) * st * mad(p0, i0, mad(p1, i1, p2 * i2));
  const T gs1 = gt * sgn(d01), gs2 = gt * sgn(d02);
  gc0 = mad(-p0 * k0, i0, gs1 + gs2);
  gc1 = mad(-p1 * k1, i1, -gs1);
  gc2 = mad(-p2 * k2, i2, -gs2);
  return r;
}

// reverse of hw_blend(): adjoints of its five arguments (overwritten) for the
// adjoint g of its value, which is returned; g1, g2, eps as in hw_blend's weights
// but g1, g2 without kappa
template <typename T>
HW_HD T hw_blend_vjp(T A, T B, T H0, T Hs, T Hd, T g1, T g2, T eps, T g, T& gA, T& gB, T& gH0,
                     T& gHs, T& gHd) {
  constexpr T a1 = T(6.067488135033763), a2 = T(3.012679250059034);
  constexpr T b1 = T(15.029579351881592), b2 = T(45.165651404159786);
  constexpr T q1 = T(0.24822509386187025), q2 = T(2.2469689522048239);
  const T u1 = H0 + A, u2 = H0 - B;
  const T lap = u1 - u2, t = u1 + u2;
  const T R0 = mad(T(1.1), lap, T(0.3) * Hd);
  const T y = mad(a1, lap, a2 * Hd);
  const T z = mad(b1, mad(T(-2), H0, Hs), b2 * t);
  const T h = mad(T(3.0 / 13.0) * H0, H0, eps);
  const T c0 = mad(q1 * lap, lap, mad(q2 * t, t, mad(z, z, mad(y, y, h))));
  T gR0, gu1, gv2, gc0, gc1, gc2;
  const T r = blend_vjp<13>(R0, u1, -u2, c0, mad(u1, u1, h), mad(u2, u2, h), g1, g2, g, gR0, gu1,
                            gv2, gc0, gc1, gc2);
  const T w = T(2) * gc0;
  const T gy = w * y, gz = w * z;
  const T glap = mad(a1, gy, mad(T(1.1), gR0, q1 * w * lap));
  const T gt = mad(b2, gz, q2 * w * t);
  gu1 = mad(T(2) * gc1, u1, gu1) + (gt + glap);
  const T gu2 = mad(T(2) * gc2, u2, -gv2) + (gt - glap);
  gA = gu1;
  gB = -gu2;
  gHs = b1 * gz;
  gHd = mad(a2, gy, T(0.3) * gR0);
  gH0 = mad(T(6.0 / 13.0) * H0, gc0 + gc1 + gc2, mad(T(-2.0) * b1, gz, gu1 + gu2));
  return r;
}

// reverse of hw_plus() (accumulates; for checks, as it is); returns the forward value
template <typename T>
HW_HD T hw_plus_vjp(T fm, T f0, T fp, T Hm, T H0, T Hp, const Weights<T>& w, T g, T& gfm,
                    T& gf0, T& gfp, T& gHm, T& gH0, T& gHp) {
  T gA, gB, gh0, gHs, gHd;
  const T r = hw_blend_vjp(T(2) * (fm - f0), T(2) * (fp - f0), T(2) * H0, T(2) * (Hm + Hp),
                           T(2) * (Hm - Hp), w.g1, w.g2, T(12.0 / 13.0) * w.eps, g * T(1.0 / 6.0),
                           gA, gB, gh0, gHs, gHd);
  gfm += gA;
  gfp += gB;
  gf0 += g - (gA + gB);
  gH0 += mad(T(0.5), g, gh0);
  gHm += gHs + gHd;
  gHp += gHs - gHd;
  return mad(T(1.0 / 12.0), r, mad(T(0.5), H0, f0));
}

// reverse of limit_blend(): adjoints of d1, d2, Vs, Vd (overwritten) for the adjoint
// g of its value, which is returned; g1, g2: the limiter's linear weights
template <typename T>
HW_HD T limit_blend_vjp(T d1, T d2, T Vs, T Vd, T g1, T g2, T eps, T g, T& gd1, T& gd2, T& gVs,
                        T& gVd) {
  constexpr T a1 = T(12.554318802466193), a2 = T(6.254843361443233);
  constexpr T q1 = T(1.0813413108057222), q2 = T(2.440625);
  const T D = d1 + d2, lap = d2 - d1, e = Vs - D;
  const T x0 = mad(T(0.5), D, T(-3.0 / 16.0) * e);
  const T y = mad(a1, lap, a2 * Vd);
  const T c0 = mad(q1 * lap, lap, mad(q2 * e, e, mad(y, y, mad(x0, x0, eps))));
  T gP0, gP1, gP2, gc0, gc1, gc2;
  const T r = blend_vjp<12>(mad(T(0.75), D, T(-0.25) * Vs), d1, d2, c0, mad(d1, d1, eps),
                            mad(d2, d2, eps), g1, g2, g, gP0, gP1, gP2, gc0, gc1, gc2);
  const T w = T(2) * gc0;
  const T gy = w * y, gx0 = w * x0;
  const T ge = mad(T(-3.0 / 16.0), gx0, q2 * w * e);
  const T glap = mad(a1, gy, q1 * w * lap);
  const T gD = mad(T(0.75), gP0, mad(T(0.5), gx0, -ge));
  gd1 = mad(T(2) * gc1, d1, gP1) + (gD - glap);
  gd2 = mad(T(2) * gc2, d2, gP2) + (gD + glap);
  gVs = mad(T(-0.25), gP0, ge);
  gVd = a2 * gy;
  return r;
}

// reverse of limit1() (accumulates): limit_blend_vjp around the scheme's own arguments,
// for checks
template <typename T>
HW_HD void limit1_vjp(T um, T u0, T up, T vm, T vp, T h, T ih, const Weights<T>& w, T g,
                      T& gum, T& gu0, T& gup, T& gvm, T& gvp) {
  const T gl = g * ih;  // adjoint of h times the limited derivative
  T gd1, gd2, gVs, gVd;
  limit_blend_vjp(u0 - um, up - u0, h * (vm + vp), h * (vm - vp), w.g1, w.g2, w.eps, gl, gd1, gd2,
                  gVs, gVd);
  gup += gd2;
  gum -= gd1;
  gu0 += gd1 - gd2;
  gvm += h * (gVs + gVd);
  gvp += h * (gVs - gVd);
}

// reverse of point_fluxes() (accumulates): from adjoints of F, A = A_n Dn, B = A_n Dt.
// HAVE_F: gF and gA are given; MIXED: gB is given.
template <typename T, int PHYS, int M, bool MIXED, bool HAVE_F = true>
HW_HD void point_fluxes_vjp(const T* U, const T* Dn, const T* Dt, const Consts<T>& k, T an,
                            const T* gF, const T* gA, const T* gB, T* gU, T* gDn, T* gDt) {
  if constexpr (PHYS == PH_EULER) {
    const T rho = U[0], mn = U[1];
    const T ir = fast_rcp(rho);
    const T un = mn * ir;
    const T ut = (M == 4) ? U[2] * ir : T(0);
    const T hq2 = T(0.5) * (M == 4 ? mad(ut, ut, un * un) : un * un);
    const T p = k.gm1 * mad(-rho, hq2, U[M - 1]);
    const T H = (U[M - 1] + p) * ir;
    T gun = T(0), gut = T(0), gH = T(0), gq = T(0), gp = T(0), gmn = T(0);
    if constexpr (HAVE_F) {
      // F = (mn, mn un + p, mn ut, mn H)
      gmn = mad(un, gF[1], mad(H, gF[M - 1], gF[0]));
      gun = mn * gF[1];
      gp = gF[1];
      gH = mn * gF[M - 1];
      if constexpr (M == 4) gmn = mad(ut, gF[2], gmn), gut = mn * gF[2];
    }
    // the flux Jacobian's product with D = (r, a, b, e), as point_fluxes forms it
    auto jvp_vjp = [&](const T* D, const T* go, T* gD) {
      const T r = D[0], a = D[1], b = (M == 4) ? D[2] : T(0), e = D[M - 1];
      const T da = mad(-un, r, a), db = (M == 4) ? mad(-ut, r, b) : T(0);
      T dp = mad(hq2, r, mad(-un, a, e));
      if constexpr (M == 4) dp = mad(-ut, b, dp);
      dp *= k.gm1;
      const T g1 = go[1], g2 = (M == 4) ? go[2] : T(0), g3 = go[M - 1];
      const T gs = k.gm1 * mad(un, g3, g1);   // adjoint of dp / gm1
      const T gda = mad(un, g1, H * g3);
      gD[0] += mad(hq2, gs, -un * gda);
      gD[1] += mad(un, g1, go[0]) + mad(-un, gs, gda);
      gD[M - 1] += mad(un, g3, gs);
      gun += mad(a + da, g1, mad(e + dp, g3, mad(-r, gda, -a * gs)));
      gH = mad(da, g3, gH);
      gq = mad(r, gs, gq);
      if constexpr (M == 4) {
        const T gdb = un * g2;
        gD[0] = mad(-ut, gdb, gD[0]);
        gD[1] = mad(ut, g2, gD[1]);
        gD[2] += mad(-ut, gs, gdb);
        gun = mad(db, g2, gun);
        gut += mad(a, g2, mad(-r, gdb, -b * gs));
      }
    };
    if constexpr (HAVE_F) jvp_vjp(Dn, gA, gDn);
    if constexpr (MIXED) jvp_vjp(Dt, gB, gDt);
    // H = (E + p) / rho, p = gm1 (E - rho hq2), hq2 = (un^2 + ut^2)/2, un = mn / rho
    const T gHr = ir * gH;
    const T gpm = k.gm1 * (gp + gHr);
    gq = mad(-rho, gpm, gq);
    gun = mad(un, gq, gun) * ir;
    gU[1] += gmn + gun;
    T gr = mad(-H, gHr, mad(-hq2, gpm, -un * gun));
    if constexpr (M == 4) {
      gut = mad(ut, gq, gut) * ir;
      gU[2] += gut;
      gr = mad(-ut, gut, gr);
    }
    gU[0] += gr;
    gU[M - 1] += gHr + gpm;
  } else if constexpr (PHYS == PH_BURGERS) {
    if constexpr (HAVE_F) {
      gU[0] += U[0] * gF[0] + Dn[0] * gA[0];
      gDn[0] += U[0] * gA[0];
    }
    if constexpr (MIXED) {
      gU[0] += Dt[0] * gB[0];
      gDt[0] += U[0] * gB[0];
    }
  } else {
    if constexpr (HAVE_F) {
      gU[0] += an * gF[0];
      gDn[0] += an * gA[0];
    }
    if constexpr (MIXED) gDt[0] += an * gB[0];
  }
}

// adjoints of the Roe eigen-system quantities used by project() / back()
template <typename T>
struct EigenAdj {
  T un = 0, ut = 0, H = 0, c = 0, ic = 0, b1 = 0, hq2 = 0;
};

// reverse of Eigen::project(): gx = L^T gw, plus eigen-system adjoints
template <typename T, int M>
HW_HD void project_vjp(const Eigen<T, M>& e, const T* x, const T* gw, T* gx, EigenAdj<T>& ge) {
  // psi = (ic/2) (un x0 - x1), phi = x3 - un x1 - ut x2 + hq2 x0,
  // w = ((b1/2) phi + psi, x0 - b1 phi, x2 - ut x0, (b1/2) phi - psi)
  T phi = mad(e.hq2, x[0], mad(-e.un, x[1], x[M - 1]));
  if constexpr (M == 4) phi = mad(-e.ut, x[2], phi);
  const T gb = mad(T(0.5), gw[0] + gw[M - 1], -gw[1]);
  const T gphi = e.b1 * gb;
  const T hpsi = T(0.5) * (gw[0] - gw[M - 1]);
  const T gt = e.ic * hpsi;
  ge.b1 = mad(phi, gb, ge.b1);
  ge.ic = mad(mad(e.un, x[0], -x[1]), hpsi, ge.ic);
  ge.un = mad(x[0], gt, mad(-x[1], gphi, ge.un));
  ge.hq2 = mad(x[0], gphi, ge.hq2);
  T g0 = mad(e.hq2, gphi, mad(e.un, gt, gw[1]));
  if constexpr (M == 4) {
    g0 = mad(-e.ut, gw[2], g0);
    gx[2] = mad(-e.ut, gphi, gw[2]);
    ge.ut = mad(-x[2], gphi, mad(-x[0], gw[2], ge.ut));
  }
  gx[0] = g0;
  gx[1] = mad(-e.un, gphi, -gt);
  gx[M - 1] = gphi;
}

// reverse of Eigen::back(), in two parts: gw = R^T gy (needs no forward
// value), and the eigen-system adjoints (need the back-projected w)
template <typename T, int M>
HW_HD void back_T(const Eigen<T, M>& e, const T* gy, T* gw) {
  if constexpr (M == 4) {
    const T gs = gy[0] + e.un * gy[1] + e.ut * gy[2];
    const T gdif = e.c * gy[1] + e.un * e.c * gy[3];
    gw[0] = gs - gdif + e.H * gy[3];
    gw[1] = gs + e.hq2 * gy[3];
    gw[2] = gy[2] + e.ut * gy[3];
    gw[3] = gs + gdif + e.H * gy[3];
  } else {
    const T gs = gy[0] + e.un * gy[1];
    const T gdif = e.c * gy[1] + e.un * e.c * gy[2];
    gw[0] = gs - gdif + e.H * gy[2];
    gw[1] = gs + e.hq2 * gy[2];
    gw[2] = gs + gdif + e.H * gy[2];
  }
}

template <typename T, int M>
HW_HD void back_eigen_adj(const Eigen<T, M>& e, const T* w, const T* gy, EigenAdj<T>& ge) {
  if constexpr (M == 4) {
    const T s = w[0] + w[1] + w[3], dif = w[3] - w[0];
    ge.un += s * gy[1] + e.c * dif * gy[3];
    ge.c += dif * gy[1] + e.un * dif * gy[3];
    ge.ut += s * gy[2] + w[2] * gy[3];
    ge.H += (w[0] + w[3]) * gy[3];
    ge.hq2 += w[1] * gy[3];
  } else {
    const T s = w[0] + w[1] + w[2], dif = w[2] - w[0];
    ge.un += s * gy[1] + e.c * dif * gy[2];
    ge.c += dif * gy[1] + e.un * dif * gy[2];
    ge.H += (w[0] + w[2]) * gy[2];
    ge.hq2 += w[1] * gy[2];
  }
}

// reverse of Eigen::roe(): eigen-system adjoints -> adjoints of UL, UR (accumulated)
template <typename T, int M>
HW_HD void roe_vjp(const T* UL, const T* UR, T gm1, const EigenAdj<T>& g, T* gUL, T* gUR) {
  // the forward's arithmetic (Eigen::roe): sqrt(rho) and 1/rho from one
  // reciprocal square root per side
  const T qL = fast_rsq(UL[0]), qR = fast_rsq(UR[0]);
  const T sL = UL[0] * qL, sR = UR[0] * qR;
  const T irL = qL * qL, irR = qR * qR;
  const T uL = UL[1] * irL, uR = UR[1] * irR;
  const T tL = (M == 4) ? UL[2] * irL : T(0), tR = (M == 4) ? UR[2] * irR : T(0);
  const T pL = gm1 * (UL[M - 1] - T(0.5) * UL[0] * (uL * uL + tL * tL));
  const T pR = gm1 * (UR[M - 1] - T(0.5) * UR[0] * (uR * uR + tR * tR));
  const T HL = (UL[M - 1] + pL) * irL, HR = (UR[M - 1] + pR) * irR;
  const T iw = fast_rcp(sL + sR);
  const T wL = sL * iw, wR = sR * iw;
  const T un = wL * uL + wR * uR, ut = wL * tL + wR * tR, H = wL * HL + wR * HR;
  const T hq2 = T(0.5) * (un * un + ut * ut);
  const T c2 = gm1 * (H - hq2);
  const T ic = fast_rsq(c2);
  // b1 = gm1 ic^2, ic = 1/c, c = sqrt(gm1 (H - hq2))
  T ghq2 = g.hq2;
  const T gic = g.ic + T(2) * gm1 * ic * g.b1;
  const T gc = g.c - ic * ic * gic;
  const T gcc = gm1 * T(0.5) * ic * gc;
  const T gH = g.H + gcc;
  ghq2 -= gcc;
  const T gun = g.un + un * ghq2, gut = g.ut + ut * ghq2;
  // Roe weights
  const T gwL = uL * gun + tL * gut + HL * gH, gwR = uR * gun + tR * gut + HR * gH;
  const T giw = sL * gwL + sR * gwR;
  const T gsL = iw * gwL - iw * iw * giw, gsR = iw * gwR - iw * iw * giw;
  // q = 1 / sqrt(rho): d sqrt(rho) / d rho = q / 2
  auto side = [&](const T* U, T ir, T q, T u, T t, T p, T w, T gs, T* gU) {
    const T gHs = w * gH, gu = w * gun, gt = w * gut;
    T gE = ir * gHs, gp = ir * gHs, gir = (U[M - 1] + p) * gHs;
    gE += gm1 * gp;
    T grho = -T(0.5) * gm1 * (u * u + t * t) * gp;
    const T gu2 = gu - gm1 * U[0] * u * gp;
    const T gt2 = gt - gm1 * U[0] * t * gp;
    const T gm = ir * gu2;
    gir += U[1] * gu2;
    T gn = 0;
    if constexpr (M == 4) {
      gn = ir * gt2;
      gir += U[2] * gt2;
    }
    grho += T(0.5) * gs * q - ir * ir * gir;
    gU[0] += grho;
    gU[1] += gm;
    if constexpr (M == 4) gU[2] += gn;
    gU[M - 1] += gE;
  };
  side(UL, irL, qL, uL, tL, pL, wL, gsL, gUL);
  side(UR, irR, qR, uR, tR, pR, wR, gsR, gUR);
}

// reverse of limit_char_d(): adjoints of the cell's state and of d1, d2, Vs, Vd
// (overwritten) for the adjoint gout of h times the limited derivative (normal
// frame).  The cell's eigen-system is the Roe average of the cell with itself, so
// reversing roe() with both sides equal to u0 differentiates it exactly.
template <typename T, int M>
HW_HD void limit_char_d_vjp(const T* u0, const T* d1, const T* d2, const T* Vs, const T* Vd, T g1,
                            T g2, T eps, T gm1, const T* gout, T* gu0, T* gd1, T* gd2, T* gVs,
                            T* gVd) {
  Eigen<T, M> e;
  e.cell(u0, gm1);
  T a[M], b[M], s[M], d[M], z[M], gz[M], ga[M], gb[M], gs[M], gd[M];
  e.project(d1, a);
  e.project(d2, b);
  e.project(Vs, s);
  e.project(Vd, d);
  back_T(e, gout, gz);
#pragma unroll
  for (int q = 0; q < M; ++q)
    z[q] = limit_blend_vjp(a[q], b[q], s[q], d[q], g1, g2, eps, gz[q], ga[q], gb[q], gs[q], gd[q]);
  EigenAdj<T> ge;
  back_eigen_adj(e, z, gout, ge);
  project_vjp(e, d1, ga, gd1, ge);
  project_vjp(e, d2, gb, gd2, ge);
  project_vjp(e, Vs, gs, gVs, ge);
  project_vjp(e, Vd, gd, gVd, ge);
#pragma unroll
  for (int q = 0; q < M; ++q) gu0[q] = T(0);
  roe_vjp<T, M>(u0, u0, gm1, ge, gu0, gu0);
}

// reverse of limit_char(), likewise (accumulates into gum, gu0, gup, gvm, gvp)
template <typename T, int M>
HW_HD void limit_char_vjp(const T* um, const T* u0, const T* up, const T* vm, const T* vp, T h,
                          T ih, const Weights<T>& w, T gm1, const T* gout, T* gum, T* gu0,
                          T* gup, T* gvm, T* gvp) {
  T d1[M], d2[M], Vs[M], Vd[M], gl[M], g0[M], gd1[M], gd2[M], gVs[M], gVd[M];
#pragma unroll
  for (int q = 0; q < M; ++q) {
    d1[q] = u0[q] - um[q], d2[q] = up[q] - u0[q];
    Vs[q] = h * (vm[q] + vp[q]), Vd[q] = h * (vm[q] - vp[q]);
    gl[q] = ih * gout[q];
  }
  limit_char_d_vjp<T, M>(u0, d1, d2, Vs, Vd, w.g1, w.g2, w.eps, gm1, gl, g0, gd1, gd2, gVs, gVd);
#pragma unroll
  for (int q = 0; q < M; ++q) {
    gum[q] -= gd1[q];
    gu0[q] += g0[q] + (gd1[q] - gd2[q]);
    gup[q] += gd2[q];
    gvm[q] += h * (gVs[q] + gVd[q]);
    gvp[q] += h * (gVs[q] - gVd[q]);
  }
}

// ---------------------------------------------------------------------------
// One side of the VJP of interface_fluxes()' nonlinear flux fh = q + R w / 6.  The
// "+" side reads points 0, 1, 2, the mirrored "-" side points 3, 2, 1, in the roles
// upwind (a), own (o), downwind (b); ld(s, U, Dn) loads a point's state and scaled
// normal derivative.  gw = R^T gfh / 6 (adjoint of the side's reconstructed fields), gfh
// the adjoint of fh.  Returns the adjoints gx, gy of x = F +- alpha U and
// y = A Dn +- alpha Dn at the three points, adds the side's fields to w and its share
// of the eigen-system's adjoint to ge.  The point data's own adjoint (through the
// point fluxes) is linear in gx, gy and the same function for every interface
// that reads the cell, so the caller sums them per cell and differentiates it once.
// ---------------------------------------------------------------------------
template <typename T, int PHYS, int M, bool PROJ, typename Loader>
HW_HD void side_vjp(const Loader& ld, const bool plus, T alpha, T an, const Consts<T>& k,
                    const Eigen<T, M>& eg, const T* gw, const T* gfh, T* w, EigenAdj<T>& ge, T* gxa,
                    T* gya, T* gxo, T* gyo, T* gxb, T* gyb) {
  const T sg = plus ? T(1) : T(-1);
  const T al = sg * alpha;
  auto point = [&](const int s, T* x, T* y) __attribute__((always_inline)) {
    T U[M], Dn[M], F[M], A[M];
    ld(s, U, Dn);
    point_fluxes<T, PHYS, M, false>(U, Dn, Dn, k, an, F, A, A);
#pragma unroll
    for (int c = 0; c < M; ++c) x[c] = mad(al, U[c], F[c]), y[c] = mad(al, Dn[c], A[c]);
  };
  T A[M], B[M], H0[M], Hs[M], Hd[M];
  {
    T xo[M], xa[M], ya[M], yb[M];
    point(plus ? 1 : 2, xo, H0);
    point(plus ? 2 : 1, B, yb);
    point(plus ? 0 : 3, xa, ya);
#pragma unroll
    for (int c = 0; c < M; ++c) {
      A[c] = xa[c] - xo[c];
      B[c] -= xo[c];
      Hs[c] = ya[c] + yb[c];
      Hd[c] = ya[c] - yb[c];
    }
  }
  T gA[M], gB[M], gH0[M], gHs[M], gHd[M];
  auto fields = [&](const T* a, const T* b, const T* h0, const T* hs, const T* hd)
      __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < M; ++c) {
      w[c] += hw_blend_vjp(a[c], b[c], sg * h0[c], sg * hs[c], sg * hd[c], k.rw.g1, k.rw.g2,
                           k.rb.eps, gw[c], gA[c], gB[c], gH0[c], gHs[c], gHd[c]);
      gH0[c] *= sg, gHs[c] *= sg, gHd[c] *= sg;
    }
  };
  if constexpr (PROJ) {
    T a[M], b[M], h0[M], hs[M], hd[M];
    eg.project(A, a);
    eg.project(B, b);
    eg.project(H0, h0);
    eg.project(Hs, hs);
    eg.project(Hd, hd);
    fields(a, b, h0, hs, hd);
    project_vjp(eg, A, gA, a, ge);
    project_vjp(eg, B, gB, b, ge);
    project_vjp(eg, H0, gH0, h0, ge);
    project_vjp(eg, Hs, gHs, hs, ge);
    project_vjp(eg, Hd, gHd, hd, ge);
#pragma unroll
    for (int c = 0; c < M; ++c) gA[c] = a[c], gB[c] = b[c], gH0[c] = h0[c], gHs[c] = hs[c], gHd[c] = hd[c];
  } else {
    fields(A, B, H0, Hs, Hd);
  }
#pragma unroll
  for (int c = 0; c < M; ++c) {
    gxa[c] = gA[c];
    gxb[c] = gB[c];
    gxo[c] = gfh[c] - (gA[c] + gB[c]);
    gya[c] = gHs[c] + gHd[c];
    gyb[c] = gHs[c] - gHd[c];
    gyo[c] = mad(sg * T(0.5), gfh[c], gH0[c]);
  }
}

}  // namespace hweno
