// Device math of the L-HWENO hot path for gfx950 (header-only, templated on
// the real type).  Zhang & Zhao, arXiv 2207.05258, Section 2.
//
// Everything here is per-lane scalar code: the stencil work is a VALU problem
// (every interface has its own 4x4 eigenbasis, so there is no shared-operand
// contraction for MFMA).  The formulas are rearranged for few divisions:
//   * the convex combination of Sections 2.1/2.2 is evaluated with a single
//     division in FP64 (numerator and denominator scaled by the product of
//     the three (beta_l + eps)) and with hardware reciprocals in FP32;
//   * the Euler characteristic projection L = R^{-1} and back projection R
//     use the closed-form eigenvectors and their shared sub-expressions;
//   * the linear derivative flux h-hat = p0'^+ + p0'^- is pre-combined over
//     the four stencil points (one set of coefficients on F, U, A U_n, U_n).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// math below is host+device so that it can be unit-checked on the CPU
#define HW_HD __host__ __device__ __forceinline__

namespace hweno {

enum { PH_LINADV = 0, PH_BURGERS = 1, PH_EULER = 2 };

template <int PHYS, int DIM>
struct Comps {
  static constexpr int M = (PHYS == PH_EULER) ? (DIM == 1 ? 3 : 4) : 1;
  static constexpr int NF = M * (1 + DIM);
};

template <typename T>
struct Weights {
  T g0, g1, g2;  // linear weights, positive, summing to one
  T eps;         // epsilon of the nonlinear weights
  T gs;          // g0 + g1 + g2: one, so no formula below reads it
};

// a b + c, rounded once
HW_HD double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }
HW_HD float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// What the nonlinear combination needs of a set of linear weights, in the units
// it works in (blend_c): of the second and third candidate's weights, and eps.
template <typename T>
struct Blend {
  T a1, a2, eps;
};

template <typename T>
struct Consts {
  Weights<T> rw;  // reconstruction weights gamma_l (Section 2.1)
  Weights<T> lw;  // limiter weights d_l (Section 2.2)
  T gm1;          // gamma_gas - 1
  T gam;          // gamma_gas
  T ax, ay;       // advection speeds (linear advection)
  int limiter_on;
  int limiter_char;  // Euler: limiter on characteristic fields of each cell
  Blend<T> rb;    // rw and lw in the kernels' units (recon_blend, limit_blend)
  Blend<T> lb;
};

// Reciprocal and reciprocal square root of finite, positive, normal
// arguments (densities, squared sound speeds, indicators) without the IEEE
// special-case scaling of the library routines.
// FP32: the hardware instructions (1 ulp).  FP64: the hardware approximation
// (relative error about 2^-24 on gfx950, measured) refined by one Newton step,
// which leaves about 2^-48.  The host build of the math (CPU unit checks) divides.
template <typename T>
HW_HD T fast_rcp(T x);
template <>
HW_HD float fast_rcp<float>(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(x);  // v_rcp_f32
#else
  return 1.0f / x;
#endif
}
template <>
HW_HD double fast_rcp<double>(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const double r = __builtin_amdgcn_rcp(x);  // v_rcp_f64
  return mad(r, mad(-x, r, 1.0), r);
#else
  return 1.0 / x;
#endif
}

template <typename T>
HW_HD T fast_rsq(T x);
template <>
HW_HD float fast_rsq<float>(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rsqf(x);  // v_rsq_f32
#else
  return 1.0f / sqrtf(x);
#endif
}
template <>
HW_HD double fast_rsq<double>(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const double y = __builtin_amdgcn_rsq(x);  // v_rsq_f64
  // y <- y (3 - x y^2) / 2
  return mad(0.5 * y, mad(-x * y, y, 1.0), y);
#else
  return 1.0 / sqrt(x);
#endif
}

// Quotient n / d of a finite n and a positive normal d, without that scaling
// either.  FP64: the error e of the hardware reciprocal (about 2^-24) is expanded to
// second order, q (1 + e + e^2), which leaves 2^-72 and the roundings of q and of the
// result, about 1 ulp.
template <typename T>
HW_HD T blend_div(T n, T d) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (sizeof(T) == 8) {
    const T r = __builtin_amdgcn_rcp(d);
    const T e = mad(-d, r, T(1));
    const T q = n * r;
    return mad(q, mad(e, e, e), q);
  } else {
    return n * fast_rcp(d);
  }
#else
  return n / d;
#endif
}

// ---------------------------------------------------------------------------
// Convex combination shared by the reconstruction (Section 2.1) and the
// limiter (Section 2.2):
//   tau = (|b0-b1| + |b0-b2|)^2 / 4,  wbar_l = g_l (1 + tau/(b_l + eps)),
//   result = w0 (P0/g0 - g1/g0 P1 - g2/g0 P2) + w1 P1 + w2 P2, w = wbar/sum.
// With c_l = b_l + eps and e_l = 1 + tau/c_l and weights that sum to one this is
//   (e0 P0 + g1 P1 (e1-e0) + g2 P2 (e2-e0)) / (e0 + g1 (e1-e0) + g2 (e2-e0)),
// and a part q common to the three candidates comes out whole: only the
// candidates' differences R_l = P_l - q are combined and divided, so q never
// passes through the projections or the quotient.
// The denominator does not cancel, whatever the weights: the high-degree indicator is
// never far below the others (c0 >= 0.89 c1, 0.89 c2 in the reconstruction, 0.80 in the
// limiter, for all data), so e0 is at most 1.25 times each e_l and the denominator at
// least 0.8 e0.
// The callers scale their indicators so that a square needs no weight; e_l is
// then 1 + kappa t^2 / c_l with t = |c0-c1| + |c0-c2|.
// FP64: numerator and denominator times c0 c1 c2 (one division), with kappa folded
// into a_l = kappa g_l:
//   m = c1 c2 (c0 + kappa t^2), s1 = a1 c2 (c0 - c1), s2 = a2 c1 (c0 - c2),
//   result = (m R0 + t^2 (s1 R1 + s2 R2)) / (m + t^2 (s1 + s2)).
// FP32: one reciprocal per indicator (the products leave the FP32 range when the
// indicators span many decades) and a_l = g_l; kappa stays in tau = kappa t^2,
// which keeps tau / c_l in range up to the same data as the scheme's own tau.
// num(m, s1, s2, f) forms the numerator from m = e0-, s_l = g_l (e_l - e0)-like
// factors (f: a common factor of the last two); KAP48: kappa in units of 1/48.
// ---------------------------------------------------------------------------
template <int KAP48>
HW_HD constexpr double sqrt_kappa() {
  static_assert(KAP48 == 13 || KAP48 == 12, "kappa of the reconstruction or of the limiter");
  return KAP48 == 13 ? 0.52041649986653316 : 0.5;
}

template <int KAP48, typename T, typename Num>
HW_HD T blend_c(T c0, T c1, T c2, const Blend<T>& w, const Num& num) {
  const T d01 = c0 - c1, d02 = c0 - c2;
  const T t = fabs(d01) + fabs(d02);
  if constexpr (sizeof(T) == 8) {
    const T t2 = t * t;
    const T m = (c1 * c2) * mad(T(KAP48 / 48.0), t2, c0);
    const T s1 = (w.a1 * c2) * d01, s2 = (w.a2 * c1) * d02;
    return blend_div(num(m, s1, s2, t2), mad(t2, s1 + s2, m));
  } else {
    const T st = T(sqrt_kappa<KAP48>()) * t;
    const T tau = st * st;
    const T k0 = tau * fast_rcp(c0);
    const T m = T(1) + k0;
    const T s1 = w.a1 * (tau * fast_rcp(c1) - k0), s2 = w.a2 * (tau * fast_rcp(c2) - k0);
    return blend_div(num(m, s1, s2, T(1)), (m + s1) + s2);
  }
}

// Reconstruction weights for hw_blend, whose data are twice the split fluxes
// and whose indicators carry 12/13: kappa = 13/48, eps 12/13 (FP32: kept normal, as
// the hardware reciprocal takes a denormal for zero).
template <typename T>
HW_HD Blend<T> recon_blend(T g1, T g2, T eps) {
  const T kap = sizeof(T) == 8 ? T(13.0 / 48.0) : T(1);
  T e = T(12.0 / 13.0) * eps;
  if constexpr (sizeof(T) == 4) e = e < T(1.17549435e-38) ? T(1.17549435e-38) : e;
  return Blend<T>{kap * g1, kap * g2, e};
}
// limiter weights for limit_blend: kappa = 1/4
template <typename T>
HW_HD Blend<T> limit_blend_weights(T d1, T d2, T eps) {
  const T kap = sizeof(T) == 8 ? T(0.25) : T(1);
  return Blend<T>{kap * d1, kap * d2, eps};
}

// Nonlinear HWENO value at x_{i+1/2} (Section 2.1) from the upwind ("+") data
// f_{i-1}, f_i, f_{i+1} and H_l = dx h_l, as f_i + H_i / 2 plus a correction:
// this returns 12 times the correction, from doubled data in the combinations
//   A = 2 (f_{i-1} - f_i), B = 2 (f_{i+1} - f_i), H0 = 2 H_i,
//   Hs = 2 (H_{i-1} + H_{i+1}), Hd = 2 (H_{i-1} - H_{i+1}).
// With u1 = H0 + A, u2 = H0 - B (the curvatures of the quadratics) and
// lap = u1 - u2, t = u1 + u2, in single data the candidates are
//   p0 = f0 + H0/2 + 11/60 lap + Hd/20, p1 = f0 + H0/2 + u1/6, p2 = f0 + H0/2 - u2/6
// and the indicators b1 = H0^2 + 13/3 u1^2, b2 = H0^2 + 13/3 u2^2 (from the
// definition, eq. GHYZ), b0 = H0^2 + a sum of four squares: in the monomial
// coefficients of the quintic
//   (a1 + a3/4 + a5/16)^2 + 13/3 (a2 + 63/130 a4)^2 + 781/20 (a3 + 8825/10934 a5)^2
//   + 1421461/2275 a4^2 + 21520059541/1377684 a5^2,
// whose first form is H0 (p0'(x_i) dx = H_i, a Hermite condition).  The second and
// fourth squares are a quadratic form of (Hd, lap), the third and fifth one of
// (Hs - 2 H0, t); each pair is rotated so that its second square is of lap, or
// t, alone.  All three indicators carry the factor 3/13 (12/13 on single data),
// which frees the squares of u1 and u2 from their weight.
template <typename T>
HW_HD T hw_blend(T A, T B, T H0, T Hs, T Hd, const Blend<T>& w) {
  const T u1 = H0 + A, u2 = H0 - B;
  const T lap = u1 - u2, t = u1 + u2;
  const T R0 = mad(T(1.1), lap, T(0.3) * Hd);  // 6 (p0 - f0 - H0/2)
  const T y = mad(T(6.067488135033763), lap, T(3.012679250059034) * Hd);
  const T z = mad(T(15.029579351881592), mad(T(-2), H0, Hs), T(45.165651404159786) * t);
  const T h = mad(T(3.0 / 13.0) * H0, H0, w.eps);
  const T c0 = mad(T(0.24822509386187025) * lap, lap,
                   mad(T(2.2469689522048239) * t, t, mad(z, z, mad(y, y, h))));
  return blend_c<13>(c0, mad(u1, u1, h), mad(u2, u2, h), w,
                     [=](T m, T s1, T s2, T f) { return mad(m, R0, f * mad(s1, u1, -(s2 * u2))); });
}

// the whole value (single data): hw_blend as the scheme's formula is written, for
// checks against it
template <typename T>
HW_HD T hw_plus(T fm, T f0, T fp, T Hm, T H0, T Hp, const Weights<T>& w) {
  const T r = hw_blend(T(2) * (fm - f0), T(2) * (fp - f0), T(2) * H0, T(2) * (Hm + Hp),
                       T(2) * (Hm - Hp), recon_blend(w.g1, w.g2, w.eps));
  return mad(T(1.0 / 12.0), r, mad(T(0.5), H0, f0));
}

// HWENO limiter (Section 2.2): h v~_i from d1 = u_i - u_{i-1}, d2 = u_{i+1} - u_i,
// Vs = h (v_{i-1} + v_{i+1}), Vd = h (v_{i-1} - v_{i+1}).  Candidates (quartic q0,
// linear q1, q2), with D = d1 + d2, lap = d2 - d1, e = Vs - D: 3/4 D - Vs/4, d1, d2,
// combined whole: a part common to them, D/2, would carry a jump's rounding into
// a limited value on its smooth side.  The quartic's indicator from its
// coefficients a1..a4,
//   (a1 + a3/4)^2 + 13/3 (a2 + 63/130 a4)^2 + 781/20 a3^2 + 1421461/2275 a4^2,
// is a sum of squares of linear forms; the second and fourth are a quadratic
// form of (Vd, lap), rotated so that one square is of lap alone.
template <typename T>
HW_HD T limit_blend(T d1, T d2, T Vs, T Vd, const Blend<T>& w) {
  const T D = d1 + d2, lap = d2 - d1, e = Vs - D;
  const T x0 = mad(T(0.5), D, T(-3.0 / 16.0) * e);  // a1 + a3/4
  const T a1 = mad(T(0.75), D, T(-0.25) * Vs);
  const T y = mad(T(12.554318802466193), lap, T(6.254843361443233) * Vd);
  const T c0 = mad(T(1.0813413108057222) * lap, lap,
                   mad(T(2.440625) * e, e, mad(y, y, mad(x0, x0, w.eps))));
  return blend_c<12>(c0, mad(d1, d1, w.eps), mad(d2, d2, w.eps), w,
                     [=](T m, T s1, T s2, T f) { return mad(m, a1, f * mad(s1, d1, s2 * d2)); });
}

// limited derivative from u_{i-1}, u_i, u_{i+1}, v_{i-1}, v_{i+1}; h = dx, ih = 1/dx
template <typename T>
HW_HD T limit1(T um, T u0, T up, T vm, T vp, T h, T ih, const Weights<T>& w) {
  return ih * limit_blend(u0 - um, up - u0, h * (vm + vp), h * (vm - vp),
                          limit_blend_weights(w.g1, w.g2, w.eps));
}

// ---------------------------------------------------------------------------
// Physics in a normal-direction frame.  For 2D Euler the components are
// ordered (rho, m_n, m_t, E): normal momentum first, so one code path serves
// both directions (y swaps the two momenta on load and store).
// ---------------------------------------------------------------------------

// flux F_n(U) and the chain-rule products A_n(U) Dn and A_n(U) Dt
// (h, xi, eta, theta of eq. EQ3), for one stencil point.
template <typename T, int PHYS, int M, bool MIXED>
HW_HD void point_fluxes(const T* U, const T* Dn, const T* Dt,
                                             const Consts<T>& k, T an, T* F,
                                             T* A, T* B) {
  if constexpr (PHYS == PH_EULER) {
    const T ir = fast_rcp(U[0]);
    const T un = U[1] * ir;
    const T ut = (M == 4) ? U[2] * ir : T(0);
    const T hq2 = T(0.5) * (M == 4 ? mad(ut, ut, un * un) : un * un);
    const T p = k.gm1 * mad(-U[0], hq2, U[M - 1]);
    const T H = (U[M - 1] + p) * ir;
    F[0] = U[1];
    F[1] = mad(U[1], un, p);
    if constexpr (M == 4) F[2] = U[1] * ut;
    F[M - 1] = U[1] * H;
    // the flux Jacobian on D = (r, a, b, e): with da = a - un r, db = b - ut r and
    // dp the pressure's change, (a, un (a + da) + dp, ut a + un db, H da + un (e + dp))
    auto jvp = [&](const T* D, T* out) {
      const T r = D[0], a = D[1], e = D[M - 1];
      const T da = mad(-un, r, a);
      T dp = mad(hq2, r, mad(-un, a, e));
      if constexpr (M == 4) dp = mad(-ut, D[2], dp);
      dp *= k.gm1;
      out[0] = a;
      out[1] = mad(un, a + da, dp);
      if constexpr (M == 4) out[2] = mad(ut, a, un * mad(-ut, r, D[2]));
      out[M - 1] = mad(H, da, un * (e + dp));
    };
    jvp(Dn, A);
    if constexpr (MIXED) jvp(Dt, B);
  } else if constexpr (PHYS == PH_BURGERS) {
    F[0] = T(0.5) * U[0] * U[0];
    A[0] = U[0] * Dn[0];
    if constexpr (MIXED) B[0] = U[0] * Dt[0];
  } else {
    F[0] = an * U[0];
    A[0] = an * Dn[0];
    if constexpr (MIXED) B[0] = an * Dt[0];
  }
}

// Roe-averaged eigen-system of the normal flux Jacobian: right eigenvectors
// (1, un-c, ut, H-un c), (1, un, ut, q^2/2), (0, 0, 1, ut), (1, un+c, ut, H+un c)
// (1D drops ut), left eigenvectors = their inverse in closed form.
template <typename T, int M>
struct Eigen {
  T un, ut, H, c, ic, b1, hq2;

  HW_HD void roe(const T* UL, const T* UR, T gm1) {
    // sqrt(rho) and 1/rho from one reciprocal square root per side
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
    un = wL * uL + wR * uR;
    ut = wL * tL + wR * tR;
    H = wL * HL + wR * HR;
    const T q2 = un * un + ut * ut;
    hq2 = T(0.5) * q2;
    const T c2 = gm1 * (H - hq2);
    ic = fast_rsq(c2);
    c = c2 * ic;
    b1 = gm1 * ic * ic;
  }

  // eigen-system at one state (what the Roe average of a state with itself gives)
  HW_HD void cell(const T* U, T gm1) {
    const T ir = fast_rcp(U[0]);
    un = U[1] * ir;
    ut = (M == 4) ? U[2] * ir : T(0);
    hq2 = T(0.5) * (un * un + ut * ut);
    const T p = gm1 * (U[M - 1] - U[0] * hq2);
    H = (U[M - 1] + p) * ir;
    const T c2 = gm1 * (H - hq2);
    ic = fast_rsq(c2);
    c = c2 * ic;
    b1 = gm1 * ic * ic;
  }

  // w = L x
  HW_HD void project(const T* x, T* w) const {
    const T psi = (T(0.5) * ic) * mad(un, x[0], -x[1]);
    T phi = mad(hq2, x[0], mad(-un, x[1], x[M - 1]));
    if constexpr (M == 4) phi = mad(-ut, x[2], phi);
    w[0] = mad(T(0.5) * b1, phi, psi);
    w[1] = mad(-b1, phi, x[0]);
    if constexpr (M == 4) w[2] = mad(-ut, x[0], x[2]);
    w[M - 1] = mad(T(0.5) * b1, phi, -psi);
  }

  // y = R w
  HW_HD void back(const T* w, T* y) const {
    const T w03 = w[0] + w[M - 1], s = w03 + w[1], cd = c * (w[M - 1] - w[0]);
    y[0] = s;
    y[1] = mad(un, s, cd);
    if constexpr (M == 4) y[2] = mad(ut, s, w[2]);
    T e = mad(hq2, w[1], mad(un, cd, H * w03));
    if constexpr (M == 4) e = mad(ut, w[2], e);
    y[M - 1] = e;
  }
};

// Characteristic variant of the limiter, h times the limited derivative, from
// the differences of limit_blend.
template <typename T, int M>
HW_HD void limit_char_d(const T* u0, const T* d1, const T* d2, const T* Vs, const T* Vd,
                        const Blend<T>& w, T gm1, T* out) {
  Eigen<T, M> e;
  e.cell(u0, gm1);
  T a[M], b[M], s[M], d[M], z[M];
  e.project(d1, a);
  e.project(d2, b);
  e.project(Vs, s);
  e.project(Vd, d);
#pragma unroll
  for (int q = 0; q < M; ++q) z[q] = limit_blend(a[q], b[q], s[q], d[q], w);
  e.back(z, out);
}

// Characteristic variant of the limiter (a choice the paper leaves open for
// systems): the five stencil vectors u_{i-1}, u_i, u_{i+1}, v_{i-1}, v_{i+1}
// (normal frame) are projected with the left eigenvectors of the cell's own
// state, each characteristic field is limited as a scalar, and the right
// eigenvectors map the result back.
template <typename T, int M>
HW_HD void limit_char(const T* um, const T* u0, const T* up, const T* vm, const T* vp, T h, T ih,
                      const Weights<T>& w, T gm1, T* out) {
  T d1[M], d2[M], Vs[M], Vd[M];
#pragma unroll
  for (int q = 0; q < M; ++q) {
    d1[q] = u0[q] - um[q], d2[q] = up[q] - u0[q];
    Vs[q] = h * (vm[q] + vp[q]), Vd[q] = h * (vm[q] - vp[q]);
  }
  limit_char_d<T, M>(u0, d1, d2, Vs, Vd, limit_blend_weights(w.g1, w.g2, w.eps), gm1, out);
#pragma unroll
  for (int q = 0; q < M; ++q) out[q] *= ih;
}

// ---------------------------------------------------------------------------
// All fluxes of one interface x_{i+1/2} along the normal direction.
// Stencil points s = 0..3 are x_{i-1}, x_i, x_{i+1}, x_{i+2};
// ld(s, U, Dn, Dt) loads the state of point s in the normal frame, the normal
// derivative times the cell size h of this direction and the tangential one
// times its own.  With x = F + alpha U, y = h (A Dn) + alpha h Dn ("+" data) and
// the same with -alpha ("-" data), i.e. twice the split fluxes, this returns
// (normal frame):
//   fh: twice f-hat (nonlinear, Section 2.1 with Remarks 2.1/2.2);
//   hh: 8 h times h-hat = p0'^+ + p0'^- (linear, component-wise):
//       x+_0 - 8 x+_1 + 7 x+_2 + (y+_0 - 2 y+_1 - 5 y+_2)/3 and its mirror image.
//       In 7 (x+_2 - x+_1) and its image alpha U cancels. As 14 (F_2 - F_1), which
//       also is the fewest instructions, it leaves no rounding behind (FP32, of the
//       point data's size: 3.5e-8 on smooth and 1.6e-8 on rough Euler stencils,
//       against 5.7e-8 and 2.3e-8 with x+ and x-);
//   xx: 12 times the mixed flux of eq. (mixed), of the scaled derivative
//       (only when MIXED).
// Each side needs its points only in the differences and sums that hw_blend
// takes; what is common to the candidates (f_i + H_i/2) stays in components and
// skips the eigenvectors.  PROJ: reconstruct in characteristic fields.
// The stage kernels are bound by VALU issue, so the form is the one with the
// fewest instructions: with the point data themselves projected, the scheme's
// factors applied where they occur and the linear fluxes summed point by point, a
// 2D Euler stage counted 3414 VALU lane-instructions per cell in FP64, in this
// form 2721; two steps of 4096^2 in FP64 went from 13.05 to 11.45 ms, four
// of 2047 x 1531 in FP32 from 2.79 to 2.57 ms.
//   alpha: global LF speed of this direction.
// ---------------------------------------------------------------------------
template <typename T, int PHYS, int M, bool MIXED, bool PROJ, typename Loader>
HW_HD void interface_fluxes(const Loader& ld, T alpha, T an, const Consts<T>& k, T* fh, T* hh,
                            T* xx) {
  Eigen<T, M> eg;
  T xp0[M], yp0[M], xp1[M], yp1[M], xm1[M], ym1[M], xp2[M], yp2[M], xm2[M], ym2[M];
  auto point = [&](const int s, T* xp, T* yp, T* xm, T* ym, T* U, T* F, T* B) __attribute__((always_inline)) {
    T Dn[M], Dt[M], A[M];
    ld(s, U, Dn, Dt);
    point_fluxes<T, PHYS, M, MIXED>(U, Dn, Dt, k, an, F, A, B);
#pragma unroll
    for (int c = 0; c < M; ++c) {
      if (s < 3) xp[c] = mad(alpha, U[c], F[c]), yp[c] = mad(alpha, Dn[c], A[c]);
      if (s > 0) xm[c] = mad(-alpha, U[c], F[c]), ym[c] = mad(-alpha, Dn[c], A[c]);
    }
  };
  // one side from its upwind neighbour (xa, ya), its own cell (xo, yo) and its
  // downwind one (xb, yb); sg: the sign that the mirror image gives derivatives
  T w[M], q[M], dF[M];
  auto side = [&](const bool plus, const T* xa, const T* ya, const T* xo, const T* yo, const T* xb,
                  const T* yb) __attribute__((always_inline)) {
    const T sg = plus ? T(1) : T(-1);
    T A[M], B[M], Hs[M], Hd[M];
#pragma unroll
    for (int c = 0; c < M; ++c) {
      A[c] = xa[c] - xo[c];
      B[c] = xb[c] - xo[c];
      Hs[c] = ya[c] + yb[c];
      Hd[c] = ya[c] - yb[c];
      const T l = mad(T(-2.0 / 3.0), Hs[c] + yo[c], mad(sg, A[c], Hd[c]));
      hh[c] = plus ? l : mad(T(14), dF[c], hh[c] + l);
      const T o = mad(sg * T(0.5), yo[c], xo[c]);
      q[c] = plus ? o : q[c] + o;
    }
    if constexpr (PROJ) {
      T a[M], b[M], h0[M], hs[M], hd[M];
      eg.project(A, a);
      eg.project(B, b);
      eg.project(yo, h0);
      eg.project(Hs, hs);
      eg.project(Hd, hd);
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const T r = plus ? hw_blend(a[c], b[c], h0[c], hs[c], hd[c], k.rb)
                         : hw_blend(a[c], b[c], -h0[c], -hs[c], -hd[c], k.rb);
        w[c] = plus ? r : w[c] + r;
      }
    } else {
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const T r = hw_blend(A[c], B[c], sg * yo[c], sg * Hs[c], sg * Hd[c], k.rb);
        w[c] = plus ? r : w[c] + r;
      }
    }
  };
  T U1[M], U2[M], Ue[M], F1[M], F2[M], b[M], bm[M];
  point(1, xp1, yp1, xm1, ym1, U1, F1, bm);
  point(2, xp2, yp2, xm2, ym2, U2, F2, b);
#pragma unroll
  for (int c = 0; c < M; ++c) dF[c] = F2[c] - F1[c];
  if constexpr (MIXED) {
#pragma unroll
    for (int c = 0; c < M; ++c) xx[c] = T(7) * (bm[c] + b[c]);
  }
  if constexpr (PROJ) eg.roe(U1, U2, k.gm1);
  point(0, xp0, yp0, nullptr, nullptr, Ue, F1, b);
  if constexpr (MIXED) {
#pragma unroll
    for (int c = 0; c < M; ++c) xx[c] -= b[c];
  }
  side(true, xp0, yp0, xp1, yp1, xp2, yp2);
  point(3, nullptr, nullptr, xp0, yp0, Ue, F1, b);
  if constexpr (MIXED) {
#pragma unroll
    for (int c = 0; c < M; ++c) xx[c] -= b[c];
  }
  side(false, xp0, yp0, xm2, ym2, xm1, ym1);
  if constexpr (PROJ) {
    T y[M];
    eg.back(w, y);
#pragma unroll
    for (int c = 0; c < M; ++c) fh[c] = mad(T(1.0 / 6.0), y[c], q[c]);
  } else {
#pragma unroll
    for (int c = 0; c < M; ++c) fh[c] = mad(T(1.0 / 6.0), w[c], q[c]);
  }
}

// wave speeds |u_n| + c (Euler), |u| (Burgers), |a| (linear advection) of
// one point in each direction, plus admissibility flags.
template <typename T, int PHYS, int DIM>
HW_HD void point_speeds(const T* U, const Consts<T>& k,
                                             T& sx, T& sy, uint32_t& flags) {
  if constexpr (PHYS == PH_EULER) {
    constexpr int M = Comps<PHYS, DIM>::M;
    const T r = U[0];
    const T ir = T(1) / r;
    const T u = U[1] * ir;
    const T v = (DIM == 2) ? U[2] * ir : T(0);
    const T p = k.gm1 * (U[M - 1] - T(0.5) * r * (u * u + v * v));
    const T c = sqrt(k.gam * p * ir);
    sx = fabs(u) + c;
    sy = (DIM == 2) ? fabs(v) + c : T(0);
    bool fin = true;
#pragma unroll
    for (int q = 0; q < M; ++q) fin = fin && isfinite(U[q]);
    if (!fin) flags |= 1u;
    if (!(r > T(0))) flags |= 2u;
    if (!(p > T(0))) flags |= 4u;
  } else if constexpr (PHYS == PH_BURGERS) {
    sx = fabs(U[0]);
    sy = (DIM == 2) ? sx : T(0);
    if (!isfinite(U[0])) flags |= 1u;
  } else {
    sx = fabs(k.ax);
    sy = (DIM == 2) ? fabs(k.ay) : T(0);
    if (!isfinite(U[0])) flags |= 1u;
  }
}

}  // namespace hweno
