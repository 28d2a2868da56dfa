// Reverse-mode (vector-Jacobian) counterparts of the per-zone and per-face
// computations of the WENO5-CT sweep, FP64, for the adjoint of a stage.
//
// Each *_vjp function recomputes what it needs of the forward pass and
// propagates a cotangent backwards through it.  Non-smooth points take the
// derivative of the branch the forward pass takes: max() of the Lax-Friedrichs
// speed follows the larger argument (ties: the first), |x| its sign (0 at 0),
// the clamps of alpha_f^2, alpha_s^2 and the degenerate constants of Appendix A
// (beta, sgn(B_n), alpha_f = alpha_s = 1/sqrt2) have zero derivative, and
// sqrt(0) contributes nothing.
#pragma once
#include <type_traits>

#include "mhd_device.hpp"

namespace wm {

// ---------------------------------------------------------------------------
// face eigen-system scalars: cotangents of the FaceEig members -> face state
// ---------------------------------------------------------------------------
// Materialises x in a register at this point of the program: the compiler may
// not sink the computation of x past it (without this, the terms of the
// cotangent sums below are kept live until their final use and spill).
__host__ __device__ __forceinline__ void pin(double& x) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+v"(x));
#else
  (void)x;
#endif
}

// Compiler-level memory clobber: loads after it are not merged with loads
// before it (re-reading the differences from LDS is cheaper than keeping them
// live in registers).
__host__ __device__ __forceinline__ void reload_fence() {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" ::: "memory");
#endif
}

// Cotangents of the face eigen-system in terms of thirteen of its scalars; each
// pair's reverse takes the others through their definitions at once (Gamma_f,
// Gamma_s, Gamma_a, v^2, c^2 by the members below, q = 1/(4 a^2), tau and c_s by
// a^2, sqrt(rho) and its reciprocal by rho), so that no more stay live across the
// next pair.
struct EigCot {
  double rho, vn, vt1, vt2, Bt1, Bt2, a2, cf, csl, by, bz, af, as;
  __host__ __device__ __forceinline__ void zero() {
    rho = vn = vt1 = vt2 = Bt1 = Bt2 = a2 = cf = csl = by = bz = af = as = 0.0;
  }
  __host__ __device__ __forceinline__ void pin_all() {
    pin(rho); pin(vn); pin(vt1); pin(vt2); pin(Bt1); pin(Bt2); pin(a2); pin(cf); pin(csl); pin(by); pin(bz);
    pin(af); pin(as);
  }
  __host__ __device__ __forceinline__ void add_v2(const FaceEig& e, double l) {
    vn += 2.0 * e.vn * l; vt1 += 2.0 * e.vt1 * l; vt2 += 2.0 * e.vt2 * l;
  }
  __host__ __device__ __forceinline__ void add_bv(const FaceEig& e, double l) {   // bv = by vt1 + bz vt2
    by += l * e.vt1; vt1 += l * e.by; bz += l * e.vt2; vt2 += l * e.bz;
  }
  // q = 1/(4 a^2) and c_s = sqrt(a^2)
  __host__ __device__ __forceinline__ void add_q(const FaceEig& e, double l) { a2 -= 4.0 * e.qa2 * e.qa2 * l; }
  __host__ __device__ __forceinline__ void add_cs(const FaceEig& e, double l) { a2 += 2.0 * e.qa2 * e.cs * l; }
  // sqrt(rho), 1/sqrt(rho)
  __host__ __device__ __forceinline__ void add_sr(const FaceEig& e, double l) { rho += 0.5 * e.isr * l; }
  __host__ __device__ __forceinline__ void add_isr(const FaceEig& e, double l) {
    rho -= 0.5 * e.isr * e.isr * e.isr * l;
  }
};

// Reverse of face_eig: out[0..7] = d/d(rho, vn, vt1, vt2, Bn, Bt1, Bt2, P).
__host__ __device__ __forceinline__ void face_eig_vjp(const double fp[8], const Phys& ph, const FaceEig& e,
                                                      const EigCot& eb, double out[8]) {
  const double rho = fp[0], Bn = fp[4], Bt1 = fp[5], Bt2 = fp[6], P = fp[7];
  const double gamma = ph.gamma;
  const double isr = rsq_nr(rho);
  const double irho = isr * isr;
  const double a2 = gamma * P * irho;
  const double Bp2 = Bt1 * Bt1 + Bt2 * Bt2;
  const double b2 = (Bn * Bn + Bp2) * irho;
  const double dab = a2 - b2;
  const double p4 = 4.0 * a2 * (Bp2 * irho);   // as in face_eig
  const double D = sqrt_nr(dab * dab + p4);
  const double cf2 = 0.5 * (a2 + b2 + D);
  double l_Bt1 = eb.Bt1, l_Bt2 = eb.Bt2, l_a2 = eb.a2, l_rho = eb.rho;
  double l_cf2 = 0.0, l_csl2 = 0.0, l_Bp2 = 0.0, l_b2 = 0.0, l_dab = 0.0, l_D = 0.0, l_irho = 0.0;
  double l_Bn = 0.0, l_P = 0.0;
  // alpha_f, alpha_s (non-degenerate branch, unclamped interior)
  if (D >= ph.eps_B * ph.eps_B) {
    const double iD = rcp_w(D);
    const double r = dab * iD;
    double cfa, csa;   // the forward's clamped alpha^2 (same arithmetic), for the interior test
    alpha_sq(dab, D, p4, cfa, csa);
    double l_r = 0.0;
    if (cfa > 0.0 && cfa < 1.0 && e.af > 0.0) l_r += eb.af * 0.25 * rcp_w(e.af);
    if (csa > 0.0 && csa < 1.0 && e.as > 0.0) l_r -= eb.as * 0.25 * rcp_w(e.as);
    l_dab += l_r * iD;
    l_D -= l_r * r * iD;
  }
  // beta
  if (Bp2 > ph.eps_B) {
    const double ib = rsq_nr(Bp2);
    l_Bt1 += eb.by * ib;
    l_Bt2 += eb.bz * ib;
    l_Bp2 -= 0.5 * ib * ib * ib * (eb.by * Bt1 + eb.bz * Bt2);
  }
  // csl = sqrt(csl2)
  if (e.csl > 0.0) l_csl2 += eb.csl * 0.5 * rcp_w(e.csl);
  // csl2 = a2 Bn^2 irho / cf2
  if (cf2 > 0.0) {
    const double icf2 = rcp_w(cf2);
    const double lN = l_csl2 * icf2;
    l_cf2 -= l_csl2 * (e.csl * e.csl) * icf2;
    l_a2 += lN * Bn * Bn * irho;
    l_Bn += lN * 2.0 * a2 * Bn * irho;
    l_irho += lN * a2 * Bn * Bn;
  }
  // cf = sqrt(cf2)
  if (e.cf > 0.0) l_cf2 += eb.cf * 0.5 * rcp_w(e.cf);
  // cf2 = (a2 + b2 + D)/2
  l_a2 += 0.5 * l_cf2; l_b2 += 0.5 * l_cf2; l_D += 0.5 * l_cf2;
  // D = sqrt(dab^2 + 4 a2 Bp2 irho)
  if (D > 0.0) {
    const double lQ = l_D * 0.5 * rcp_w(D);
    l_dab += 2.0 * dab * lQ;
    l_a2 += 4.0 * Bp2 * irho * lQ;
    l_Bp2 += 4.0 * a2 * irho * lQ;
    l_irho += 4.0 * a2 * Bp2 * lQ;
  }
  // dab = a2 - b2
  l_a2 += l_dab; l_b2 -= l_dab;
  // b2 = (Bn^2 + Bp2) irho
  l_Bn += 2.0 * Bn * irho * l_b2; l_Bp2 += irho * l_b2; l_irho += (Bn * Bn + Bp2) * l_b2;
  // Bp2
  l_Bt1 += 2.0 * Bt1 * l_Bp2; l_Bt2 += 2.0 * Bt2 * l_Bp2;
  // a2 = gamma P irho
  l_P += gamma * irho * l_a2; l_irho += gamma * P * l_a2;
  // irho = 1/rho
  l_rho -= irho * irho * l_irho;
  out[0] = l_rho; out[1] = eb.vn; out[2] = eb.vt1; out[3] = eb.vt2;
  out[4] = l_Bn; out[5] = l_Bt1; out[6] = l_Bt2; out[7] = l_P;
}

// ---------------------------------------------------------------------------
// phi_N = omega_0 X/3 + (omega_2 - 1/2) Y/6 (X = a-2b+c, Y = b-2c+d; Sect. 2.2) and its
// gradient with respect to its four arguments.  With omega = alpha/sum, g = X/3, h = Y/6
// and W3 = g omega_0 + h omega_2, dphi/dalpha_k = (G_k - W3)/sum, G = (g, 0, h).
// ---------------------------------------------------------------------------
// Jiang-Shu weights, WENO-Z weights, and the Jiang-Shu weights of the smallest eps.
enum AdjWeights { ADJ_JS, ADJ_Z, ADJ_JS_TINY };
// The scale of the left rows, and so of phi's arguments and value.  ADJ_JS forms products of
// four s_k (one reciprocal for value and gradient), whose range the scale centres: it takes
// eps from 5e-51 and arguments up to 5e50.  ADJ_JS_TINY forms products of three, unscaled, with
// a reciprocal more, and takes eps down to 1e-102.  Below 1e-50 the host picks it.
template <int W> constexpr double AdjScale = W == ADJ_JS ? 0x1p-43 : 1.0;

template <int W>
__host__ __device__ __forceinline__ void phiN_val_grad(double a, double b, double c, double d, double eps,
                                                       double epsZ, bool lit, double& val, double gr[4]) {
  const double t0 = a - b, t1 = a - 3.0 * b;
  const double t2 = b - c, t3 = b + c;
  const double t4 = c - d, t5 = 3.0 * c - d;
  const double X = t0 - t2, Y = t2 - t4;   // a - 2b + c, b - 2c + d
  if constexpr (W == ADJ_JS) {
    // As phiN, with s_k = (eps + IS_k)/3 (eps at the scale of the arguments), S_k = s_k^2, c = 3 p01 - m and Q = 3 p01 + m:
    // phi = (4 p12 X + c Y)/(12 Q), and with A = Y/12 - phi, B = Y/12 + phi,
    // C = X/3 - Y/12 - phi
    //   dphi/ds_0 = (6 s_0/Q)(S_1 A - 2 S_2 B),  dphi/ds_1 = (2 s_1/Q)(S_2 C + 3 S_0 A),
    //   dphi/ds_2 = (2 s_2/Q)(S_1 C - 6 S_0 B).
    (void)epsZ;
    (void)lit;
    const double e3 = eps * (AdjScale<W> * AdjScale<W> / 3.0);
    const double T0 = (13.0 / 3.0) * t0, T2 = (13.0 / 3.0) * t2, T4 = (13.0 / 3.0) * t4;
    const double s0 = fma(T0, t0, fma(t1, t1, e3));
    const double s1 = fma(T2, t2, fma(t3, t3, e3));
    const double s2 = fma(T4, t4, fma(t5, t5, e3));
    const double S0 = s0 * s0, S1 = s1 * s1, S2 = s2 * s2;
    const double p12 = S1 * S2, p02 = S0 * S2, p01 = S0 * S1;
    const double m = fma(6.0, p02, p12);
    const double rq = rcp_w(fma(3.0, p01, m));
    const double cX = p12 * (rq * (1.0 / 3.0)), cY = fma(3.0, p01, -m) * (rq * (1.0 / 12.0));
    val = fma(cX, X, cY * Y);
    const double y = Y * (1.0 / 12.0);
    const double A = y - val, B = y + val, C = fma(X, 1.0 / 3.0, -B);
    const double r4 = 4.0 * rq;
    // twice dphi/ds_k
    const double l0 = 3.0 * (s0 * r4) * fma(-2.0, S2 * B, S1 * A);
    const double l1 = (s1 * r4) * fma(3.0, S0 * A, S2 * C);
    const double l2 = (s2 * r4) * fma(-6.0, S0 * B, S1 * C);
    // ds_k by its two squares: 2 (13/3) t dt and 2 t' dt'
    const double u0 = l0 * T0, v0 = l0 * t1, u1 = l1 * T2, v1 = l1 * t3, u2 = l2 * T4, v2 = l2 * t5;
    gr[0] = cX + (u0 + v0);
    gr[1] = fma(-2.0, cX, cY) - u0 - 3.0 * v0 + (u1 + v1);
    gr[2] = fma(-2.0, cY, cX) - u1 + v1 + (u2 + 3.0 * v2);
    gr[3] = cY - (u2 + v2);
    return;
  }
  const double g = X * (1.0 / 3.0), h = Y * (1.0 / 6.0);
  double w0, w2, l0, l1, l2;   // normalised weights 0, 2 and dphi/dIS_k
  if constexpr (W == ADJ_JS_TINY) {
    // with s_k = eps + IS_k, alpha_k = d_k/s_k^2: dphi/ds_0 = (2 omega_0/s_0)(W - g),
    // dphi/ds_1 = (2 omega_1/s_1) W, dphi/ds_2 = (2 omega_2/s_2)(W - h)
    (void)epsZ;
    (void)lit;
    const double s0 = eps + 13.0 * t0 * t0 + 3.0 * t1 * t1;
    const double s1 = eps + 13.0 * t2 * t2 + 3.0 * t3 * t3;
    const double s2 = eps + 13.0 * t4 * t4 + 3.0 * t5 * t5;
    const double s12 = s1 * s2, r = rcp_w(s0 * s12);
    const double i0 = s12 * r, i1 = s0 * s2 * r, i2 = s0 * s1 * r;   // 1/s_k
    const double al0 = i0 * i0, al1 = 6.0 * i1 * i1, al2 = 3.0 * i2 * i2;
    const double isum = rcp_w(al0 + al1 + al2);
    w0 = al0 * isum;
    const double w1 = al1 * isum;
    w2 = al2 * isum;
    const double W3 = g * w0 + h * w2;
    l0 = 2.0 * w0 * i0 * (W3 - g);
    l1 = 2.0 * w1 * i1 * W3;
    l2 = 2.0 * w2 * i2 * (W3 - h);
  } else {
    // WENO-Z: alpha_k = d_k (1 + u_k), q_k = 1/(eps_Z + IS_k), r_k = tau5 q_k, tau5 = |IS_0 - IS_2|,
    // u_k = r_k^2, or u_k = tau5 q_k^2 = r_k q_k as printed (`lit`).  Both give
    // du_k/dIS_k = -2 u_k q_k; du_k/dtau5 is 2 r_k q_k, or q_k^2 as printed.
    (void)eps;
    const double IS0 = 13.0 * t0 * t0 + 3.0 * t1 * t1;
    const double IS1 = 13.0 * t2 * t2 + 3.0 * t3 * t3;
    const double IS2 = 13.0 * t4 * t4 + 3.0 * t5 * t5;
    const double dIS = IS0 - IS2, tau = fabs(dIS);
    const double q0 = rcp_w(epsZ + IS0), q1 = rcp_w(epsZ + IS1), q2 = rcp_w(epsZ + IS2);
    const double r0 = tau * q0, r1 = tau * q1, r2 = tau * q2;
    const double s0 = lit ? q0 : r0, s1 = lit ? q1 : r1, s2 = lit ? q2 : r2;
    const double u0 = r0 * s0, u1 = r1 * s1, u2 = r2 * s2;
    const double al0 = 1.0 + u0, al1 = 6.0 * (1.0 + u1), al2 = 3.0 * (1.0 + u2);
    const double isum = rcp_w(al0 + al1 + al2);
    w0 = al0 * isum;
    w2 = al2 * isum;
    const double W3 = g * w0 + h * w2;
    // dphi/du_k = (G_k - W3)/sum(alpha) * d_k, G = (g, 0, h)
    const double M0 = (g - W3) * isum, M1 = -W3 * isum * 6.0, M2 = (h - W3) * isum * 3.0;
    const double ct = lit ? 1.0 : 2.0;   // du_k/dtau5 = ct s_k q_k
    const double ltau = ct * (M0 * s0 * q0 + M1 * s1 * q1 + M2 * s2 * q2);   // dphi/dtau5
    const double sg = dIS > 0.0 ? 1.0 : (dIS < 0.0 ? -1.0 : 0.0);
    l0 = -2.0 * M0 * u0 * q0 + sg * ltau;
    l1 = -2.0 * M1 * u1 * q1;
    l2 = -2.0 * M2 * u2 * q2 - sg * ltau;
  }
  const double cX = w0 * (1.0 / 3.0), cY = (w2 - 0.5) * (1.0 / 6.0);
  val = cX * X + cY * Y;
  // dIS_0/da = 26 t0 + 6 t1, dIS_0/db = -26 t0 - 18 t1
  // dIS_1/db = 26 t2 + 6 t3, dIS_1/dc = -26 t2 + 6 t3
  // dIS_2/dc = 26 t4 + 18 t5, dIS_2/dd = -26 t4 - 6 t5
  gr[0] = cX + l0 * (26.0 * t0 + 6.0 * t1);
  gr[1] = -2.0 * cX + cY + l0 * (-26.0 * t0 - 18.0 * t1) + l1 * (26.0 * t2 + 6.0 * t3);
  gr[2] = cX - 2.0 * cY + l1 * (-26.0 * t2 + 6.0 * t3) + l2 * (26.0 * t4 + 18.0 * t5);
  gr[3] = cY + l2 * (-26.0 * t4 - 6.0 * t5);
}

// ---------------------------------------------------------------------------
// eigen pairs: forward and reverse in a single pass
// ---------------------------------------------------------------------------
// A pair has the left rows S + A (upper) and S - A (lower) with the
// Lax-Friedrichs speeds alu, all; S is nonzero on the components in SM, A on
// A0 .. A0+NA-1 (TWO = false: the single row S).  Split values as in
// face_corr; f = phi(v7, v6, v5, v4) - phi(v0, v1, v2, v3) per row.  The
// cotangents lfu, lfl of the two f only involve the right eigenvectors, so they
// are known before the pass, which computes f (needed for the right-vector
// cotangents) and the cotangents of S, A, the two speeds and the interface
// differences.
struct PairRows {
  double S[7], A[4];
  double alu, all;   // Lax-Friedrichs speeds of the upper / lower row
  double lfu, lfl;   // cotangents of f_upper, f_lower
};
struct PairCot {
  double fu = 0.0, fl = 0.0;                       // forward values
  double lS[7] = {0, 0, 0, 0, 0, 0, 0}, lA[4] = {0, 0, 0, 0};
  double lalu = 0.0, lall = 0.0;                   // cotangents of the speeds
};

template <int A0, int NA, bool TWO, int SM>
struct PairShape {
  // projections of the rows at one interface: d[0..6] Delta F, d[7..13] Delta q
  __host__ __device__ static __forceinline__ void proj(const PairRows& r, const double d[14], double& uF, double& uq,
                                                       double& lF, double& lq) {
    double sF = 0.0, sq = 0.0, aF = 0.0, aq = 0.0;
#pragma unroll
    for (int j = 0; j < 7; ++j)
      if (SM & (1 << j)) { sF += r.S[j] * d[j]; sq += r.S[j] * d[7 + j]; }
#pragma unroll
    for (int j = 0; j < NA; ++j) { aF += r.A[j] * d[A0 + j]; aq += r.A[j] * d[7 + A0 + j]; }
    uF = sF + aF; uq = sq + aq; lF = sF - aF; lq = sq - aq;
  }
  // cotangents of S, A from one interface (sFb = lP_u + lP_l, aFb = lP_u - lP_l, ...)
  __host__ __device__ static __forceinline__ void rowcot(const double d[14], double sFb, double aFb, double sqb,
                                                         double aqb, PairCot& c) {
#pragma unroll
    for (int j = 0; j < 7; ++j)
      if (SM & (1 << j)) c.lS[j] += sFb * d[j] + sqb * d[7 + j];
#pragma unroll
    for (int j = 0; j < NA; ++j) c.lA[j] += aFb * d[A0 + j] + aqb * d[7 + A0 + j];
  }
  // cotangent of the interface differences: lD += (S + A) lP_u + (S - A) lP_l (F and q parts)
  __host__ __device__ static __forceinline__ void difcot(const PairRows& r, double sFb, double aFb, double sqb,
                                                         double aqb, double lD[14]) {
#pragma unroll
    for (int j = 0; j < 7; ++j)
      if (SM & (1 << j)) { lD[j] += r.S[j] * sFb; lD[7 + j] += r.S[j] * sqb; }
#pragma unroll
    for (int j = 0; j < NA; ++j) { lD[A0 + j] += r.A[j] * aFb; lD[7 + A0 + j] += r.A[j] * aqb; }
  }
};

// Split values, phi and its gradient for one row: from the projections uF, uq
// (interfaces 0..4) to f, the cotangents g[0..3] of Delta F^+ and g[4..7] of
// Delta F^- (of uF at interface k: g[k] + g[3 + k], of uq al times their
// difference, where they exist) and the cotangent of alpha.
template <int W>
__host__ __device__ __forceinline__ void row_split_grad(const double uF[5], const double uq[5], double al, double lf,
                                                        double eps, double epsZ, bool lit, double& f, double g[8],
                                                        double& lal) {
  constexpr double unscale = 1.0 / AdjScale<W>;   // of the projections, which the scaled rows formed
  lf *= unscale;
  double g4[4], pa, pb;
  phiN_val_grad<W>(uF[4] - al * uq[4], uF[3] - al * uq[3], uF[2] - al * uq[2], uF[1] - al * uq[1], eps, epsZ, lit,
                    pa, g4);
  g[7] = g4[0] * lf; g[6] = g4[1] * lf; g[5] = g4[2] * lf; g[4] = g4[3] * lf;
  sched_fence();
  phiN_val_grad<W>(uF[0] + al * uq[0], uF[1] + al * uq[1], uF[2] + al * uq[2], uF[3] + al * uq[3], eps, epsZ, lit,
                    pb, g4);
  g[0] = -g4[0] * lf; g[1] = -g4[1] * lf; g[2] = -g4[2] * lf; g[3] = -g4[3] * lf;
  f = (pa - pb) * unscale;
#pragma unroll
  for (int k = 0; k < 5; ++k)
    lal += uq[k] * (k == 0 ? g[0] : (k == 4 ? -g[7] : g[k] - g[3 + k]));
  sched_fence();
}

struct PairGrad {
  double u[8], l[8];   // row_split_grad's g of the upper and lower row
};
// Cotangents of the projections at interface k, summed and subtracted over the two
// rows: sF, aF of S.dF and A.dF, sq, aq of S.dq and A.dq.
template <bool TWO>
__host__ __device__ __forceinline__ void pair_sums(const PairRows& r, const PairGrad& g, int k, double& sF, double& aF,
                                                   double& sq, double& aq) {
  auto lP = [](const double* v, int i) { return i == 0 ? v[0] : (i == 4 ? v[7] : v[i] + v[3 + i]); };
  auto lQ = [](const double* v, int i) { return i == 0 ? v[0] : (i == 4 ? -v[7] : v[i] - v[3 + i]); };
  const double Pu = lP(g.u, k), Qu = r.alu * lQ(g.u, k);
  if (TWO) {
    const double Pl = lP(g.l, k), Ql = r.all * lQ(g.l, k);
    sF = Pu + Pl; aF = Pu - Pl; sq = Qu + Ql; aq = Qu - Ql;
  } else {
    sF = aF = Pu; sq = aq = Qu;
  }
}
// Forward and reverse of one pair up to the cotangents of its rows.  row(k) points
// at the differences of interface k, PITCH values apart; they are read again for
// the row cotangents rather than held.
template <class PA, bool TWO, int W, int PITCH, class ROW>
__host__ __device__ __forceinline__ void pair_rev(const PairRows& r, ROW row, double eps, double epsZ, bool lit,
                                                  PairCot& c, PairGrad& g) {
  {
    double uF[5], uq[5], lF[5], lq[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const double* p = row(k);
      double d[14];
#pragma unroll
      for (int j = 0; j < 14; ++j) d[j] = p[j * PITCH];
      PA::proj(r, d, uF[k], uq[k], lF[k], lq[k]);
      sched_fence();
    }
    row_split_grad<W>(uF, uq, r.alu, r.lfu, eps, epsZ, lit, c.fu, g.u, c.lalu);
    if (TWO) row_split_grad<W>(lF, lq, r.all, r.lfl, eps, epsZ, lit, c.fl, g.l, c.lall);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    pin(g.u[j]);
    if (TWO) pin(g.l[j]);
  }
  reload_fence();
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const double* p = row(k);
    double d[14], sF, aF, sq, aq;
#pragma unroll
    for (int j = 0; j < 14; ++j) d[j] = p[j * PITCH];
    pair_sums<TWO>(r, g, k, sF, aF, sq, aq);
    PA::rowcot(d, sF, aF, sq, aq, c);
    sched_fence();
  }
#pragma unroll
  for (int j = 0; j < 7; ++j) pin(c.lS[j]);
#pragma unroll
  for (int j = 0; j < 4; ++j) pin(c.lA[j]);
}

// Adds the pair's cotangents of the differences of interface k to lD.
template <class PA, bool TWO>
__host__ __device__ __forceinline__ void pair_difcot(const PairRows& r, const PairGrad& g, int k, double lD[14]) {
  double sF, aF, sq, aq;
  pair_sums<TWO>(r, g, k, sF, aF, sq, aq);
  PA::difcot(r, sF, aF, sq, aq, lD);
}

// ---------------------------------------------------------------------------
// rows and right-vector cotangents of each pair (Appendix A), with the
// reverse of the row construction into the eigen-scalar cotangents eb
// ---------------------------------------------------------------------------
// fast pair (m = 1, 7) and slow pair (m = 3, 5).  With (x, y, c, o, G, z) = (alpha_f,
// alpha_s, c_f, c_s, Gamma_f, +1) for the fast and (alpha_s, alpha_f, c_s, c_f, Gamma_s, -1)
// for the slow pair (c_s the slow speed here), W = omg (-v2/2, vn, vt1, vt2, Bt1, Bt2, -1):
//   S = q (x W + z sra y beta),  A = q (G, -x c, z o y s by, z o y s bz),  q = 1/(4 a^2)
// (times SC, the AdjScale of the rows, here and in the other pairs),
// and the right columns add to corr, with sp = fu + fl, sm = fu - fl,
//   x sp;  x vn sp - x c sm;  x vt1 sp + z o y s by sm;  x vt2 sp + z o y s bz sm;
//   z cs y isr by sp;  z cs y isr bz sp;  x (v2/2 + c^2 - g2 a^2) sp - G sm.
template <bool FAST> struct Magneto {
  double x, y, c, o, G, bv, zo, zs;   // zo = z o y s, zs = z y
  __host__ __device__ __forceinline__ explicit Magneto(const FaceEig& e) {
    bv = e.by * e.vt1 + e.bz * e.vt2;
    if (FAST) { x = e.af; y = e.as; c = e.cf; o = e.csl; }
    else      { x = e.as; y = e.af; c = e.csl; o = e.cf; }
    zs = FAST ? y : -y;
    zo = zs * o * e.s;
    G = x * c * e.vn - zo * bv;
  }
};
template <bool FAST, int W, class ALF>
__host__ __device__ __forceinline__ void magneto_rows(const FaceEig& e, ALF alf, const double lam[7], PairRows& r) {
  const Magneto<FAST> m(e);
  const double q = e.qa2 * AdjScale<W>, qw = q * e.omg * m.x, qb = q * (e.sr * e.cs) * m.zs, hv2 = 0.5 * e.v2;
  r.S[0] = -qw * hv2; r.S[1] = qw * e.vn; r.S[2] = qw * e.vt1; r.S[3] = qw * e.vt2;
  r.S[4] = qw * e.Bt1 + qb * e.by; r.S[5] = qw * e.Bt2 + qb * e.bz; r.S[6] = -qw;
  r.A[0] = q * m.G; r.A[1] = -q * (m.x * m.c); r.A[2] = q * m.zo * e.by; r.A[3] = q * m.zo * e.bz;
  const double lb = e.by * lam[2] + e.bz * lam[3], lB = e.by * lam[4] + e.bz * lam[5];
  const double Rs6 = hv2 + m.c * m.c - e.g2 * (e.cs * e.cs);
  const double lsp = m.x * (lam[0] + e.vn * lam[1] + e.vt1 * lam[2] + e.vt2 * lam[3] + Rs6 * lam[6]) +
                     e.cs * e.isr * m.zs * lB;
  const double lsm = -m.x * m.c * lam[1] + m.zo * lb - m.G * lam[6];
  r.lfu = lsp + lsm;
  r.lfl = lsp - lsm;
  r.alu = alf(FAST ? 0 : 2);
  r.all = alf(FAST ? 6 : 4);
}
template <bool FAST, int W>
__host__ __device__ __forceinline__ void magneto_post(const FaceEig& e, const double lam[7], const PairCot& p,
                                                      EigCot& eb) {
  const Magneto<FAST> m(e);
  constexpr double SC = AdjScale<W>;
  const double q = e.qa2 * SC, sra = e.sr * e.cs, z = FAST ? 1.0 : -1.0, hv2 = 0.5 * e.v2;
  const double sp = p.fu + p.fl, sm = p.fu - p.fl;
  const double lb = e.by * lam[2] + e.bz * lam[3], lB = e.by * lam[4] + e.bz * lam[5];
  // right columns
  double lx = sp * (lam[0] + e.vn * lam[1] + e.vt1 * lam[2] + e.vt2 * lam[3] +
                    (hv2 + m.c * m.c - e.g2 * (e.cs * e.cs)) * lam[6]) - sm * m.c * lam[1];
  const double xs = m.x * sp;
  eb.vn += xs * lam[1]; eb.vt1 += xs * lam[2]; eb.vt2 += xs * lam[3];
  eb.a2 -= e.g2 * xs * lam[6];
  double lv2 = 0.5 * xs * lam[6];
  double lc = 2.0 * m.c * xs * lam[6] - m.x * sm * lam[1];
  double lzo = sm * lb;                          // cotangent of zo
  double lzs = e.cs * e.isr * sp * lB;           // of zs
  eb.by += sm * m.zo * lam[2] + sp * e.cs * e.isr * m.zs * lam[4];
  eb.bz += sm * m.zo * lam[3] + sp * e.cs * e.isr * m.zs * lam[5];
  double lcs = e.isr * m.zs * sp * lB;
  eb.add_isr(e, e.cs * m.zs * sp * lB);
  double lG = -sm * lam[6];
  // rows
  const double LW = e.omg * (e.vn * p.lS[1] + e.vt1 * p.lS[2] + e.vt2 * p.lS[3] + e.Bt1 * p.lS[4] + e.Bt2 * p.lS[5] -
                             hv2 * p.lS[0] - p.lS[6]);
  const double LB = e.by * p.lS[4] + e.bz * p.lS[5], LC = e.by * p.lA[2] + e.bz * p.lA[3];
  eb.add_q(e, SC * (m.x * LW + sra * m.zs * LB + m.G * p.lA[0] - m.x * m.c * p.lA[1] + m.zo * LC));
  const double qw = q * e.omg * m.x;
  lx += q * LW - q * m.c * p.lA[1];
  lv2 -= 0.5 * qw * p.lS[0];
  eb.vn += qw * p.lS[1]; eb.vt1 += qw * p.lS[2]; eb.vt2 += qw * p.lS[3];
  eb.Bt1 += qw * p.lS[4]; eb.Bt2 += qw * p.lS[5];
  lzs += q * sra * LB;
  eb.by += q * (sra * m.zs * p.lS[4] + m.zo * p.lA[2]);
  eb.bz += q * (sra * m.zs * p.lS[5] + m.zo * p.lA[3]);
  eb.add_sr(e, q * e.cs * m.zs * LB);
  lcs += q * e.sr * m.zs * LB;
  lc -= q * m.x * p.lA[1];
  lzo += q * LC;
  lG += q * p.lA[0];
  // G = x c vn - zo bv
  lx += lG * m.c * e.vn;
  lc += lG * m.x * e.vn;
  eb.vn += lG * m.x * m.c;
  lzo -= lG * m.bv;
  eb.add_bv(e, -lG * m.zo);
  // zo = zs o s, zs = z y
  lzs += lzo * m.o * e.s;
  const double lo = lzo * m.zs * e.s, ly = z * lzs;
  if (FAST) { eb.af += lx; eb.as += ly; eb.cf += lc; eb.csl += lo; }
  else      { eb.as += lx; eb.af += ly; eb.csl += lc; eb.cf += lo; }
  eb.add_cs(e, lcs);
  eb.add_v2(e, lv2);
}

// Alfven pair (m = 2, 6): S = (Ga/4, 0, -bz s/4, by s/4, 0, 0, 0), A = (-sr bz/4, sr by/4) on components 4, 5
template <int W, class ALF>
__host__ __device__ __forceinline__ void alfven_rows(const FaceEig& e, ALF alf, const double lam[7], PairRows& r) {
  constexpr double Q = 0.25 * AdjScale<W>;
  const double s = e.s, Ga = s * (e.bz * e.vt1 - e.by * e.vt2);
  r.S[0] = Q * Ga; r.S[1] = 0.0; r.S[2] = -Q * e.bz * s; r.S[3] = Q * e.by * s;
  r.S[4] = 0.0; r.S[5] = 0.0; r.S[6] = 0.0;
  r.A[0] = -Q * e.sr * e.bz; r.A[1] = Q * e.sr * e.by; r.A[2] = 0.0; r.A[3] = 0.0;
  // corr += (0, 0, -bz s sp, by s sp, -bz isr sm, by isr sm, -Ga sp)
  const double lsp = s * (e.by * lam[3] - e.bz * lam[2]) - Ga * lam[6];
  const double lsm = e.isr * (e.by * lam[5] - e.bz * lam[4]);
  r.lfu = lsp + lsm;
  r.lfl = lsp - lsm;
  r.alu = alf(1);
  r.all = alf(5);
}
template <int W>
__host__ __device__ __forceinline__ void alfven_post(const FaceEig& e, const double lam[7], const PairCot& c,
                                                     EigCot& eb) {
  constexpr double Q = 0.25 * AdjScale<W>;
  const double s = e.s;
  const double sp = c.fu + c.fl, sm = c.fu - c.fl;
  eb.bz -= s * (sp * lam[2] + Q * c.lS[2]) + e.isr * sm * lam[4] + Q * e.sr * c.lA[0];
  eb.by += s * (sp * lam[3] + Q * c.lS[3]) + e.isr * sm * lam[5] + Q * e.sr * c.lA[1];
  eb.add_isr(e, sm * (e.by * lam[5] - e.bz * lam[4]));
  eb.add_sr(e, Q * (e.by * c.lA[1] - e.bz * c.lA[0]));
  const double lGa = s * (Q * c.lS[0] - sp * lam[6]);   // Ga = s (bz vt1 - by vt2)
  eb.bz += lGa * e.vt1; eb.vt1 += lGa * e.bz; eb.by -= lGa * e.vt2; eb.vt2 -= lGa * e.by;
}

// entropy (m = 4): the single row L/2 = (1/2 - tau v^2/4, tau vn/2, tau vt1/2, tau vt2/2, tau Bt1/2, tau Bt2/2, -tau/2),
// tau = (gamma - 1)/a^2 = -4 omg q
template <int W, class ALF>
__host__ __device__ __forceinline__ void entropy_rows(const FaceEig& e, ALF alf, const double lam[7], PairRows& r) {
  constexpr double SC = AdjScale<W>;
  const double ht = -2.0 * SC * e.omg * e.qa2;
  r.S[0] = 0.5 * SC - 0.5 * ht * e.v2; r.S[1] = ht * e.vn; r.S[2] = ht * e.vt1; r.S[3] = ht * e.vt2;
  r.S[4] = ht * e.Bt1; r.S[5] = ht * e.Bt2; r.S[6] = -ht;
  r.A[0] = r.A[1] = r.A[2] = r.A[3] = 0.0;
  // corr += (f4, vn f4, vt1 f4, vt2 f4, 0, 0, v2/2 f4)
  r.lfu = lam[0] + e.vn * lam[1] + e.vt1 * lam[2] + e.vt2 * lam[3] + 0.5 * e.v2 * lam[6];
  r.lfl = 0.0;
  r.alu = alf(3);
  r.all = r.alu;
}
template <int W>
__host__ __device__ __forceinline__ void entropy_post(const FaceEig& e, const double lam[7], const PairCot& c,
                                                      EigCot& eb) {
  constexpr double SC = AdjScale<W>;
  const double ht = -2.0 * SC * e.omg * e.qa2;
  const double f4 = c.fu;
  eb.vn += f4 * lam[1] + ht * c.lS[1];
  eb.vt1 += f4 * lam[2] + ht * c.lS[2];
  eb.vt2 += f4 * lam[3] + ht * c.lS[3];
  eb.Bt1 += ht * c.lS[4];
  eb.Bt2 += ht * c.lS[5];
  eb.add_v2(e, 0.5 * (f4 * lam[6] - ht * c.lS[0]));
  const double lht = -0.5 * e.v2 * c.lS[0] + e.vn * c.lS[1] + e.vt1 * c.lS[2] + e.vt2 * c.lS[3] +
                     e.Bt1 * c.lS[4] + e.Bt2 * c.lS[5] - c.lS[6];
  eb.add_q(e, -2.0 * SC * e.omg * lht);
}

using MagnetoShape = PairShape<0, 4, true, 127>;
using AlfvenShape = PairShape<4, 2, true, 13>;
using EntropyShape = PairShape<0, 0, false, 127>;

// New names for the eigen scalars that the pairs use: the compiler may not keep
// products of them from one pair, or from a pair's rows, for the next.
__host__ __device__ __forceinline__ void renew(FaceEig& e, double lam[7]) {
  pin(e.vn); pin(e.vt1); pin(e.vt2); pin(e.Bt1); pin(e.Bt2); pin(e.by); pin(e.bz); pin(e.s); pin(e.af); pin(e.as);
  pin(e.cf); pin(e.csl); pin(e.cs); pin(e.sr); pin(e.isr); pin(e.qa2);
#pragma unroll
  for (int j = 0; j < 7; ++j) pin(lam[j]);
  e.v2 = e.vn * e.vn + e.vt1 * e.vt1 + e.vt2 * e.vt2;
}

// Reverse of face_corr (FP64) at one face: given the eigen scalars e, the
// Lax-Friedrichs speeds alf(m), the differences (row, PITCH) and the cotangent lam
// of corr, forms the cotangents of the eigen scalars (eb), of the LF speeds
// (lal[7]) and, via emit (five calls per pair), of the interface differences, where
// the central flux (F_L + F_R)/2 + (Delta F_{i-1/2} - Delta F_{i+3/2})/12 adds its own
// (lam/12 on differences 1 and 3: with them the emission, not in additions apart).  The
// face-state cotangents follow from face_eig_vjp(eb).  One pair at a time: two at
// once share the reads of the differences but need twice the registers, and two
// waves per SIMD are worth more than those reads.
template <int W, int PITCH, class ALF, class ROW, class EMIT>
__host__ __device__ __forceinline__ void face_corr_vjp(FaceEig& e, ALF alf, double lam[7], ROW row,
                                                       const Phys& ph, EigCot& eb, double lal[7], EMIT emit) {
  const double eps = ph.eps, epsZ = ph.eps_Z;
  const bool lit = ph.weno_z == 2;
  eb.zero();
  {
    // the entropy row's gradient waits for the Alfven pair's, so that one round of
    // additions carries both (its row is formed again)
    PairGrad gn, ga;
    {
      renew(e, lam);
      PairRows r;
      entropy_rows<W>(e, alf, lam, r);
      PairCot c;
      pair_rev<EntropyShape, false, W, PITCH>(r, row, eps, epsZ, lit, c, gn);
      renew(e, lam);
      entropy_post<W>(e, lam, c, eb);
      lal[3] = c.lalu;
      eb.pin_all();
      pin(lal[3]);
      sched_fence();
    }
    renew(e, lam);
    PairRows ra, rn;
    alfven_rows<W>(e, alf, lam, ra);
    PairCot c;
    pair_rev<AlfvenShape, true, W, PITCH>(ra, row, eps, epsZ, lit, c, ga);
    renew(e, lam);
    alfven_post<W>(e, lam, c, eb);
    lal[1] = c.lalu; lal[5] = c.lall;
    eb.pin_all();
    pin(lal[1]); pin(lal[5]);
    sched_fence();
    renew(e, lam);
    entropy_rows<W>(e, alf, lam, rn);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      double lD[14] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
      if (k == 1 || k == 3) {   // the central term's part
#pragma unroll
        for (int j = 0; j < 7; ++j) lD[j] = (k == 1 ? 1.0 / 12.0 : -1.0 / 12.0) * lam[j];
      }
      pair_difcot<EntropyShape, false>(rn, gn, k, lD);
      pair_difcot<AlfvenShape, true>(ra, ga, k, lD);
      emit(k, lD);
    }
  }
  sched_fence();
  auto magneto = [&](auto fast) {
    constexpr bool FAST = decltype(fast)::value;
    renew(e, lam);
    PairRows r;
    magneto_rows<FAST, W>(e, alf, lam, r);
    PairCot c;
    PairGrad g;
    pair_rev<MagnetoShape, true, W, PITCH>(r, row, eps, epsZ, lit, c, g);
    renew(e, lam);
    magneto_post<FAST, W>(e, lam, c, eb);
    double& lu = lal[FAST ? 0 : 2];
    double& ll = lal[FAST ? 6 : 4];
    lu = c.lalu; ll = c.lall;
    eb.pin_all();
    pin(lu); pin(ll);
    sched_fence();
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      double lD[14] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
      pair_difcot<MagnetoShape, true>(r, g, k, lD);
      emit(k, lD);
    }
    sched_fence();
  };
  magneto(std::false_type{});
  magneto(std::true_type{});
}

// ---------------------------------------------------------------------------
// zone prologue: cotangents of (q, F, primitives, speeds) -> zone inputs
// ---------------------------------------------------------------------------
// Inputs in the sweep frame: u = (rho, m_n, m_t1, m_t2, E, B_n, B_t1, B_t2).
// lz[Z_NVAR] are the cotangents of the prologue outputs; out[8] += d/du.
__host__ __device__ __forceinline__ void zone_prologue_vjp(const double u[8], double gamma, const double lz[Z_NVAR],
                                                  double out[8]) {
  const double rho = u[0], mn = u[1], mt1 = u[2], mt2 = u[3], E = u[4], Bn = u[5], Bt1 = u[6], Bt2 = u[7];
  const double irho = rcp_w(rho);
  const double vn = mn * irho, vt1 = mt1 * irho, vt2 = mt2 * irho;
  const double Bp2 = Bt1 * Bt1 + Bt2 * Bt2;
  const double B2 = Bn * Bn + Bp2;
  const double P = (gamma - 1.0) * (E - 0.5 * ((mn * vn + mt1 * vt1 + mt2 * vt2) + B2));
  const double Pstar = P + 0.5 * B2;
  const double vB = vn * Bn + vt1 * Bt1 + vt2 * Bt2;
  const double a2 = gamma * P * irho, b2 = B2 * irho, bn2 = Bn * Bn * irho;
  const double dab = a2 - b2;
  const double D = sqrt_nr(dab * dab + 4.0 * a2 * (Bp2 * irho));
  const double cf2 = 0.5 * (a2 + b2 + D);
  const double icf2 = cf2 > 0.0 ? rcp_w(cf2) : 0.0;
  const double cs2 = a2 * bn2 * icf2;
  const double cf = sqrt_nr(cf2), cA = sqrt_nr(bn2), cs = sqrt_nr(cs2);
  double l_rho = lz[Z_RHO], l_mn = lz[Z_MN], l_mt1 = lz[Z_MT1], l_mt2 = lz[Z_MT2];
  double l_Bt1 = lz[Z_BT1], l_Bt2 = lz[Z_BT2], l_E = lz[Z_E];
  double l_vn = lz[Z_VN], l_vt1 = lz[Z_VT1], l_vt2 = lz[Z_VT2], l_Bn = lz[Z_BN], l_P = lz[Z_P];
  double l_cf2 = 0.0, l_cs2 = 0.0, l_bn2 = 0.0, l_a2 = 0.0, l_b2 = 0.0, l_D = 0.0, l_dab = 0.0;
  double l_irho = 0.0, l_Bp2 = 0.0, l_B2 = 0.0, l_Pstar = 0.0, l_vB = 0.0;
  // speeds
  if (cf > 0.0) l_cf2 += lz[Z_CF] * 0.5 * rcp_w(cf);
  if (cA > 0.0) l_bn2 += lz[Z_CA] * 0.5 * rcp_w(cA);
  if (cs > 0.0) l_cs2 += lz[Z_CS] * 0.5 * rcp_w(cs);
  if (cf2 > 0.0) {
    l_a2 += l_cs2 * bn2 * icf2;
    l_bn2 += l_cs2 * a2 * icf2;
    l_cf2 -= l_cs2 * cs2 * icf2;
  }
  l_a2 += 0.5 * l_cf2; l_b2 += 0.5 * l_cf2; l_D += 0.5 * l_cf2;
  if (D > 0.0) {
    const double lQ = l_D * 0.5 * rcp_w(D);
    l_dab += 2.0 * dab * lQ;
    l_a2 += 4.0 * Bp2 * irho * lQ;
    l_Bp2 += 4.0 * a2 * irho * lQ;
    l_irho += 4.0 * a2 * Bp2 * lQ;
  }
  l_a2 += l_dab; l_b2 -= l_dab;
  l_Bn += 2.0 * Bn * irho * l_bn2; l_irho += Bn * Bn * l_bn2;
  l_B2 += irho * l_b2; l_irho += B2 * l_b2;
  l_P += gamma * irho * l_a2; l_irho += gamma * P * l_a2;
  // fluxes
  const double F0 = lz[Z_F0], F1 = lz[Z_F1], F2 = lz[Z_F2], F3 = lz[Z_F3], F4 = lz[Z_F4], F5 = lz[Z_F5], F6 = lz[Z_F6];
  // F0 = rho vn
  l_rho += F0 * vn; l_vn += F0 * rho;
  // F1 = rho vn vn + Pstar - Bn Bn
  l_rho += F1 * vn * vn; l_vn += F1 * 2.0 * rho * vn; l_Pstar += F1; l_Bn -= F1 * 2.0 * Bn;
  // F2 = rho vn vt1 - Bn Bt1, F3 = rho vn vt2 - Bn Bt2
  l_rho += F2 * vn * vt1 + F3 * vn * vt2;
  l_vn += F2 * rho * vt1 + F3 * rho * vt2;
  l_vt1 += F2 * rho * vn; l_vt2 += F3 * rho * vn;
  l_Bn -= F2 * Bt1 + F3 * Bt2; l_Bt1 -= F2 * Bn; l_Bt2 -= F3 * Bn;
  // F4 = Bt1 vn - Bn vt1, F5 = Bt2 vn - Bn vt2
  l_Bt1 += F4 * vn; l_vn += F4 * Bt1 + F5 * Bt2; l_Bn -= F4 * vt1 + F5 * vt2; l_vt1 -= F4 * Bn;
  l_Bt2 += F5 * vn; l_vt2 -= F5 * Bn;
  // F6 = (E + Pstar) vn - Bn vB
  l_E += F6 * vn; l_Pstar += F6 * vn; l_vn += F6 * (E + Pstar); l_Bn -= F6 * vB; l_vB -= F6 * Bn;
  // vB = vn Bn + vt1 Bt1 + vt2 Bt2
  l_vn += l_vB * Bn; l_Bn += l_vB * vn; l_vt1 += l_vB * Bt1; l_Bt1 += l_vB * vt1; l_vt2 += l_vB * Bt2;
  l_Bt2 += l_vB * vt2;
  // Pstar = P + B2/2
  l_P += l_Pstar; l_B2 += 0.5 * l_Pstar;
  // P = (gamma-1)(E - (mn vn + mt1 vt1 + mt2 vt2 + B2)/2)
  const double gm = gamma - 1.0;
  l_E += gm * l_P;
  l_mn -= 0.5 * gm * l_P * vn; l_vn -= 0.5 * gm * l_P * mn;
  l_mt1 -= 0.5 * gm * l_P * vt1; l_vt1 -= 0.5 * gm * l_P * mt1;
  l_mt2 -= 0.5 * gm * l_P * vt2; l_vt2 -= 0.5 * gm * l_P * mt2;
  l_B2 -= 0.5 * gm * l_P;
  // B2 = Bn^2 + Bp2, Bp2 = Bt1^2 + Bt2^2
  l_Bn += 2.0 * Bn * l_B2; l_Bp2 += l_B2;
  l_Bt1 += 2.0 * Bt1 * l_Bp2; l_Bt2 += 2.0 * Bt2 * l_Bp2;
  // v = m irho
  l_mn += l_vn * irho; l_mt1 += l_vt1 * irho; l_mt2 += l_vt2 * irho;
  l_irho += l_vn * mn + l_vt1 * mt1 + l_vt2 * mt2;
  // irho = 1/rho
  l_rho -= irho * irho * l_irho;
  out[0] += l_rho; out[1] += l_mn; out[2] += l_mt1; out[3] += l_mt2;
  out[4] += l_E; out[5] += l_Bn; out[6] += l_Bt1; out[7] += l_Bt2;
}

}  // namespace wm
