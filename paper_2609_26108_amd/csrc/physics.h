// Device-side local physics of the CHERT cache builder (gfx950, FP64).
//
// Complex energy velocity of a transversely isotropic viscoelastic medium at
// a complex slowness angle theta_R + i theta_I in the sagittal plane of the
// local symmetry-axis frame:
//   complex moduli a = a^R (1 - i/Q)                         (eq 2)
//   n = (sin z, 0, cos z), z = theta_R + i theta_I           (eq 7)
//   Christoffel matrix Gamma_jk = a_ijkl n_i n_l, eigenpair (eq 4)
//   c = sqrt(G), p = n / c                                   (eq 5)
//   MEV: v_m = a_mjkl p_l Re(g_j conj g_k) / (g^H g)          (eqs 13-14)
//   OEV: v_m = a_mjkl p_l g_j g_k / (g^T g)                   (eq 12)
// plus the homogeneity residual (eq 9) and the ray quantities (eqs 10-11).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "chert.h"

namespace chert {

constexpr double kPi = 3.14159265358979323846;
constexpr double kTwoPi = 6.28318530717958647692;
constexpr double kThiStep = 0.25 * kPi / 180.0;  // outward scan step for theta_I
constexpr int kThiSteps = 120;                    // 120 * 0.25 deg = 30 deg
constexpr double kThiTol = 1e-15;
constexpr double kIllSlope = 1e-2;
constexpr double kTieRel = 1e-12;

// sinh and cosh of the outward scan's angles (k + 1) kThiStep, filled at
// compile time from the power series (|x| <= 0.53: eleven terms are exact to
// the last bit); the scan index is uniform over a wavefront, so a lane reads
// a scalar instead of evaluating expm1 and a division
struct ScanTable {
  double sh[kThiSteps], ch[kThiSteps];
};
constexpr ScanTable make_scan_table() {
  ScanTable t{};
  for (int k = 0; k < kThiSteps; ++k) {
    const double x = (k + 1) * kThiStep, x2 = x * x;
    double s = 1.0, c = 1.0;
    for (int n = 11; n >= 1; --n) {
      s = 1.0 + s * x2 / ((2.0 * n) * (2.0 * n + 1.0));
      c = 1.0 + c * x2 / ((2.0 * n - 1.0) * (2.0 * n));
    }
    t.sh[k] = x * s;
    t.ch[k] = c;
  }
  return t;
}
__constant__ constexpr ScanTable kScan = make_scan_table();

struct cd {
  double re, im;
};

__device__ __forceinline__ cd mk(double r, double i) { return cd{r, i}; }
__device__ __forceinline__ cd operator+(cd a, cd b) { return cd{a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cd operator-(cd a, cd b) { return cd{a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cd operator*(cd a, cd b) {
  return cd{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cd operator*(double s, cd a) { return cd{s * a.re, s * a.im}; }
__device__ __forceinline__ double norm2(cd a) { return a.re * a.re + a.im * a.im; }
__device__ __forceinline__ cd conjg(cd a) { return cd{a.re, -a.im}; }
__device__ __forceinline__ cd cdiv(cd a, cd b) {
  double d = norm2(b);
  return cd{(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}
// a / b and c / b with one reciprocal of |b|^2 (one division instead of four)
__device__ __forceinline__ void cdiv2(cd a, cd c, cd b, cd* qa, cd* qc) {
  const double inv = 1.0 / norm2(b);
  *qa = cd{(a.re * b.re + a.im * b.im) * inv, (a.im * b.re - a.re * b.im) * inv};
  *qc = cd{(c.re * b.re + c.im * b.im) * inv, (c.im * b.re - c.re * b.im) * inv};
}
// sinh x and cosh x from one expm1 (half the instructions of the two
// library calls): e^x - e^-x = m + m / (1 + m) with m = e^x - 1, no
// cancellation for either sign; exact at x = 0
__device__ __forceinline__ void sinh_cosh(double x, double* sh, double* ch) {
  const double m = expm1(x);
  const double e = 1.0 + m;
  const double ie = 1.0 / e;
  *sh = 0.5 * (m + m * ie);
  *ch = 0.5 * (e + ie);
}
// principal square root (Re >= 0), cancellation-free form
__device__ __forceinline__ cd csqrt_p(cd z) {
  double ax = fabs(z.re);
  double r = sqrt(z.re * z.re + z.im * z.im);
  if (r == 0.0) return cd{0.0, 0.0};
  double t = sqrt(0.5 * (ax + r));
  if (z.re >= 0.0) return cd{t, z.im / (2.0 * t)};
  return cd{fabs(z.im) / (2.0 * t), copysign(t, z.im)};
}

// complex moduli of one class, over 4^unit: a power of four near a33, so that
// products of many moduli (the Newton determinant holds twenty-two) stay in
// range whatever the caller's units; angles and residuals do not change by a
// bit, velocities are over 2^unit
struct Medium {
  cd a11, a13, a33, a44, a66;
  int unit;
  double q_ps, q_sh;  // largest quality factor of the coupled modes' a11, a33, a44; of qSH's
  bool elastic_ps, elastic_sh;
  bool fluid;  // no shear stiffness and a11 = a13 = a33: isotropic fluid
  double tilt;
};

__device__ __forceinline__ cd complex_modulus(double aR, double q) {
  double aI = isinf(q) ? 0.0 : aR / q;
  return cd{aR, -aI};
}

__device__ __forceinline__ Medium load_medium(const chert_class& c) {
  Medium m;
  int e = 0;
  (void)frexp(c.a33, &e);  // (unusable classes: any)
  m.unit = e >> 1;
  const int s = -2 * m.unit;
  m.a11 = complex_modulus(ldexp(c.a11, s), c.q11);
  m.a13 = complex_modulus(ldexp(c.a13, s), c.q13);
  m.a33 = complex_modulus(ldexp(c.a33, s), c.q33);
  m.a44 = complex_modulus(ldexp(c.a44, s), c.q44);
  m.a66 = complex_modulus(ldexp(c.a66, s), c.q66);
  const double q44 = c.a44 == 0.0 ? 0.0 : c.q44;
  m.q_ps = fmax(q44, fmax(c.q11, c.q33));
  m.q_sh = fmax(q44, c.q66);
  m.elastic_ps = m.a11.im == 0.0 && m.a13.im == 0.0 && m.a33.im == 0.0 && m.a44.im == 0.0;
  m.elastic_sh = m.a44.im == 0.0 && m.a66.im == 0.0;
  m.fluid = m.a44.re == 0.0 && m.a44.im == 0.0 && m.a66.re == 0.0 && m.a66.im == 0.0 &&
            m.a11.re == m.a13.re && m.a11.im == m.a13.im && m.a11.re == m.a33.re &&
            m.a11.im == m.a33.im;
  m.tilt = c.tilt;
  return m;
}

__device__ __forceinline__ bool mode_elastic(const Medium& m, int mode) {
  return mode == CHERT_QSH ? m.elastic_sh : m.elastic_ps;
}

// Modes whose homogeneous solution is theta_I = 0 exactly: elastic modes and
// qP of an isotropic fluid (its residual is cubic in theta_I, so a numerical
// root would only be determined to ~1e-6 rad).
__device__ __forceinline__ bool theta_i_zero(const Medium& m, int mode) {
  return mode_elastic(m, mode) || (mode == CHERT_QP && m.fluid);
}

// complex energy velocity (local frame): v = (v1, v3)
struct Vel {
  cd v1, v3;
};

// sin, cos of theta_R and sinh, cosh of theta_I: the only transcendental
// inputs of the evaluation, so loops that hold theta_R (the theta_I scan)
// or step it by a fixed amount (difference quotients) compute them once
struct Trig {
  double sr, cr, sh, ch;
};

__device__ __forceinline__ Trig trig_of(double thR, double thI) {
  Trig t;
  sincos(thR, &t.sr, &t.cr);
  sinh_cosh(thI, &t.sh, &t.ch);
  return t;
}

__device__ __forceinline__ Vel energy_velocity_t(const Medium& m, int mode, int kernel,
                                                 const Trig& t) {
  const double sr = t.sr, cr = t.cr, sh = t.sh, ch = t.ch;
  cd n1 = cd{sr * ch, cr * sh};   // sin(z)
  cd n3 = cd{cr * ch, -sr * sh};  // cos(z)
  cd n11 = n1 * n1, n33 = n3 * n3;
  Vel out;
  if (mode == CHERT_QSH) {
    cd G = m.a66 * n11 + m.a44 * n33;
    cd c = csqrt_p(G);
    cd p1, p3;
    cdiv2(n1, n3, c, &p1, &p3);
    out.v1 = m.a66 * p1;
    out.v3 = m.a44 * p3;
    return out;
  }
  cd G11 = m.a11 * n11 + m.a44 * n33;
  cd G33 = m.a44 * n11 + m.a33 * n33;
  cd a1344 = m.a13 + m.a44;
  cd G13 = a1344 * (n1 * n3);
  cd mean = 0.5 * (G11 + G33);
  cd half = 0.5 * (G11 - G33);
  cd root = csqrt_p(half * half + G13 * G13);
  cd G = (mode == CHERT_QP) ? mean + root : mean - root;
  // the better conditioned of (G13, G - G11) and (G - G33, G13)
  const cd ub = G - G11, wa = G - G33;
  const bool u = norm2(ub) >= norm2(wa);
  cd g1 = u ? G13 : wa;
  cd g3 = u ? ub : G13;
  cd c = csqrt_p(G);
  cd p1, p3;
  cdiv2(n1, n3, c, &p1, &p3);
  if (kernel == CHERT_KERNEL_OEV) {
    cd N = g1 * g1 + g3 * g3;
    cd S11 = cdiv(g1 * g1, N);
    cd S33 = cdiv(g3 * g3, N);
    cd S13 = cdiv(g1 * g3, N);
    out.v1 = p1 * (m.a11 * S11 + m.a44 * S33) + p3 * (a1344 * S13);
    out.v3 = p3 * (m.a33 * S33 + m.a44 * S11) + p1 * (a1344 * S13);
    return out;
  }
  // MEV: S = Re(g g^H) / (g^H g) is real, so moduli scale by reals
  double q1 = norm2(g1), q3 = norm2(g3);
  const double invN = 1.0 / (q1 + q3);
  const double S11 = q1 * invN, S33 = q3 * invN;
  const double S13 = (g1.re * g3.re + g1.im * g3.im) * invN;
  const cd B = S13 * a1344;
  out.v1 = p1 * (S11 * m.a11 + S33 * m.a44) + p3 * B;
  out.v3 = p3 * (S33 * m.a33 + S11 * m.a44) + p1 * B;
  return out;
}

__device__ __forceinline__ Vel energy_velocity(const Medium& m, int mode, int kernel,
                                               double thR, double thI) {
  return energy_velocity_t(m, mode, kernel, trig_of(thR, thI));
}

// sine of the angle between v^R and v^I (eq 9): zero when collinear
__device__ __forceinline__ double homog_residual(const Vel& v) {
  double r1 = v.v1.re, r3 = v.v3.re, i1 = v.v1.im, i3 = v.v3.im;
  return (r1 * i3 - r3 * i1) / sqrt((r1 * r1 + r3 * r3) * (i1 * i1 + i3 * i3));
}

__device__ __forceinline__ double ray_angle(const Vel& v) { return atan2(v.v1.re, v.v3.re); }

// into (-pi, pi]
__device__ __forceinline__ double wrap_pi(double a) {
  if (a > kPi) a -= kTwoPi;
  else if (a <= -kPi) a += kTwoPi;
  return a;
}

// The energy velocity up to a factor: v = w / D with D = c (qSH), c (g^H g)
// (MEV) or c (g^T g) (OEV).  The direction of Re v, its homogeneity
// (Im(conj(v1) v3) = 0) and the residual's sign need no normalisation of g
// and no division: Im(conj(w1) w3) has the residual's sign and its zeros,
// with one complex square root instead of two and none of the divisions of
// energy_velocity_t (the root searches below evaluate nothing else).  The
// builds are bound by FP64 issue: with these values, the interpolating
// refinement and the exact Jacobian below, the plain per-node build of 10,201
// nodes x 2 modes went from 41.2 to 27.7 ms, MSPM's corner solves on 40 x 20
// cells from 50.7 to 24.8 ms, the surrogate-started build of 80,601 nodes
// from 7.7 to 6.0 ms, the five-class 2D cache from 290 to 117 us.
struct Raw {
  cd w1, w3;  // unnormalised velocity
  cd G;       // eigenvalue, c = sqrt(G)
  cd N;       // OEV: g^T g (MEV, qSH: real and positive, left at 1)
};

__device__ __forceinline__ Raw energy_raw(const Medium& m, int mode, int kernel, const Trig& t) {
  const double sr = t.sr, cr = t.cr, sh = t.sh, ch = t.ch;
  const cd n1 = cd{sr * ch, cr * sh}, n3 = cd{cr * ch, -sr * sh};
  const cd n11 = n1 * n1, n33 = n3 * n3;
  Raw o;
  o.N = cd{1.0, 0.0};
  if (mode == CHERT_QSH) {
    o.G = m.a66 * n11 + m.a44 * n33;
    o.w1 = m.a66 * n1;
    o.w3 = m.a44 * n3;
    return o;
  }
  const cd G11 = m.a11 * n11 + m.a44 * n33;
  const cd G33 = m.a44 * n11 + m.a33 * n33;
  const cd b = m.a13 + m.a44;
  const cd G13 = b * (n1 * n3);
  const cd mean = 0.5 * (G11 + G33);
  const cd half = 0.5 * (G11 - G33);
  const cd root = csqrt_p(half * half + G13 * G13);
  o.G = (mode == CHERT_QP) ? mean + root : mean - root;
  const cd ub = o.G - G11, wa = o.G - G33;
  const bool u = norm2(ub) >= norm2(wa);  // the better conditioned of the two eigenvectors
  const cd g1 = u ? G13 : wa, g3 = u ? ub : G13;
  if (kernel == CHERT_KERNEL_OEV) {
    const cd S11 = g1 * g1, S33 = g3 * g3, S13 = b * (g1 * g3);
    o.N = S11 + S33;
    o.w1 = n1 * (m.a11 * S11 + m.a44 * S33) + n3 * S13;
    o.w3 = n3 * (m.a33 * S33 + m.a44 * S11) + n1 * S13;
    return o;
  }
  const double q1 = norm2(g1), q3 = norm2(g3);
  const cd B = (g1.re * g3.re + g1.im * g3.im) * b;
  o.w1 = n1 * (q1 * m.a11 + q3 * m.a44) + n3 * B;
  o.w3 = n3 * (q3 * m.a33 + q1 * m.a44) + n1 * B;
  return o;
}

// One Newton system of the local solve: unknowns (theta_R, theta_I) = (x, y),
// equations h = 0 (eq 9) and ray angle = psi*, both up to positive factors.
//   f1 = Im(conj(U1) U3), f2 = sin(miss) cos(miss) |Re U|^2, U = w conj(D)
// (a positive multiple of v).  f2 also vanishes where the ray is reversed or
// perpendicular to the target; `near` tells the target's own zero from those.
// Everything but the MEV products Re(g_j
// conj g_k) is analytic in z = x + i y, so one complex derivative gives both
// columns (d/dy = i d/dz): about the cost of one evaluation more instead of
// the two of difference quotients, and the iteration is truly quadratic.
struct NewtonSys {
  double f1, f2;
  double a11, a12, a21, a22;  // rows of f1 and f2
  double r2;                  // |Re U|^2: d psi / dx = a21 / r2
  bool near;                  // |miss| < pi / 4
};

__device__ __forceinline__ cd times_i(cd a) { return cd{-a.im, a.re}; }

__device__ __forceinline__ NewtonSys newton_sys(const Medium& m, int mode, int kernel,
                                                const Trig& t, double sp, double cp) {
  const cd n1 = cd{t.sr * t.ch, t.cr * t.sh}, n3 = cd{t.cr * t.ch, -t.sr * t.sh};
  const cd n11 = n1 * n1, n33 = n3 * n3, n13 = n1 * n3;
  cd w1, w3, w1x, w3x, w1y, w3y, D, Dz;
  if (mode == CHERT_QSH) {
    const cd G = m.a66 * n11 + m.a44 * n33;
    const cd Gz = 2.0 * ((m.a66 - m.a44) * n13);
    D = csqrt_p(G);
    Dz = cdiv(0.5 * Gz, D);
    w1 = m.a66 * n1;
    w3 = m.a44 * n3;
    w1x = m.a66 * n3;
    w3x = mk(0.0, 0.0) - m.a44 * n1;
    w1y = times_i(w1x);
    w3y = times_i(w3x);
  } else {
    const cd G11 = m.a11 * n11 + m.a44 * n33;
    const cd G33 = m.a44 * n11 + m.a33 * n33;
    const cd b = m.a13 + m.a44;
    const cd G13 = b * n13;
    const cd G11z = 2.0 * ((m.a11 - m.a44) * n13);
    const cd G33z = 2.0 * ((m.a44 - m.a33) * n13);
    const cd G13z = b * (n33 - n11);
    const cd half = 0.5 * (G11 - G33), halfz = 0.5 * (G11z - G33z);
    cd root = csqrt_p(half * half + G13 * G13);
    cd rootz = cdiv(half * halfz + G13 * G13z, root);
    if (mode != CHERT_QP) {
      root = mk(0.0, 0.0) - root;
      rootz = mk(0.0, 0.0) - rootz;
    }
    const cd G = 0.5 * (G11 + G33) + root;
    const cd Gz = 0.5 * (G11z + G33z) + rootz;
    const cd c = csqrt_p(G);
    const cd cz = cdiv(0.5 * Gz, c);
    const cd ub = G - G11, wa = G - G33;
    const bool u = norm2(ub) >= norm2(wa);
    const cd g1 = u ? G13 : wa, g3 = u ? ub : G13;
    const cd g1z = u ? G13z : Gz - G33z, g3z = u ? Gz - G11z : G13z;
    if (kernel == CHERT_KERNEL_OEV) {
      const cd S11 = g1 * g1, S33 = g3 * g3, B = b * (g1 * g3);
      const cd S11z = 2.0 * (g1 * g1z), S33z = 2.0 * (g3 * g3z);
      const cd Bz = b * (g1z * g3 + g1 * g3z);
      const cd P = m.a11 * S11 + m.a44 * S33, Q = m.a33 * S33 + m.a44 * S11;
      w1 = n1 * P + n3 * B;
      w3 = n3 * Q + n1 * B;
      w1x = n3 * P - n1 * B + n1 * (m.a11 * S11z + m.a44 * S33z) + n3 * Bz;
      w3x = n3 * B - n1 * Q + n3 * (m.a33 * S33z + m.a44 * S11z) + n1 * Bz;
      w1y = times_i(w1x);
      w3y = times_i(w3x);
      const cd N = S11 + S33;
      D = c * N;
      Dz = cz * N + c * (S11z + S33z);
    } else {
      const double q1 = norm2(g1), q3 = norm2(g3);
      const double q13 = g1.re * g3.re + g1.im * g3.im;
      // d|g|^2/dx = 2 Re(conj(g) g'), d/dy = -2 Im(conj(g) g')
      const cd e1 = conjg(g1) * g1z, e3 = conjg(g3) * g3z;
      const cd e13 = conjg(g3) * g1z + conjg(g1) * g3z;
      const cd P = q1 * m.a11 + q3 * m.a44, Q = q3 * m.a33 + q1 * m.a44;
      const cd B = q13 * b;
      w1 = n1 * P + n3 * B;
      w3 = n3 * Q + n1 * B;
      const cd d1 = n3 * P - n1 * B, d3 = n3 * B - n1 * Q;  // through n alone
      const double x1 = 2.0 * e1.re, x3 = 2.0 * e3.re, x13 = e13.re;
      w1x = d1 + n1 * (x1 * m.a11 + x3 * m.a44) + n3 * (x13 * b);
      w3x = d3 + n3 * (x3 * m.a33 + x1 * m.a44) + n1 * (x13 * b);
      const double y1 = -2.0 * e1.im, y3 = -2.0 * e3.im, y13 = -e13.im;
      w1y = times_i(d1) + n1 * (y1 * m.a11 + y3 * m.a44) + n3 * (y13 * b);
      w3y = times_i(d3) + n3 * (y3 * m.a33 + y1 * m.a44) + n1 * (y13 * b);
      D = c;
      Dz = cz;
    }
  }
  const cd Dc = conjg(D), Dzc = conjg(Dz), Dyc = cd{-Dzc.im, Dzc.re};  // conj(i D') = -i conj(D')
  const cd U1 = w1 * Dc, U3 = w3 * Dc;
  const cd U1x = w1x * Dc + w1 * Dzc, U3x = w3x * Dc + w3 * Dzc;
  const cd U1y = w1y * Dc - w1 * Dyc, U3y = w3y * Dc - w3 * Dyc;
  NewtonSys o;
  o.f1 = U1.re * U3.im - U3.re * U1.im;
  o.a11 = U1x.re * U3.im + U1.re * U3x.im - U3x.re * U1.im - U3.re * U1x.im;
  o.a12 = U1y.re * U3.im + U1.re * U3y.im - U3y.re * U1.im - U3.re * U1y.im;
  const double cr = U1.re * cp - U3.re * sp, dt = U3.re * cp + U1.re * sp;
  o.f2 = cr * dt;
  o.a21 = (U1x.re * cp - U3x.re * sp) * dt - cr * (U3x.re * cp + U1x.re * sp);
  o.a22 = (U1y.re * cp - U3y.re * sp) * dt - cr * (U3y.re * cp + U1y.re * sp);
  o.r2 = cr * cr + dt * dt;
  o.near = fabs(cr) < dt;
  return o;
}

// sign and zeros of the homogeneity residual (eq 9) at theta_R with
// sine/cosine (sr, cr) and theta_I with (sh, ch).  LIT: the residual itself
// (literal normalised velocities; see bisect_root)
template <bool LIT = false>
__device__ __forceinline__ double h_sign(const Medium& m, int mode, int kernel, double sr,
                                         double cr, double sh, double ch) {
  if constexpr (LIT) return homog_residual(energy_velocity_t(m, mode, kernel, Trig{sr, cr, sh, ch}));
  const Raw r = energy_raw(m, mode, kernel, Trig{sr, cr, sh, ch});
  return r.w1.re * r.w3.im - r.w3.re * r.w1.im;
}

// the outward scan's values at +-(k + 1) kThiStep (sinh is odd, cosh even)
template <bool LIT = false>
__device__ __forceinline__ void h_scan_pair(const Medium& m, int mode, int kernel, double sr,
                                            double cr, int k, double* hp, double* hn) {
  const double sb = kScan.sh[k], cb = kScan.ch[k];
  *hp = h_sign<LIT>(m, mode, kernel, sr, cr, sb, cb);
  *hn = h_sign<LIT>(m, mode, kernel, sr, cr, -sb, cb);
}

__device__ __forceinline__ bool brackets(double fa, double fb) {
  if (isnan(fa) || isnan(fb)) return false;
  return (fa < 0.0) != (fb < 0.0);
}

template <bool LIT = false>
__device__ __forceinline__ double h_at_thi(const Medium& m, int mode, int kernel, double sr,
                                           double cr, double y) {
  double sh, ch;
  sinh_cosh(y, &sh, &ch);
  return h_sign<LIT>(m, mode, kernel, sr, cr, sh, ch);
}

// root of the parabola through (a, fa), (b, fb), (e, fe) nearest the secant
// point of a and b: the secant point, then one Newton step on the parabola
// (the remaining error is of the third order in the spread); the secant
// point itself where the step leaves [a, b]
__device__ __forceinline__ double parabola_root(double a, double b, double e, double fa,
                                                double fb, double fe) {
  const double d1 = (fb - fa) / (b - a);
  const double d2 = ((fe - fb) / (e - b) - d1) / (e - a);
  const double c = b - fb / d1;
  const double y = c - (c - a) * (c - b) * d2 / (d1 + d2 * (2.0 * c - a - b));
  const double lo = fmin(a, b), hi = fmax(a, b);
  return (y > lo && y < hi) ? y : ((c > lo && c < hi) ? c : 0.5 * (a + b));
}

// Root of h(thR, .) in the bracket [a, b]; (e, fe) is a third sample near it,
// (sr, cr) sine and cosine of thR.  Two interpolation steps leave an error of
// ~1e-12 and 1e-19 rad on the smooth residual (bracket 4.4e-3 rad), so a
// secant through them ends the search after two evaluations; where the last
// step is not small yet (LIT: at once), Illinois (modified regula falsi) on the
// bracket held so far.
constexpr double kThiStepDone = 1e-10;
template <bool LIT = false>
__device__ __forceinline__ double refine_thi(const Medium& m, int mode, int kernel, double sr,
                                             double cr, double a, double b, double fa,
                                             double fb, double e, double fe) {
  if constexpr (!LIT) {
    const double y0 = parabola_root(a, b, e, fa, fb, fe);
    const double f0 = h_at_thi<LIT>(m, mode, kernel, sr, cr, y0);
    if (f0 == 0.0) return y0;
    double xe, fxe;  // the bracket end that y0 replaces stays as the third point
    if ((f0 < 0.0) == (fa < 0.0)) {
      xe = a; fxe = fa; a = y0; fa = f0;
    } else {
      xe = b; fxe = fb; b = y0; fb = f0;
    }
    const double y1 = parabola_root(a, b, xe, fa, fb, fxe);
    const double f1 = h_at_thi<LIT>(m, mode, kernel, sr, cr, y1);
    if (f1 == 0.0) return y1;
    const double y2 = y1 - f1 * (y1 - y0) / (f1 - f0);
    if ((f1 < 0.0) == (fa < 0.0)) {
      a = y1; fa = f1;
    } else {
      b = y1; fb = f1;
    }
    // (where y1 is already the root to rounding, y2 may leave the bracket by
    // an ulp)
    if (fabs(y2 - y1) <= kThiStepDone && fabs(y1 - y0) <= 1e-4) return y2;
  }
  int side = 0;
  double c = 0.5 * (a + b);
  for (int it = 0; it < 80; ++it) {
    double cn = (a * fb - b * fa) / (fb - fa);
    if (!(cn > fmin(a, b) && cn < fmax(a, b))) cn = 0.5 * (a + b);
    const double fc = h_at_thi<LIT>(m, mode, kernel, sr, cr, cn);
    double step = fabs(cn - c);
    c = cn;
    if (fc == 0.0) break;
    if ((fc < 0.0) == (fa < 0.0)) {
      a = c;
      fa = fc;
      if (side == -1) fb *= 0.5;
      side = -1;
    } else {
      b = c;
      fb = fc;
      if (side == 1) fa *= 0.5;
      side = 1;
    }
    if (fabs(b - a) <= kThiTol || step <= 1e-17) break;
  }
  return c;
}

// theta_I(theta_R): root of the homogeneity residual nearest 0 in [-30, 30]
// deg, found by an outward 0.25-degree scan.  Returns false if none.
// Written for wavefront lockstep: every lane first scans until the whole
// wavefront has its bracket, then all lanes refine together, whichever side
// their bracket is on.  (sr, cr) = sine and cosine of thR.
template <bool LIT = false>
__device__ __forceinline__ bool theta_imag_sc(const Medium& m, int mode, int kernel, double sr,
                                              double cr, double* thI) {
  if (theta_i_zero(m, mode)) {
    *thI = 0.0;
    return true;
  }
  const double h0 = h_sign<LIT>(m, mode, kernel, sr, cr, 0.0, 1.0);
  bool done = (h0 == 0.0);
  bool bp = false, bn = false;
  int kb = 0;  // the bracket is [kb, kb + 1] steps out
  double p0 = h0, p1 = h0, p2 = h0;  // values at kb - 1 (k = 0: the other side), kb, kb + 1
  double n0 = h0, n1 = h0, n2 = h0;
  for (int k = 0; k < kThiSteps; ++k) {
    if (!done) {
      p0 = p1;
      p1 = p2;
      n0 = n1;
      n1 = n2;
      h_scan_pair<LIT>(m, mode, kernel, sr, cr, k, &p2, &n2);
      if (k == 0) {
        p0 = n2;
        n0 = p2;
      }
      bp = brackets(p1, p2);
      bn = brackets(n2, n1);
      kb = k;
      done = bp || bn;
    }
    if (__all(done)) break;
  }
  if (h0 == 0.0) {
    *thI = 0.0;
    return true;
  }
  if (!bp && !bn) return false;
  const double s = bp ? 1.0 : -1.0;
  double r = refine_thi<LIT>(m, mode, kernel, sr, cr, s * (kb * kThiStep), s * ((kb + 1) * kThiStep),
                        bp ? p1 : n1, bp ? p2 : n2, s * ((kb - 1) * kThiStep), bp ? p0 : n0);
  if (bp && bn) {  // a bracket on each side: the root nearer 0, the positive one on a tie
    const double rn = refine_thi<LIT>(m, mode, kernel, sr, cr, -(kb * kThiStep),
                                 -((kb + 1) * kThiStep), n1, n2, -((kb - 1) * kThiStep), n0);
    if (fabs(rn) < fabs(r)) r = rn;
  }
  *thI = r;
  return true;
}

template <bool LIT = false>
__device__ __forceinline__ bool theta_imag(const Medium& m, int mode, int kernel, double thR,
                                           double* thI) {
  double sr, cr;
  sincos(thR, &sr, &cr);
  return theta_imag_sc<LIT>(m, mode, kernel, sr, cr, thI);
}

// ray angle at (thR, thI) given sin, cos of thR
template <bool LIT = false>
__device__ __forceinline__ double ray_angle_sc(const Medium& m, int mode, int kernel, double sr,
                                               double cr, double thI) {
  double sh, ch;
  sinh_cosh(thI, &sh, &ch);
  if constexpr (LIT) return ray_angle(energy_velocity_t(m, mode, kernel, Trig{sr, cr, sh, ch}));
  const Raw r = energy_raw(m, mode, kernel, Trig{sr, cr, sh, ch});
  const cd D = conjg(kernel == CHERT_KERNEL_OEV ? csqrt_p(r.G) * r.N : csqrt_p(r.G));
  return atan2((r.w1 * D).re, (r.w3 * D).re);
}

// Ray angle of the elastic medium with m's real moduli at a real theta_R: the
// map above with everything real (both kernels then agree), a seventh of its
// operations.  NaN where the eigenvalue is not positive (unstable moduli).
__device__ __forceinline__ double ray_angle_elastic(const Medium& m, int mode, double sr,
                                                    double cr) {
  const double n11 = sr * sr, n33 = cr * cr, a44 = m.a44.re;
  if (mode == CHERT_QSH) {
    const double a66 = m.a66.re;
    return a66 * n11 + a44 * n33 > 0.0 ? atan2(a66 * sr, a44 * cr) : NAN;
  }
  const double G11 = m.a11.re * n11 + a44 * n33, G33 = a44 * n11 + m.a33.re * n33;
  const double b = m.a13.re + a44, G13 = b * (sr * cr);
  const double half = 0.5 * (G11 - G33), root = sqrt(half * half + G13 * G13);
  const double G = 0.5 * (G11 + G33) + (mode == CHERT_QP ? root : -root);
  const double ub = G - G11, wa = G - G33;
  const bool u = ub * ub >= wa * wa;
  const double g1 = u ? G13 : wa, g3 = u ? ub : G13;
  const double S11 = g1 * g1, S33 = g3 * g3, B = b * (g1 * g3);
  const double w1 = sr * (m.a11.re * S11 + a44 * S33) + cr * B;
  const double w3 = cr * (m.a33.re * S33 + a44 * S11) + sr * B;
  return G > 0.0 ? atan2(w1, w3) : NAN;
}

struct Entry {
  double V, A, Q, r1, r3, thR, thI, res;
};

// ray quantities from a homogeneous complex energy velocity (eqs 10-11) over
// 2^unit
__device__ __forceinline__ void ray_quantities(const Vel& v, int unit, Entry* e) {
  double r1 = v.v1.re, r3 = v.v3.re, i1 = v.v1.im, i3 = v.v3.im;
  double vr = sqrt(r1 * r1 + r3 * r3);
  double u1 = r1 / vr, u3 = r3 / vr;
  double vi = i1 * u1 + i3 * u3;
  double s = vr * vr + vi * vi;
  e->V = ldexp(s / vr, unit);
  e->A = ldexp(-vi / s, -unit);
  e->Q = (vi == 0.0) ? INFINITY : -(vr * vr - vi * vi) / (2.0 * vr * vi);
  e->r1 = u1;
  e->r3 = u3;
}

}  // namespace chert
