// The local solve of one target ray direction (eqs 9-11), shared by the
// cache build's kernels and by the host-side operation count: bracket the
// target on a theta_R sweep table, refine each bracket by a 2D Newton
// iteration on (homogeneity residual, ray-direction miss) with a nested
// bisection as fallback, keep the first arrival; and the surrogate start's
// Newton polish with the check that its theta_I is the root nearest 0.
#pragma once

#include "physics.h"

namespace chert {

// What the solve steps read of a build's arguments.
struct SolveParams {
  int kernel;        // CHERT_KERNEL_MEV or _OEV
  int n_sweep;       // theta_R samples of the sweep table
  double resid_tol;  // entries whose residual is above this get CHERT_ST_NOCONV
  int newton_iters;  // Newton steps per bracket
  int bisect_iters;  // halvings of the bisection fallback
};

constexpr double kWarmWindow = 0.35;  // the polish may move theta_R this far [rad]
constexpr double kWarmSlope = 0.05;   // its accepted roots: slope at least this

// Newton steps below this end the iteration: it is quadratic, so the error
// left is the square of the last step (times the curvature), far below the
// rounding of the equations
constexpr double kNewtonDone = 1e-10;

constexpr double kBisectStop = 1e-14;  // the bisection's last interval [rad]

// One Newton step of (h, ray angle - psi*) at (x, y); (sp, cp) = sine and
// cosine of psi*.  `el`: theta_I stays 0 and only the direction equation is
// solved.  *slope: d psi / d theta_R along h = 0 (`el`: along y = 0).  False
// where the ray at (x, y) is more than pi / 4 from the target: an iteration
// that settles there has found the target's reverse or its perpendicular.
__device__ __forceinline__ bool newton_step(const Medium& m, int mode, int kernel, bool el,
                                            double x, double y, double sp, double cp, double* dx,
                                            double* dy, double* slope) {
  const NewtonSys q = newton_sys(m, mode, kernel, trig_of(x, y), sp, cp);
  if (el) {
    *dx = -q.f2 / q.a21;
    *dy = 0.0;
    *slope = q.a21 / q.r2;
    return q.near;
  }
  const double det = q.a11 * q.a22 - q.a12 * q.a21;
  const double inv = 1.0 / det;
  *dx = -(q.a22 * q.f1 - q.a12 * q.f2) * inv;
  *dy = -(q.a11 * q.f2 - q.a21 * q.f1) * inv;
  *slope = -det / (q.a12 * q.r2);
  return q.near;
}

// Newton on newton_sys's equations from the bracket interpolant; only the
// target's own direction is accepted.  Elastic modes keep theta_I = 0 exactly
// and solve the 1D direction equation.
__device__ __forceinline__ bool newton_root(const Medium& m, int mode, int kernel,
                                         double psi_star, double ta, double tb,
                                         double ya, double yb, double fa, double fb,
                                         int iters, double* xo, double* yo) {
  const bool el = theta_i_zero(m, mode);
  const double dth = tb - ta;
  double t = fa / (fa - fb);
  double x = ta + t * dth;
  double y = el ? 0.0 : ya + t * (yb - ya);
  double last = 1.0, sp, cp;
  sincos(psi_star, &sp, &cp);
  bool near = false;
  for (int it = 0; it < iters; ++it) {
    double dx, dy, slope;
    near = newton_step(m, mode, kernel, el, x, y, sp, cp, &dx, &dy, &slope);
    if (!isfinite(dx) || !isfinite(dy)) return false;
    x += dx;
    y += dy;
    if (x < ta - dth || x > tb + dth || fabs(y) > 30.0 * kPi / 180.0) return false;
    last = fmax(fabs(dx), fabs(dy));
    if (last < kNewtonDone) break;
  }
  if (!(last < kNewtonDone) || !near) return false;
  *xo = x;
  *yo = y;
  return true;
}

// Fallback: nested bisection on theta_R with the inner theta_I solve at every
// trial point (slow, used only when Newton does not settle or the entry's
// attenuation cancels).  LIT: the definition in its literal operations --
// normalised velocities and residuals, regula falsi -- at twice the cost.
template <bool LIT>
__device__ __forceinline__ bool bisect_root(const Medium& m, int mode, int kernel,
                                         double psi_star, double ta, double tb, double fa,
                                         int iters, double* xo, double* yo) {
  double lo = ta, hi = tb;
  bool neg_lo = fa < 0.0;
  for (int it = 0; it < iters && hi - lo > kBisectStop; ++it) {
    double mid = 0.5 * (lo + hi);
    double thI, sr, cr;
    sincos(mid, &sr, &cr);
    if (!theta_imag_sc<LIT>(m, mode, kernel, sr, cr, &thI)) return false;
    double fm = wrap_pi(ray_angle_sc<LIT>(m, mode, kernel, sr, cr, thI) - psi_star);
    if ((fm < 0.0) == neg_lo) lo = mid;
    else hi = mid;
  }
  double x = 0.5 * (lo + hi);
  double y;
  if (!theta_imag<LIT>(m, mode, kernel, x, &y)) return false;
  *xo = x;
  *yo = y;
  return true;
}

// Is y the theta_I that theta_imag's outward scan returns at theta_R = x?
// No bracket of the residual closer to 0 on either side, the bracket
// holding y on its side, none in the same step on the other side.
__device__ __forceinline__ bool thi_is_nearest(const Medium& m, int mode, int kernel, double x,
                                               double y) {
  const int kr = (int)floor(fabs(y) / kThiStep);
  if (kr >= kThiSteps || y == 0.0) return false;
  double sr, cr;
  sincos(x, &sr, &cr);
  const double h0 = h_sign(m, mode, kernel, sr, cr, 0.0, 1.0);
  if (h0 == 0.0) return false;
  double hp_lo = h0, hn_hi = h0;
  for (int k = 0; k <= kr; ++k) {
    double hp_hi, hn_lo;  // the same evaluations as theta_imag's scan
    h_scan_pair(m, mode, kernel, sr, cr, k, &hp_hi, &hn_lo);
    const bool bp = brackets(hp_lo, hp_hi);
    const bool bn = brackets(hn_lo, hn_hi);
    if (k < kr) {
      if (bp || bn) return false;
    } else {
      const bool mine = y > 0.0 ? bp : bn;
      const bool other = y > 0.0 ? bn : bp;
      if (!mine || other) return false;
    }
    hp_lo = hp_hi;
    hn_hi = hn_lo;
  }
  return true;
}

__device__ __forceinline__ double ang_dist(double a, double b) { return fabs(wrap_pi(a - b)); }

constexpr int kMaxBr = 6;  // brackets kept per lane for the lockstep refinement

// does the sweep interval with end points sa, sb hold the target angle?
__device__ __forceinline__ bool is_bracket(double2 sa, double2 sb, double psi_star) {
  if (isnan(sa.y) || isnan(sb.y)) return false;
  double fa = wrap_pi(sa.y - psi_star);
  double fb = wrap_pi(sb.y - psi_star);
  if (fabs(fb - fa) >= kPi) return false;  // the +-pi seam, not a crossing
  return brackets(fa, fb);
}

// Sweep tables: (theta_I, ray angle) of theta_R sample j, NaN angle where
// the sample has no root.
//
// The sweep of a class.  v(theta_R + pi) = -v(theta_R), so with an even
// number of samples only the first half is solved and stored (h = n / 2):
// sample j + h has the same theta_I and the ray angle turned by pi.
// With `rng` the samples are grouped in chunks of kSweepChunk intervals, each
// with the range of ray angles it spans (base, lowest and highest offset from
// it): a target tests 2 h / kSweepChunk ranges and then the intervals of the
// one or two chunks that hold it, instead of all n intervals.  (An odd chunk
// length: lanes reading different chunks then fall on different LDS banks.)
constexpr int kSweepChunk = 15;
__host__ __device__ inline int sweep_stored(int n) { return (n & 1) ? n : n / 2; }
__host__ __device__ inline int sweep_chunks(int n) {
  return (sweep_stored(n) + kSweepChunk - 1) / kSweepChunk;
}

__device__ __forceinline__ double2 sweep_at(const double2* t, int h, int j) {
  if (j < h) return t[j];
  const double2 v = t[j - h];
  return make_double2(v.x, wrap_pi(v.y + kPi));
}

struct SweepTable {
  const double2* t;   // [h]
  const double* rng;  // [chunks][3], or null: every interval is tested
  int n, h;
  __device__ __forceinline__ double2 at(int j) const { return sweep_at(t, h, j); }
  // f(j, sample j, sample j + 1) for every interval j holding psi, ascending
  template <class Fn>
  __device__ __forceinline__ void for_brackets(double psi, Fn&& f) const {
    if (!rng) {
      scan(0, n, psi, f);
      return;
    }
    const int nc = (h + kSweepChunk - 1) / kSweepChunk;
    for (int j0 = 0; j0 < n; j0 += h) {
      const double tgt = j0 ? wrap_pi(psi - kPi) : psi;
      for (int c0 = 0; c0 < nc; c0 += 64) {
        // the chunks that may hold the target first, so that the lanes of a
        // wavefront then walk their own chunks side by side
        const int nw = nc - c0 < 64 ? nc - c0 : 64;
        unsigned long long hit = 0ull;
        for (int q = 0; q < nw; ++q) {
          const double* r = rng + 3 * (c0 + q);
          const double d = wrap_pi(tgt - r[0]);
          if (d >= r[1] && d <= r[2]) hit |= 1ull << q;
        }
        while (hit) {
          const int c = c0 + __builtin_ctzll(hit);
          hit &= hit - 1ull;
          const int lo = c * kSweepChunk;
          scan(j0 + lo, j0 + (lo + kSweepChunk < h ? lo + kSweepChunk : h), psi, f);
        }
      }
    }
  }
  template <class Fn>
  __device__ __forceinline__ void scan(int lo, int hi, double psi, Fn&& f) const {
    double2 sa = at(lo);
    for (int j = lo; j < hi; ++j) {
      const double2 sb = at(j + 1 == n ? 0 : j + 1);
      if (is_bracket(sa, sb, psi)) f(j, sa, sb);
      sa = sb;
    }
  }
};

// The range of chunk c of a stored sweep: base angle, lowest and highest
// offset (widened by far more than the rounding of the sums).  A chunk with a
// missing sample, or spanning more than 3 rad, is always searched.
__device__ __forceinline__ void sweep_range(const double2* t, int n, int h, int c, double* r) {
  const int lo = c * kSweepChunk, hi = lo + kSweepChunk < h ? lo + kSweepChunk : h;
  double prev = t[lo].y, off = 0.0, mn = 0.0, mx = 0.0;
  r[0] = prev;
  bool all = isnan(prev);
  for (int j = lo; j < hi; ++j) {
    const double y = sweep_at(t, h, j + 1 == n ? 0 : j + 1).y;
    all = all || isnan(y);
    off = off + wrap_pi(y - prev);
    mn = fmin(mn, off);
    mx = fmax(mx, off);
    prev = y;
  }
  if (all || mx - mn > 3.0) {
    r[0] = 0.0;
    mn = -4.0;
    mx = 4.0;
  }
  r[1] = mn - 1e-9;
  r[2] = mx + 1e-9;
}

// One theta_R sample of a class's sweep.
__device__ __forceinline__ double2 sweep_sample(const Medium& m, int mode, int kernel, int n_sweep,
                                                int j) {
  const double thR = (j + 0.5) * (kTwoPi / n_sweep);
  double thI, sr, cr;
  sincos(thR, &sr, &cr);
  if (theta_imag_sc(m, mode, kernel, sr, cr, &thI)) {
    const double psi = ray_angle_sc(m, mode, kernel, sr, cr, thI);
    if (isfinite(psi)) return make_double2(thI, psi);
  }
  return make_double2(0.0, NAN);
}

// A windowed table holds the marked ones of the h stored samples in ascending
// order (pos[j] is the slot of sample j or -1) and reads every other sample as
// NaN; the second half of the sweep is the image of the first, as above.
struct WindowTable {
  const int16_t* pos;
  const double2* ent;
  int h;
  __device__ __forceinline__ double2 at(int j) const {
    const int p = pos[j < h ? j : j - h];
    if (p < 0) return make_double2(0.0, NAN);
    const double2 v = ent[p];
    return j < h ? v : make_double2(v.x, wrap_pi(v.y + kPi));
  }
};

// A bracket of the target ray angle: its theta_R interval and the misses at
// the ends.
struct Bracket {
  double ta, tb, fa, fb;
};
__device__ __forceinline__ Bracket bracket_at(const SolveParams& a, int j, double2 sa, double2 sb,
                                              double psi_star) {
  const double dth = kTwoPi / a.n_sweep;
  Bracket b;
  b.fa = wrap_pi(sa.y - psi_star);
  b.fb = wrap_pi(sb.y - psi_star);
  b.ta = (j + 0.5) * dth;
  b.tb = b.ta + dth;
  return b;
}

// Newton step of a bracket whose ends have theta_I = ya, yb; false where the
// bisection has to decide.
__device__ __forceinline__ bool bracket_newton(const SolveParams& a, const Medium& m, int mode,
                                               const Bracket& b, double ya, double yb,
                                               double psi_star, bool el, double* xo, double* yo) {
  double x, y;
  bool ok = newton_root(m, mode, a.kernel, psi_star, b.ta, b.tb, ya, yb, b.fa, b.fb,
                        a.newton_iters, &x, &y);
  // The 2D Newton iteration does not know which homogeneity root theta_I
  // must be: keep its root only if y is the root nearest 0 at the final
  // theta_R (the outward scan's answer there); otherwise -- theta_I(theta_R)
  // switching branches inside the bracket -- the nested bisection follows
  // that definition.
  // It must also lie in its own bracket (the bisection's interval), not
  // wander into a neighbouring one.
  if (ok) ok = x >= b.ta - 1e-12 && x <= b.tb + 1e-12;
  // (y in the first bracket of the scan, alone there, is that answer without
  // refining it; anything else is compared with the scan's own root.)
  if (ok && !el && !thi_is_nearest(m, mode, a.kernel, x, y)) {
    double sx, cx, ys;
    sincos(x, &sx, &cx);
    ok = theta_imag_sc(m, mode, a.kernel, sx, cx, &ys) && fabs(ys - y) <= 1e-9;
  }
  *xo = x;
  *yo = y;
  return ok;
}

// The ray quantities of a bracket's root.  *ill: the bracket's ray-angle
// slope is below kIllSlope.
__device__ __forceinline__ void bracket_entry(const SolveParams& a, const Medium& m, int mode,
                                              const Bracket& b, double psi_star, bool el, double x,
                                              double y, Entry* cand, bool* ill) {
  if (x >= kTwoPi) x -= kTwoPi;
  if (x < 0.0) x += kTwoPi;
  Vel v = energy_velocity(m, mode, a.kernel, x, y);
  ray_quantities(v, m.unit, cand);
  cand->thR = x;
  cand->thI = y;
  double h = el ? 0.0 : homog_residual(v);
  cand->res = fmax(fabs(h), fabs(wrap_pi(ray_angle(v) - psi_star)));
  *ill = fabs((b.fb - b.fa) / (b.tb - b.ta)) < kIllSlope;
}

// Has the attenuation of an entry cancelled to under a thousandth of the
// least of the mode's losses?  (The OEV maps pass through zero next to their
// branch changes; MEV's do not.)  The angles' last bit then moves A by 1e-10 of
// itself, so which of the neighbouring 64-bit angles is stored decides its
// last six digits.  Every build takes the literal bisection's, which are the
// sequential definition's, digit for digit; they are no closer to the exact
// root than Newton's (240,000 OEV qSV entries against 80-bit roots: A off by
// more than 1e-10 in one of them, without this rule in none, by finite
// differences and bisection alone in five).
__device__ __forceinline__ bool loss_cancelled(const Medium& m, int mode, bool el,
                                               const Entry& e) {
  // (the loss of a modulus, |Im a| / Re a, is 1 / Q)
  return !el && fabs(e.A) * e.V * (mode == CHERT_QSH ? m.q_sh : m.q_ps) < 1e-3;
}

// Can the bisection of bracket b reach its stop within the halvings that the
// caller allows?  A converged Newton root is not given up for fewer.
__device__ __forceinline__ bool bisection_completes(const SolveParams& a, const Bracket& b) {
  const long long steps = 1ll << (a.bisect_iters < 62 ? a.bisect_iters : 62);
  return b.tb - b.ta <= kBisectStop * (double)steps;
}

// Is the literal bisection's theta_R the root x again?  (Where the ray-angle
// map jumps inside the bracket, it may close on the jump instead.)
__device__ __forceinline__ bool same_root(double lit, double x) { return fabs(lit - x) <= 1e-6; }

// The root of the bracket at sweep sample j and its ray quantities; false if
// neither the Newton step nor the bisection converges.
__device__ __forceinline__ bool bracket_root(const SolveParams& a, const Medium& m, int mode,
                                             int j, double2 sa, double2 sb, double psi_star,
                                             bool el, Entry* cand, bool* cand_ill) {
  const Bracket b = bracket_at(a, j, sa, sb, psi_star);
  double x, y;
  if (!bracket_newton(a, m, mode, b, sa.x, sb.x, psi_star, el, &x, &y) &&
      !bisect_root<false>(m, mode, a.kernel, psi_star, b.ta, b.tb, b.fa, a.bisect_iters, &x, &y))
    return false;
  bracket_entry(a, m, mode, b, psi_star, el, x, y, cand, cand_ill);
  double xl, yl;
  if (loss_cancelled(m, mode, el, *cand) && bisection_completes(a, b) &&
      bisect_root<true>(m, mode, a.kernel, psi_star, b.ta, b.tb, b.fa, a.bisect_iters, &xl, &yl) &&
      same_root(xl, x))
    bracket_entry(a, m, mode, b, psi_star, el, xl, yl, cand, cand_ill);
  return true;
}

// Fold a refined bracket into the running first-arrival choice, brackets in
// scan order: a root (residual within tol) beats a refinement that closed on
// a jump of the ray-angle map; among equals the first, then a larger ray
// velocity; ties (kTieRel) go to the smaller |theta_R - psi*|.
__device__ __forceinline__ void fold_choice(const Entry& cand, bool cand_ill, double psi_star,
                                            double tol, bool* found, bool* ill, Entry* best) {
  bool take;
  const bool cand_root = cand.res <= tol, best_root = *found && best->res <= tol;
  if (!*found) take = true;
  else if (cand_root != best_root) take = cand_root;
  else if (cand.V > best->V * (1.0 + kTieRel)) take = true;
  else take = fabs(cand.V - best->V) <= kTieRel * best->V &&
              ang_dist(cand.thR, psi_star) < ang_dist(best->thR, psi_star);
  if (take) {
    *best = cand;
    *ill = cand_ill;
    *found = true;
  }
}

__device__ __forceinline__ void refine_bracket_at(const SolveParams& a, const Medium& m,
                                                  int mode,
                                                  int j, double2 sa, double2 sb, double psi_star,
                                                  bool el, bool* found, bool* ill, Entry* best) {
  Entry cand;
  bool cand_ill;
  if (bracket_root(a, m, mode, j, sa, sb, psi_star, el, &cand, &cand_ill))
    fold_choice(cand, cand_ill, psi_star, a.resid_tol, found, ill, best);
}

// status of a solved direction from the folded choice (as the plain search)
__device__ __forceinline__ int32_t solve_status(bool found, bool ill, const Entry& best) {
  if (!found) return CHERT_ST_NO_BRACKET;
  int32_t st = ill ? CHERT_ST_ILL : CHERT_ST_OK;
  if (!(best.A >= 0.0) || !isfinite(best.V) || !(best.V > 0.0)) st |= CHERT_ST_NONPHYS;
  return st;
}

// Solve target direction psi_star for one (class, mode) from its sweep
// table.  Lanes of a wavefront run it in step (brackets first, then the
// refinements together); `br` is this lane's kMaxBr bracket slots in LDS.
__device__ __forceinline__ int32_t solve_dir(const SolveParams& a, const Medium& m, int mode,
                                             const SweepTable& tab, double psi_star, int* br,
                                             Entry* best) {
  const bool el = theta_i_zero(m, mode);
  // phase 1: every sign change of the ray-direction miss over the sweep
  int nbr = 0;
  tab.for_brackets(psi_star, [&](int j, double2, double2) {
    if (nbr < kMaxBr) br[nbr] = j;
    ++nbr;
  });
  // phase 2: refine the kept brackets with all lanes in step
  bool found = false, ill = false;
  for (int sidx = 0; sidx < kMaxBr; ++sidx) {
    if (__all(sidx >= nbr)) break;
    if (sidx < nbr) {
      const int j = br[sidx];
      refine_bracket_at(a, m, mode, j, tab.at(j), tab.at(j + 1 == a.n_sweep ? 0 : j + 1),
                        psi_star, el, &found, &ill, best);
    }
  }
  // rare: more brackets than slots; refine the rest in scan order
  if (nbr > kMaxBr) {
    int seen = 0;
    tab.for_brackets(psi_star, [&](int j, double2 sa, double2 sb) {
      if (seen++ < kMaxBr) return;
      refine_bracket_at(a, m, mode, j, sa, sb, psi_star, el, &found, &ill, best);
    });
  }
  return solve_status(found, ill, *best);
}

// Newton on the same equations from (x0, y0), as newton_root but started
// from a prediction and kept within kWarmWindow of it; *slope is
// d psi / d theta_R along the homogeneous curve h = 0 at the last iterate.
__device__ __forceinline__ bool warm_newton(const Medium& m, int mode, int kernel, bool el,
                                         double psi_star, double x0, double y0, double* xo,
                                         double* yo, double* slope) {
  double x = x0, y = el ? 0.0 : y0, last = 1.0, sl = NAN, sp, cp;
  sincos(psi_star, &sp, &cp);
  bool near = false;
  for (int it = 0; it < 16; ++it) {
    double dx, dy;
    near = newton_step(m, mode, kernel, el, x, y, sp, cp, &dx, &dy, &sl);
    if (!isfinite(dx) || !isfinite(dy)) return false;
    x += dx;
    y += dy;
    if (fabs(x - x0) > kWarmWindow || fabs(y) > 30.0 * kPi / 180.0) return false;
    last = fmax(fabs(dx), fabs(dy));
    if (last < kNewtonDone) break;
  }
  if (!(last < kNewtonDone) || !near) return false;
  *xo = x;
  *yo = y;
  *slope = sl;
  return true;
}

// The entry of a polished root whose slope and theta_I have passed, and whether
// it stands as the plain search's: a physical root within resid_tol whose
// attenuation has not cancelled.
__device__ __forceinline__ bool warm_entry(const Medium& m, int mode, int kernel, bool el,
                                           double psi_star, double x, double y, double resid_tol,
                                           Entry* e) {
  if (fabs(x) >= kTwoPi) x = fmod(x, kTwoPi);
  if (x < 0.0) x += kTwoPi;
  const Vel v = energy_velocity(m, mode, kernel, x, y);
  ray_quantities(v, m.unit, e);
  e->thR = x;
  e->thI = y;
  const double h = el ? 0.0 : homog_residual(v);
  e->res = fmax(fabs(h), fabs(wrap_pi(ray_angle(v) - psi_star)));
  return e->res <= resid_tol && e->V > 0.0 && isfinite(e->V) && e->A >= 0.0 &&
         !loss_cancelled(m, mode, el, *e);
}

}  // namespace chert
