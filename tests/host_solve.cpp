// The local solve (physics.h, solve.h) on the host, for tests: every bracket of
// every direction of the classes on stdin (13 numbers per line, the chert_class
// fields), one line each:
//   class direction newton_ok newton_miss newton_residual root_ok root_residual
// where the Newton columns are bracket_newton's answer and the root columns
// bracket_root's.  Arguments: mode kernel n_sweep n_dirs newton_iters
// bisect_iters.  With a seventh, "warm", one line per direction instead:
//   class direction status V A rejected V A
// of the plain search and of the surrogate start from 1e-3 rad off its root.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "chert.h"
#include "physics.h"
#include "solve.h"

using namespace chert;

int main(int argc, char** argv) {
  if (argc < 7) return 2;
  const int mode = atoi(argv[1]), n_dirs = atoi(argv[4]);
  SolveParams a{};
  a.kernel = atoi(argv[2]);
  a.n_sweep = atoi(argv[3]);
  a.resid_tol = 1e-9;
  a.newton_iters = atoi(argv[5]);
  a.bisect_iters = atoi(argv[6]);
  double v[13];
  for (int k = 0;; ++k) {
    int got = 0;
    for (int i = 0; i < 13; ++i) got += scanf("%lf", &v[i]) == 1;
    if (got < 13) break;
    const chert_class c{v[0], v[1], v[2], v[3], v[4],  v[5], v[6],
                        v[7], v[8], v[9], v[10], v[11], v[12]};
    const Medium m = load_medium(c);
    const bool el = theta_i_zero(m, mode);
    const int h = sweep_stored(a.n_sweep);
    std::vector<double2> tab((size_t)h);
    for (int j = 0; j < h; ++j) tab[j] = sweep_sample(m, mode, a.kernel, a.n_sweep, j);
    const SweepTable t{tab.data(), nullptr, a.n_sweep, h};
    for (int d = 0; d < n_dirs / 2; ++d) {
      const double psi = wrap_pi(d * (kTwoPi / n_dirs) - m.tilt);
      if (argc > 7) {
        int br[kMaxBr];
        Entry p{}, w{};
        const int st = solve_dir(a, m, mode, t, psi, br, &p);
        double x, y, slope;
        const bool ok = warm_newton(m, mode, a.kernel, el, psi, p.thR + 1e-3, p.thI + 2e-4, &x, &y,
                                    &slope) &&
                        slope >= kWarmSlope && (el || thi_is_nearest(m, mode, a.kernel, x, y)) &&
                        warm_entry(m, mode, a.kernel, el, psi, x, y, 1e-11, &w);
        printf("%d %d %d %.17g %.17g %d %.17g %.17g\n", k, d, st, p.V, p.A, ok ? 0 : 1, w.V, w.A);
        continue;
      }
      t.for_brackets(psi, [&](int j, double2 sa, double2 sb) {
        const Bracket b = bracket_at(a, j, sa, sb, psi);
        double x = 0.0, y = 0.0, miss = NAN;
        Entry ne{}, re{};
        bool ill;
        const bool ok = bracket_newton(a, m, mode, b, sa.x, sb.x, psi, el, &x, &y);
        if (ok) {
          miss = fabs(wrap_pi(ray_angle(energy_velocity(m, mode, a.kernel, x, y)) - psi));
          bracket_entry(a, m, mode, b, psi, el, x, y, &ne, &ill);
        }
        const bool got_root = bracket_root(a, m, mode, j, sa, sb, psi, el, &re, &ill);
        printf("%d %d %d %.17g %.17g %d %.17g\n", k, d, ok ? 1 : 0, miss, ne.res, got_root ? 1 : 0,
               re.res);
      });
    }
  }
  return 0;
}
