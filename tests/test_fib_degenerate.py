"""3D stars whose offsets have no direction (an infinite spacing, or spacings
whose squared length underflows): the call returns, with the bins that a search
over every direction gives (index 0 where no dot product is a number).  In a
process of its own, so that a search without an end fails the test."""
import subprocess
import sys

import pytest

CODE = """
import numpy as np
import paper_2609_26108_amd as C
hx, hy, hz = {spacing}
n = {n_dirs}
i = np.arange(n, dtype=np.float64)
z = 1.0 - (2.0 * i + 1.0) / n
r = np.sqrt(1.0 - z * z)
ph = i * (np.pi * (3.0 - np.sqrt(5.0)))
f = (r * np.cos(ph), r * np.sin(ph), z)
ox, oy, oz, L, b = C.chert_star_3d(2, hx, hy, hz, n)
assert len(ox) > 0
with np.errstate(all="ignore"):
    for o in range(len(ox)):
        d = sum(fi * (np.float64(x) * h / L[o]) for fi, x, h in
                zip(f, (ox[o], oy[o], oz[o]), (hx, hy, hz)))
        d = np.where(np.isnan(d), -2.0, d)
        assert 0 <= b[o] < n
        if d.max() > -2.0:
            tie = np.inf if np.isinf(d.max()) else 4e-16 * max(1.0, abs(d.max()))
            assert d[b[o]] == d.max() or d[b[o]] >= d.max() - tie
        else:
            assert b[o] == 0
print("ok")
"""


@pytest.mark.parametrize("n_dirs", [2, 100, 41253])
@pytest.mark.parametrize("spacing", ["(np.inf, 10.0, 10.0)", "(1e-200, 1e-200, 1e-200)",
                                     "(1e-170, 1.0, 1e-170)", "(1e-162, 3e-162, 2e-162)",
                                     "(1e200, 1.0, 1.0)"])
def test_star_without_directions_returns(spacing, n_dirs):
    r = subprocess.run([sys.executable, "-c", CODE.format(spacing=spacing, n_dirs=n_dirs)],
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ok" in r.stdout, r.stderr[-2000:]
