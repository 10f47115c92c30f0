"""The 3D star's bins (the Fibonacci direction closest to each offset) against
a search over every direction: the library evaluates only the directions whose
polar angle and azimuth can be close enough, and must still return the largest
dot product's lowest index, for every direction count from the smallest on and
for uneven spacings (offsets near the poles and the equator included)."""
import numpy as np
import pytest

import paper_2609_26108_amd as C


def directions(n):
    i = np.arange(n, dtype=np.float64)
    z = 1.0 - (2.0 * i + 1.0) / n
    r = np.sqrt(1.0 - z * z)
    ph = i * (np.pi * (3.0 - np.sqrt(5.0)))
    return r * np.cos(ph), r * np.sin(ph), z


@pytest.mark.parametrize("n_dirs", [2, 3, 7, 17, 20, 100, 999, 41253, 300001])
@pytest.mark.parametrize("spacing", [(10.0, 10.0, 10.0), (1.0, 30.0, 0.02), (25.0, 3.0, 400.0)])
def test_star_bins_equal_the_full_search(n_dirs, spacing):
    radius = 4 if n_dirs < 300000 else 1
    hx, hy, hz = spacing
    ox, oy, oz, L, b = C.chert_star_3d(radius, hx, hy, hz, n_dirs)
    fx, fy, fz = directions(n_dirs)
    for o in range(len(ox)):
        u = (ox[o] * hx / L[o], oy[o] * hy / L[o], oz[o] * hz / L[o])
        d = fx * u[0] + fy * u[1] + fz * u[2]
        # numpy's sine may differ from libm's in the last bit: the bin's dot
        # product is the largest up to two roundings, and the first such one
        # wherever the runner-up is clearly apart
        assert d[b[o]] >= d.max() - 4e-16
        clear = np.flatnonzero(d >= d.max() - 1e-14)
        if len(clear) == 1:
            assert b[o] == clear[0]
