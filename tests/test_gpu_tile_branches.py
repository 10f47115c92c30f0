"""The branches of the tile visits at their edges, on imported oracle caches:
2D boxes of one class, with the class-pair table in LDS and too large for it;
homogeneous elastic media, where fans of exact ties give nodes more tight edges
than a thread holds; stars larger than a small tile and offset groups that do
not divide a workgroup; 3D boxes of one class, of more classes than a staged
weight code covers, and more classes than the code table holds.  Fields,
predecessors and t* equal the oracle's Dijkstra bitwise (the same sums and tie
rules, so no tolerance)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
import workloads as W  # noqa: E402
from test_gpu_3d import trace3  # noqa: E402
from test_gpu_trace import assert_fields_equal  # noqa: E402


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import chert_gpu
    return chert_gpu


def classes(K, elastic=False, tilt=True):
    q = np.inf if elastic else 60.0
    return np.stack([O.class_from_thomsen(2500.0 + 11 * k, 1400.0 + 6 * k, 2300,
                                          0.1 if tilt else 0.0, 0.05 if tilt else 0.0, 0.08,
                                          np.radians(7.3 * k - 25) if tilt else 0.0, 0, q, 0.7 * q)
                     for k in range(K)])


@pytest.mark.parametrize("K,elastic,nx,nz,radius,tile,group,launch", [
    (1, True, 61, 43, 5, (0, 0), 0, 0), (1, True, 40, 70, 5, (16, 64), 4, 0),
    (1, False, 37, 29, 8, (8, 8), 2, 1), (1, True, 33, 31, 1, (32, 32), 8, 0),
    (3, False, 53, 47, 8, (8, 12), 1, 0), (3, False, 41, 39, 4, (5, 7), 2, 1),
    (14, False, 45, 38, 5, (16, 16), 2, 0), (14, False, 45, 38, 5, (32, 32), 4, 1)])
def test_2d_tiles(G, K, elastic, nx, nz, radius, tile, group, launch):
    import paper_2609_26108_amd as C
    cls = classes(K, elastic, tilt=not elastic)
    f, s = O.build_cache_2d(cls, mode_mask=0b011, n_sweep=360)
    desc = C.cache_desc(modes=(0, 1), n_sweep=360)
    cache = G.import_cache(f, s, desc, K)
    rng = np.random.default_rng(K * 100 + nx)
    cid = rng.integers(0, K, (nz, nx)).astype(np.int32)
    cid[: nz // 2, : nx // 2] = 0  # boxes of one class among mixed ones
    srcs = [0, nx * nz - 1, (nz // 2) * nx + nx // 3]
    g = G.trace(cache, desc, K, nx, nz, 10.0, 10.0, radius, cid, 1, srcs, tile_x=tile[0],
                tile_z=tile[1], launch=launch, push_group=group)
    for si, src in enumerate(srcs):
        o = O.trace_2d(nx, nz, 10.0, 10.0, cid, radius, f[0, 1], f[1, 1], s[1], src)
        assert_fields_equal(g, o, si)


@pytest.mark.parametrize("K,radius,tile,launch", [(1, 2, (0, 0), 0), (5, 2, (4, 4), 1),
                                                  (5, 3, (0, 0), 0), (70, 1, (0, 0), 1),
                                                  (70, 2, (4, 16), 0)])
def test_3d_tiles(G, K, radius, tile, launch):
    import paper_2609_26108_amd as C
    cls = classes(K)
    f, s = O.build_cache_3d(cls, N=200, mode_mask=0b001, n_sweep=180)
    desc = C.cache_desc(dim=3, n_dirs=200, modes=(0,), n_sweep=180)
    cache = G.import_cache(f, s, desc, K)
    nx, ny, nz = 19, 14, 17
    rng = np.random.default_rng(K + radius)
    cid = rng.integers(0, K, (nz, ny, nx)).astype(np.int32)
    m = W.config5(nx=nx, ny=ny, nz=nz, n_interfaces=1, radius=radius,
                  sources=((0, 0, 0), (9, 7, 16)))
    m = W.Model3D(m.name, nx, ny, nz, m.h, m.layers, cid, m.sources, m.modes, radius)
    g, _ = trace3(G, m, cache, desc, K, 0, full=True, launch=launch, tile=tile)
    for si, src in enumerate(m.sources):
        o = O.trace_3d(nx, ny, nz, m.h, m.h, m.h, cid, radius, f[0, 0], f[1, 0], s[0], src, N=200)
        for key in ("tauR", "tauI", "tstar", "predP", "predA"):
            assert np.array_equal(g[key][si], o[key]), (si, key)
