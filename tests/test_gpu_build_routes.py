"""The routes of the 2D cache build against each other and the oracle where
their tables and lists have remainders: sweeps that are odd (no half table),
shorter than a chunk, or not a multiple of one; few classes (half sweep, chunk
ranges, lanes sharing a direction) and many (one wavefront per class, every
interval tested); and surrogate-started builds whose rows, jobs and directions
do not fill a workgroup.  Bars: those of the cache parity tests (1e-10 relative,
statuses equal); the routes solve the same equations to the same 1e-10 Newton
step."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
import workloads as W  # noqa: E402
from test_gpu_cache import compare_cache  # noqa: E402
from test_gpu_surrogate import G, compare_to_plain, trained, warm_build  # noqa: E402,F401


def tilted(K, q=60.0):
    return np.stack([O.class_from_thomsen(2500.0 + 37 * k, 1400.0 + 20 * k, 2300, 0.20 - 0.01 * k,
                                          0.03 + 0.01 * k, 0.08, np.radians(9.3 * k - 25.7), 0, q,
                                          0.7 * q) for k in range(K)])


@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("n_sweep,n_dirs", [(16, 8), (17, 24), (31, 360), (77, 24), (208, 360),
                                            (721, 24), (1024, 360)])
def test_plain_routes_agree_with_the_oracle(G, kernel, n_sweep, n_dirs):  # noqa: F811
    import paper_2609_26108_amd as C
    cls, modes = tilted(5), (0, 1, 2)
    fo, so = O.build_cache_2d(cls, n_dirs=n_dirs, mode_mask=0b111, reading=kernel,
                              n_sweep=n_sweep)
    desc = C.cache_desc(n_dirs=n_dirs, modes=modes, kernel=kernel, n_sweep=n_sweep)
    for rep in (1, 200):  # few classes, then one wavefront per (mode, class)
        many = np.tile(cls, (rep, 1))
        cache = G.build_cache(G.classes_from_arrays(many), desc)
        fg, sg = G.cache_to_numpy(cache, desc, many.shape[0])
        for r in (0, rep - 1):
            k = slice(5 * r, 5 * r + 5)
            compare_cache(fg[:, :, k], sg[:, k], fo, so, modes)


@pytest.mark.parametrize("K,n_dirs,n_sweep,modes", [(1, 8, 720, (1,)), (3, 24, 721, (0, 1, 2)),
                                                    (7, 130, 1440, (1, 2)), (41, 8, 1440, (0, 1)),
                                                    (67, 360, 720, (1,))])
def test_surrogate_route_agrees_with_the_plain_one(G, trained, K, n_dirs, n_sweep, modes):  # noqa: F811
    import paper_2609_26108_amd as C
    rows = W.surrogate_training_rows(K, seed=90 + K)
    cls = torch.empty((K, 13), dtype=torch.float64, device=G.DEV)
    C.chert_classes_from_thomsen(torch.from_numpy(rows).to(G.DEV), cls)
    desc = C.cache_desc(n_dirs=n_dirs, modes=modes, n_sweep=n_sweep)
    plain = G.build_cache(cls, desc)
    warm, st = warm_build(G, cls, desc, trained[0], K)
    assert st["jobs"] == len(modes) * K
    fw, sw = G.cache_to_numpy(warm, desc, K)
    fp, sp = G.cache_to_numpy(plain, desc, K)
    compare_to_plain(fw, sw, fp, sp, modes)
