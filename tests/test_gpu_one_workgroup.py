"""Cell networks whose rounds and BFS run in one workgroup per problem, at the
edges of that path: boundary counts on both sides of the register-held weights
(16, 24, 32 nodes per cell), a class-pair table too large to stage, more cells
than the key table holds (rounds by launches), an abort word that is never
raised (likewise), and zero weights, where every segment is tight and a BFS
level holds more nodes and pairs than its LDS lists.  Every output equals the
oracle's node Dijkstra bitwise (the same sums and tie rules, so no tolerance)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from test_oracle_cells import layered_cells  # noqa: E402

KEYS = ("tauR", "tauI", "tstar", "predP", "predA")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import chert_gpu
    return chert_gpu


def classes(K, elastic):
    q = np.inf if elastic else 60.0
    return np.stack([O.class_from_thomsen(2500.0 + 150 * k, 1400.0 + 80 * k, 2300, 0.02 * k,
                                          0.01 * k, 0.08, np.radians(9 * k - 25), 0, q, 0.7 * q)
                     for k in range(K)])


@pytest.mark.parametrize("cn,ncx,ncz,K,elastic,width", [
    (4, 23, 9, 3, False, 8.0), (5, 13, 11, 3, False, 8.0), (6, 11, 9, 3, False, 0.0),
    (7, 9, 8, 2, False, 8.0), (8, 8, 7, 3, False, 8.0), (9, 7, 6, 3, False, 0.0),
    (5, 12, 8, 14, False, 8.0), (1, 150, 120, 3, False, 8.0),
    (5, 30, 30, 2, True, 0.0), (16, 40, 40, 1, True, 0.0)])
def test_networks_bitwise(G, cn, ncx, ncz, K, elastic, width):
    import paper_2609_26108_amd as C
    f, s = O.build_cache_2d(classes(K, elastic), n_dirs=180, mode_mask=0b001, n_sweep=360)
    desc = C.cache_desc(n_dirs=180, modes=(0,))
    cache = G.import_cache(f, s, desc, K)
    cid = layered_cells(ncx, ncz, cn, K, 0)
    NX = ncx * cn + 1
    src = (ncx // 2) * cn + NX * ((ncz // 2) * cn)
    g = G.trace_cells(cache, desc, K, ncx, ncz, cn, 10.0, 7.0, cid, 0, [src], bucket_width=width)
    o = O.trace_cells_2d(ncx, ncz, cn, 10.0, 7.0, cid, f[:, 0], s[0], src)
    for key in KEYS:
        assert np.array_equal(g[key][0], o[key]), key


def test_abort_word_takes_the_launches_per_round(G):
    import paper_2609_26108_amd as C
    K, cn, ncx, ncz = 3, 5, 14, 10
    f, s = O.build_cache_2d(classes(K, False), n_dirs=180, mode_mask=0b001, n_sweep=360)
    desc = C.cache_desc(n_dirs=180, modes=(0,))
    cache = G.import_cache(f, s, desc, K)
    NX, NZ = ncx * cn + 1, ncz * cn + 1
    cid = torch.from_numpy(layered_cells(ncx, ncz, cn, K, 0).reshape(-1).astype(np.int32)).to(G.DEV)
    grid = C.make_cell_grid(ncx, ncz, cn, 10.0, 7.0, cid)
    word = torch.zeros(1, dtype=torch.int32).pin_memory()
    got = []
    for flag in (None, word):
        o = C.trace_opts(C.OUT_ALL, bucket_width=8.0, abort_flag=flag)
        t = {k: torch.empty((1, NX * NZ), dtype=d, device=G.DEV) for k, d in
             (("tau_r", torch.float64), ("tau_i", torch.float64), ("tstar", torch.float64),
              ("pred_p", torch.int32), ("pred_a", torch.int32))}
        ws = torch.empty(C.chert_trace_cells_workspace_bytes(desc, K, grid, 1, o),
                         dtype=torch.uint8, device=G.DEV)
        C.chert_trace_cells(desc, cache, K, grid, 0, [0], o, workspace_dev=ws, **t)
        torch.cuda.synchronize()
        got.append({k: v.cpu().numpy() for k, v in t.items()})
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
