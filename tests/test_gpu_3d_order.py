"""Tile ordering of large 3D batches (switched on above twice the resident
workgroups when the caller gives no round cap): the rounds stay of the order of
the unordered relaxation's whatever the weights' contrast, and the fields are
bitwise the unordered ones.  A nearly lossless class (Q 1e6 beside 40) makes the
smallest attenuation weight 25,000 times smaller than the others, a fine axis
the smallest traveltime weight 200 times; ordered by the smallest weight, a
round held about one tile a problem."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import chert_gpu
    return chert_gpu


def model(nx, ny, nz, contrast):
    import paper_2609_26108_amd as C
    rows = [C.chert_class_from_thomsen(2600.0 + 500 * k, 1500.0 + 250 * k, 2300.0, 0.1, 0.05, 0.08,
                                       0.3 * k, 0.5 * k, 40.0, 25.0).as_array() for k in range(3)]
    if contrast:
        rows[1][5:10] = 1e6
    z = np.arange(nz)[:, None, None] + 0.1 * np.arange(nx)[None, None, :]
    cid = np.minimum((z * 3 / (1.3 * nz)).astype(np.int32), 2) + np.zeros((nz, ny, nx), np.int32)
    return np.stack(rows), np.ascontiguousarray(cid)


@pytest.mark.parametrize("launch", [0, 1])
@pytest.mark.parametrize("contrast,hz", [(False, 10.0), (True, 10.0), (True, 0.05)])
def test_ordered_rounds_are_bounded(G, contrast, hz, launch):
    import paper_2609_26108_amd as C
    nx, ny, nz = 104, 96, 56  # 13 x 12 x 7 tiles, 2 sources x 2 fields: 4,368
    rows, cid = model(nx, ny, nz, contrast)
    K = len(rows)
    desc = C.cache_desc(dim=3, n_dirs=400, modes=(0,), n_sweep=360)
    cache = G.build_cache(G.classes_from_arrays(rows), desc)
    g = C.make_grid3(nx, ny, nz, 10.0, 2, torch.from_numpy(cid.reshape(-1)).to(G.DEV), hz=hz)
    n, src = nx * ny * nz, [0, nx * ny * nz // 2 + nx // 3]
    out = []
    for cap in (0, 5000):  # by themselves; a caller's cap: unordered
        st = C.TraceStats()
        o = C.trace_opts(C.OUT_TAU_R | C.OUT_TAU_I, max_rounds=cap, launch=launch, stats=st)
        tr = torch.empty((2, n), dtype=torch.float64, device=G.DEV)
        ti = torch.empty((2, n), dtype=torch.float64, device=G.DEV)
        ws = torch.empty(C.chert_trace_workspace_bytes(desc, K, g, 2, o), dtype=torch.uint8,
                         device=G.DEV)
        C.chert_trace_field(desc, cache, K, g, 0, src, o, tr, ti, None, None, None, ws)
        torch.cuda.synchronize()
        d = st.as_dict()
        print(contrast, hz, launch, cap, d["rounds"][0], d["tile_visits"][0], flush=True)
        out.append((tr, ti, d["rounds"][0]))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    # ordered rounds (64 + 2 x 32 tiles along the axes at most), then no more
    # than the unordered relaxation takes, which starts with less done
    assert out[0][2] <= 64 + 2 * (13 + 12 + 7) + out[1][2] + 8
