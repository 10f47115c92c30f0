"""The two forms of the cell and block networks' rounds and trees: one
workgroup per problem (k_cell_march, k_cell_tree), and a launch per round and
per BFS level (k_cell_relax, k_cell_level and their 3D forms), which a call with
an abort word takes so that the host can poll it.  Every output of the launched
form equals the oracle's bitwise, and the one-workgroup form's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from test_gpu_blocks3d import banded, tti3_classes  # noqa: E402
from test_gpu_cells import KEYS, tti_classes  # noqa: E402
from test_oracle_cells import layered_cells  # noqa: E402


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import chert_gpu
    return chert_gpu


class Recorded:
    """Options with an abort word that stays 0, and the kernels of the calls."""

    def __init__(self, monkeypatch, word):
        import paper_2609_26108_amd as C
        self.C, self.word, make = C, None, C.trace_opts
        if word:
            self.word = torch.zeros(1, dtype=torch.int32).pin_memory()
            monkeypatch.setattr(C, "trace_opts",
                                lambda *a, **k: make(*a, **{**k, "abort_flag": self.word}))

    def __enter__(self):
        self.C.chert_prof_enable(True)
        return self

    def __exit__(self, *exc):
        self.kernels = set(self.C.chert_prof_read())
        self.C.chert_prof_enable(False)


def both_forms(monkeypatch, call, launched, single):
    out = []
    for word in (True, False):
        with monkeypatch.context() as mp, Recorded(mp, word) as r:
            out.append(call())
        assert set(launched if word else single) <= r.kernels, r.kernels
        if word:
            assert not set(single) & r.kernels, r.kernels
    for key in out[0]:
        assert np.array_equal(out[0][key], out[1][key], equal_nan=True), key
    return out[0]


@pytest.mark.parametrize("cn,ncx,ncz,bucket", [(1, 9, 7, 0.0), (5, 13, 8, 16.0), (16, 3, 2, 0.0)])
def test_cells_with_abort_word_bitwise(G, monkeypatch, cn, ncx, ncz, bucket):
    import paper_2609_26108_amd as C
    cls = tti_classes()
    f, s = O.build_cache_2d(cls, n_dirs=360, mode_mask=0b011)
    desc = C.cache_desc(n_dirs=360, modes=(0, 1))
    cache = G.import_cache(f, s, desc, 3)
    NX, NZ, _ = O.cell_lattice(ncx, ncz, cn)
    cid = layered_cells(ncx, ncz, cn, 3, 0)
    srcs = [0, NX * NZ - 1]
    g = both_forms(monkeypatch, lambda: G.trace_cells(cache, desc, 3, ncx, ncz, cn, 10.0, 7.0, cid,
                                                      1, srcs, bucket_width=bucket),
                   ("k_cell_relax", "k_cell_level"), ("k_cell_tight", "k_cell_tree"))
    for si, src in enumerate(srcs):
        o = O.trace_cells_2d(ncx, ncz, cn, 10.0, 7.0, cid, f[:, 1], s[1], src)
        for key in KEYS:
            assert np.array_equal(g[key][si], o[key]), (si, key)


@pytest.mark.parametrize("cn", [1, 3])
def test_blocks_with_abort_word_bitwise(G, monkeypatch, cn):
    import paper_2609_26108_amd as C
    f, s = O.build_cache_3d(tti3_classes(), N=400, mode_mask=0b010, n_sweep=360)
    desc = C.cache_desc(dim=3, n_dirs=400, modes=(1,), n_sweep=360)
    cache = G.import_cache(f, s, desc, 3)
    n, h = (4, 3, 5), (10.0, 12.0, 9.0)
    NX, NY, NZ, _ = O.block_lattice(*n, cn)
    cid = banded(NX, NY, NZ, 3, cn)
    srcs = [0, NX * NY * NZ - 1]
    g = both_forms(monkeypatch, lambda: G.trace_blocks(cache, desc, 3, *n, cn, *h, cid, 1, srcs),
                   ("k_block_relax", "k_block_level"), ("k_cell_tight", "k_cell_tree"))
    for si, src in enumerate(srcs):
        o = O.trace_blocks_3d(*n, cn, *h, cid, f[0, 1], f[1, 1], s[1], src, N=400)
        for key in KEYS:
            assert np.array_equal(g[key][si], o[key]), (si, key)


def test_mspm_with_abort_word_bitwise(G, monkeypatch):
    import paper_2609_26108_amd as C
    cls = tti_classes()
    cid = layered_cells(6, 5, 3, 3, 0)
    both_forms(monkeypatch, lambda: G.trace_mspm(cls, 6, 5, 3, 10.0, 10.0, cid, 0, [0],
                                                 outputs=C.OUT_ALL, n_sweep=360),
               ("k_cell_relax", "k_cell_level"), ("k_cell_tight", "k_cell_tree"))


@pytest.mark.parametrize("ncx,ncz,cn,n_src,bucket,launched", [
    (20, 12, 5, 1, 0.0, False), (80, 40, 5, 1, 0.0, True), (80, 40, 5, 16, 0.0, False),
    (80, 40, 5, 1, 16.0, False), (160, 80, 5, 1, 0.0, True), (20, 10, 16, 1, 0.0, True)])
def test_rounds_take_the_faster_form(G, ncx, ncz, cn, n_src, bucket, launched):
    """Networks on both sides of the rule between one workgroup per problem and
    a launch per round: the form taken, and both forms' fields bitwise alike."""
    import paper_2609_26108_amd as C
    cls = tti_classes()
    f, s = O.build_cache_2d(cls, n_dirs=360, mode_mask=0b001)
    desc = C.cache_desc(n_dirs=360, modes=(0,))
    cache = G.import_cache(f, s, desc, 3)
    NX, NZ, _ = O.cell_lattice(ncx, ncz, cn)
    cid = layered_cells(ncx, ncz, cn, 3, 0)
    srcs = [(q * 977 * cn) % NX for q in range(n_src)]  # on the top edge
    run = lambda: G.trace_cells(cache, desc, 3, ncx, ncz, cn, 10.0, 10.0, cid, 0, srcs,  # noqa: E731
                                bucket_width=bucket)
    with pytest.MonkeyPatch.context() as mp:
        with Recorded(mp, False) as r:
            a = run()
    assert ("k_cell_relax" in r.kernels) == launched and ("k_cell_march" in r.kernels) != launched
    with pytest.MonkeyPatch.context() as mp:
        with Recorded(mp, True):
            b = run()
    for key in KEYS:
        assert np.array_equal(a[key], b[key]), key


@pytest.mark.parametrize("nc,n_src,launched", [((8, 8, 8), 1, False), ((14, 14, 14), 1, True),
                                               ((14, 14, 14), 8, False)])
def test_block_trees_take_the_faster_form(G, nc, n_src, launched):
    import paper_2609_26108_amd as C
    f, s = O.build_cache_3d(tti3_classes(), N=400, mode_mask=0b001, n_sweep=360)
    desc = C.cache_desc(dim=3, n_dirs=400, modes=(0,), n_sweep=360)
    cache = G.import_cache(f, s, desc, 3)
    NX, NY, NZ, _ = O.block_lattice(*nc, 3)
    cid = banded(NX, NY, NZ, 3, 3)
    srcs = [3 * q for q in range(n_src)]
    run = lambda: G.trace_blocks(cache, desc, 3, *nc, 3, 10.0, 10.0, 10.0, cid, 0, srcs)  # noqa: E731
    with pytest.MonkeyPatch.context() as mp:
        with Recorded(mp, False) as r:
            a = run()
    assert ("k_block_level" in r.kernels) == launched and ("k_cell_tree" in r.kernels) != launched
    with pytest.MonkeyPatch.context() as mp:
        with Recorded(mp, True):
            b = run()
    for key in KEYS:
        assert np.array_equal(a[key], b[key]), key
