"""Training gradients at batch sizes around the sample tile (32) and around the
number of partials summed together (16 tiles), against the BF16 emulation: the
bars of the ragged-batch gradient test (loss 1e-3, every parameter block 1e-2
relative)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import surrogate as S  # noqa: E402
from test_gpu_surrogate import G, _fit_random_norm, new_blob, random_params, standardise  # noqa: E402,F401


@pytest.mark.parametrize("batch", [1, 17, 31, 32, 33, 511, 512, 513, 545])
def test_gradient_at_tile_edges(G, batch):  # noqa: F811
    import paper_2609_26108_amd as C
    p = random_params(16, 0.3)
    blob = new_blob(G, p)
    _fit_random_norm(G, blob, 7)
    rng = np.random.default_rng(batch)
    X = rng.normal(0.5, 2.0, (700, 16)).astype(np.float32)
    Y = rng.normal(0.3, 1.5, (700, 4)).astype(np.float32)
    idx = rng.choice(700, batch, replace=False).astype(np.int32)
    grad = torch.empty(S.N_PARAMS, dtype=torch.float32, device=G.DEV)
    loss = torch.empty(1, dtype=torch.float32, device=G.DEV)
    ws = torch.empty(C.chert_surrogate_grad_workspace_bytes(batch), dtype=torch.uint8, device=G.DEV)
    C.chert_surrogate_grad(blob, torch.from_numpy(X).to(G.DEV), torch.from_numpy(Y).to(G.DEV),
                           torch.from_numpy(idx).to(G.DEV), grad, loss, ws)
    torch.cuda.synchronize()
    g = grad.cpu().numpy().astype(np.float64)
    Le, ge = S.backward_bf16(p, *standardise(blob, X[idx], Y[idx]))
    assert abs(float(loss.item()) - Le) <= 1e-3 * Le
    off = 0
    for name, shp in S.SHAPES:
        k = int(np.prod(shp))
        a, b = g[off:off + k], ge[off:off + k].astype(np.float64)
        assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b), name
        off += k
