"""MLP kernels at the edges of their tiles: forward blocks of 16 samples, gradient
tiles of 64 samples, and the batch sizes where the number of partial gradients
changes (one chunk up to 72 samples, as many as the scratch holds beyond).

Tolerance: FP32 sums of B (gradient) or 64 (forward) terms of O(1) against the
FP64 oracle on the same rounded inputs, as in the other MLP tests."""
import numpy as np
import pytest

from oracle import mlp as omlp

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 36, 37, 63, 64, 65, 72, 73, 128, 129, 1000, 4099])
def test_forward_and_gradient_at_tile_edges(B):
    print(f"[B = {B}]", flush=True)
    rng = np.random.default_rng(B)

    def rounded(a):
        return np.asarray(a, dtype=np.float32).astype(np.float64)

    p = rounded(omlp.init(7) + 0.05 * rng.standard_normal(omlp.N_PARAMS))
    X, T = rounded(rng.standard_normal((B, omlp.D_IN))), rounded(rng.standard_normal((B, omlp.D_OUT)))
    pd, Xd, Td = (torch.tensor(a.astype(np.float32), device="cuda") for a in (p, X, T))
    Y, work = D.mlp_forward(pd, Xd)
    ref, (_, h1, h2) = omlp.forward(p, X)
    assert np.allclose(Y.double().cpu().numpy(), ref, rtol=1e-5, atol=1e-5)
    w = work.double().cpu().numpy()
    assert np.allclose(w[:, :64], h1, atol=1e-6) and np.allclose(w[:, 64:], h2, atol=1e-6)
    g = D.mlp_backward(pd, Xd, Td, Y, work).double().cpu().numpy()
    gref = omlp.grad(p, X, T)
    assert np.abs(g - gref).max() <= 2e-5 * np.abs(gref).max() + 1e-7
