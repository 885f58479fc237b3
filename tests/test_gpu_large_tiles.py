"""Patch tiles at the limit of the LDS: P = 32 without overlap, whose element-centred FP32
tile (33 x 33 x 33) is solved in LDS with its matrices beside it while the FP64 one and the
face-centred tiles go through global memory, one sweep of each kind against the separable
sweep built from the oracle's 1D patches, and the FP32 V-cycle that smooths on that tile.

Tolerances as for the other P = 32 sweeps (transforms of 64 terms): FP64 1e-10, FP32 5e-3
of the largest value."""
import numpy as np
import pytest

import synth
from gpu_util import to_elem, to_lex
from oracle import multigrid as mg
from test_gpu_strips import _separable_sweep

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu


def _problem(n, periodic, smoother, **kw):
    rng = np.random.default_rng(32)
    g = synth.Grid(3, tuple(rng.uniform(0.5, 1.5, k) for k in n), periodic)
    return g, synth.Method(P=32, smoother=smoother, overlap="zero", **kw), rng


@pytest.mark.parametrize("n, periodic", [((1, 2, 1), (False,) * 3), ((1, 1, 3), (False, False, True))])
def test_sweeps_without_overlap(n, periodic):
    print(f"[{n} periodic {periodic}]", flush=True)
    g, m, rng = _problem(n, periodic, "FA")
    H = mg.Hierarchy(g, m, assemble=False, coarse=False)
    S = D.Solver(g, m)
    try:
        u, f = rng.standard_normal((2, g.n_dof(32)))
        for normal in (-1, 0, 1, 2):
            ref = _separable_sweep(H, u, f, normal)
            for dt, tol in ((torch.float64, 1e-10), (torch.float32, 5e-3)):
                print(f"  normal {normal} {dt}", flush=True)
                ud = torch.tensor(to_elem(u, g, 32), dtype=dt, device="cuda")
                S.sweep(H.L, ud, torch.tensor(to_elem(f, g, 32), dtype=dt, device="cuda"), normal)
                got = to_lex(ud.double().cpu().numpy(), g, 32)
                assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (normal, dt)
    finally:
        S.close()


def test_mixed_vcycle_without_overlap():
    """The FP32 V-cycle that smooths on the FP32 tile against the FP64 handle's."""
    g, m, rng = _problem((2, 1, 2), (False,) * 3, "EA")
    z = {}
    r = torch.tensor(rng.uniform(-1.0, 1.0, g.n_dof(32)), device="cuda")
    for precision, dt in (("fp64", torch.float64), ("mixed", torch.float32)):
        S = D.Solver(g, synth.Method(P=32, smoother="EA", overlap="zero", precision=precision))
        try:
            z[precision] = S.vcycle(r.to(dt)).double().cpu().numpy()
        finally:
            S.close()
    assert np.abs(z["mixed"] - z["fp64"]).max() <= 5e-3 * np.abs(z["fp64"]).max()
