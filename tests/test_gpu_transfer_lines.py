"""3D transfers at orders from 12 on (a thread per line): one element, odd counts and more
blocks than CUs, both precisions, against the oracle's transfers.

Tolerances: three contractions of at most P + 1 terms each, 1e-13 (FP64) and 2e-6 (FP32)
of the largest value per term and contraction, 3 P of them."""
import numpy as np
import pytest

import synth
from gpu_util import to_elem, to_lex
from oracle import multigrid as mg

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, P", [((1, 1, 1), 12), ((1, 1, 1), 16), ((3, 1, 2), 16), ((3, 5, 1), 12), ((7, 7, 6), 12)])
def test_transfer_lines(n, P):
    print(f"[{n} P {P}]", flush=True)
    rng = np.random.default_rng(P)
    g = synth.Grid(3, tuple(rng.uniform(0.5, 1.5, k) for k in n), (False,) * 3)
    m = synth.Method(P=P, smoother="FA")
    H = mg.Hierarchy(g, m, assemble=False, coarse=False)
    S = D.Solver(g, m)
    L = H.L
    try:
        r, uc, u = (rng.standard_normal(g.n_dof(q)) for q in (P, P // 2, P))
        rc, pu = H.restrict(L, r), H.prolong(L, uc)
        for dt, tol in ((torch.float64, 1e-13), (torch.float32, 2e-6)):
            dev = lambda v, q: torch.tensor(to_elem(v, g, q), dtype=dt, device="cuda")  # noqa: E731
            got = to_lex(S.restrict(L, dev(r, P)).double().cpu().numpy(), g, P // 2)
            assert np.abs(got - rc).max() <= tol * 3 * P * np.abs(rc).max()
            ud = dev(u, P)
            S.prolong(L, dev(uc, P // 2), ud)
            got = to_lex(ud.double().cpu().numpy(), g, P)
            assert np.abs(got - (u + pu)).max() <= tol * 3 * P * np.abs(pu).max()
    finally:
        S.close()
