"""Operator apply in its forms (3D: directions in turn, lines of all directions at once on
small grids; 2D: a thread per node, lines on large grids) at the edges of its blocks: element counts that leave a ragged last
block, rows along direction 0 shorter than a block or cut by one, periodic and Dirichlet
ends (three, four and five elements around), every compiled order, 2D and 3D, against the
oracle's operator; and the V-cycle with the residual and restriction in one launch
against the two launches.

Tolerances: sums of at most 6 (P + 1) terms bounded by dim ||L|| ||M||^(dim-1) ||u||, to
1e-12 (FP64) and 2e-5 (FP32) of it; the fused restriction takes the same values in the
same order, 1e-13 (FP64) of the largest."""
import numpy as np
import pytest

import synth
from gpu_util import to_elem, to_lex
from oracle import multigrid as mg

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [((n, 3, 2), (per, per, False), 8) for n in (3, 4, 5) for per in (False, True)] + [
    ((1, 3, 2), False, 8), ((2, 3, 2), False, 8), ((3, 2, 3), (True, False, True), 8), ((7, 1, 1), (True, False, False), 8),
    ((1, 1, 1), False, 8), ((5, 3, 3), True, 4), ((3, 3, 4), True, 4), ((7, 5, 1), False, 6), ((4, 3, 3), True, 6),
    ((5, 7, 4), True, 2), ((3, 4, 3), True, 3), ((3, 3, 2), (True, True, False), 12), ((3, 1, 2), False, 12),
    ((2, 3, 1), (False, True, False), 16), ((1, 3, 2), False, 16), ((7, 5), True, 2), ((5, 3), False, 3), ((3, 7), True, 4),
    ((1, 1), False, 4), ((4, 5), True, 6), ((3, 5), True, 8), ((3, 2), False, 12), ((4, 3), True, 16),
    ((1, 3), (False, True), 32), ((3, 2), False, 32),
    # large enough for the directions in turn (3D) and for lines (2D) in both precisions
    ((3, 12, 11), True, 8), ((4, 10, 10), (True, False, True), 8), ((5, 9, 9), False, 8), ((1, 20, 20), False, 8),
    ((2, 14, 15), (False, True, True), 8), ((7, 8, 7), True, 8), ((9, 9, 10), (True, True, False), 6), ((13, 13, 13), True, 4),
    ((17, 16, 16), False, 3), ((22, 21, 22), True, 2), ((37, 38), False, 16), ((70, 71), True, 8), ((127, 126), False, 4),
]


@pytest.mark.parametrize("n, periodic, P", CASES)
def test_apply_forms(n, periodic, P, monkeypatch):
    print(f"[{n} periodic {periodic} P {P}]", flush=True)
    rng = np.random.default_rng(100 * P + n[0])
    per = periodic if isinstance(periodic, tuple) else (periodic,) * len(n)
    g = synth.Grid(len(n), tuple(rng.uniform(0.5, 1.5, k) for k in n), per)
    m = synth.Method(P=P, smoother="FA")
    H = mg.Hierarchy(g, m, assemble=False, coarse=False)
    S = D.Solver(g, m)
    try:
        for l, orders in enumerate(mg.level_orders(P)):
            u, f = rng.standard_normal(g.n_dof(orders)), rng.standard_normal(g.n_dof(orders))
            scale = max(np.abs(K).sum(axis=1).max() for M, K in H.levels[l].ops) \
                * max(np.abs(M).max() for M, K in H.levels[l].ops) ** (g.dim - 1) * g.dim * np.abs(u).max()
            ref = H.apply(l, u)
            for dt, tol in ((torch.float64, 1e-12), (torch.float32, 2e-5)):
                ud, fd = (torch.tensor(to_elem(v, g, orders), dtype=dt, device="cuda") for v in (u, f))
                Au = to_lex(S.apply(l, ud).double().cpu().numpy(), g, orders)
                assert np.abs(Au - ref).max() <= tol * scale, (l, dt)
                r = to_lex(S.residual(l, fd, ud).double().cpu().numpy(), g, orders)
                assert np.abs(r - (f - ref)).max() <= tol * (scale + np.abs(f).max()), (l, dt)
        r = torch.tensor(rng.standard_normal(g.n_dof(P)), device="cuda")
        z = S.vcycle(r - r.mean())
        monkeypatch.setenv("DGMG_NO_FUSED_RESTRICTION", "1")
        S2 = D.Solver(g, m)
        try:
            assert (S2.vcycle(r - r.mean()) - z).abs().max() <= 1e-13 * z.abs().max()
        finally:
            S2.close()
    finally:
        S.close()
