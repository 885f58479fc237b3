"""Coarse solves on both sides of the lines between their forms (one block, planes, a launch
per direction and way, with or without means): the forms give the same bits, so a batch whose
grids share one launch of blocks gives what each grid gives alone in the form that its size
takes, and both match the oracle's operator as in the tests of the forms."""
import numpy as np
import pytest

import synth
from gpu_util import to_elem, to_lex
from oracle import multigrid as mg

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu

# elements: one block / passes (2D and periodic), one block / planes / passes (3D), all within a
# block's LDS
SETS = [
    ([(22, 22), (24, 24), (26, 27), (34, 33), (60, 8)], False),
    ([(22, 22), (24, 24), (26, 27), (34, 33), (8, 60)], True),
    ([(7, 5, 6), (8, 8, 9), (10, 10, 10), (2, 2, 60), (30, 4, 4)], False),
    ([(7, 5, 6), (8, 8, 9), (10, 9, 10), (3, 3, 20), (30, 4, 4)], True),
]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes, periodic", SETS)
def test_batch_equals_grids_alone(sizes, periodic, precision):
    rng = np.random.default_rng(len(sizes[0]))
    dim = len(sizes[0])
    probs = [(synth.Grid(dim, tuple(rng.uniform(0.5, 1.5, k) for k in n), (periodic,) * dim),
              synth.Method(P=2, smoother="EA", precision=precision)) for n in sizes]
    B = D.BatchSolver(probs, max_iter=3)
    try:
        assert B.plan_info()[0] is True
        f = torch.zeros(B.n_dof, dtype=torch.float64, device="cuda")
        for i in range(len(probs)):
            sl = slice(B.offsets[i], B.offsets[i + 1])
            f[sl] = torch.tensor(rng.uniform(-1, 1, sl.stop - sl.start), device="cuda")
            if periodic:
                f[sl] -= f[sl].mean()
        xb = torch.zeros_like(f)
        B.solve(f, xb, tol=1e-12)
        for i, (g, m) in enumerate(probs):
            sl = slice(B.offsets[i], B.offsets[i + 1])
            S = D.Solver(g, m, max_iter=3)
            try:
                x = torch.zeros_like(f[sl])
                S.solve(f[sl].clone(), x, tol=1e-12)
                assert torch.equal(x, xb[sl]), sizes[i]
            finally:
                S.close()
    finally:
        B.close()


@pytest.mark.parametrize("n, periodic", [(n, p) for sizes, p in SETS for n in sizes] + [
    ((16, 16, 17), False), ((17, 17, 17), False), ((4, 4, 36), False), ((3, 3, 60), False)])
def test_defining_equation(n, periodic):
    """As for the forms: backward error 1e-12 of ||A|| ||u|| + ||f||."""
    rng = np.random.default_rng(n[0])
    g = synth.Grid(len(n), tuple(rng.uniform(0.5, 1.5, k) for k in n), (periodic,) * len(n))
    H = mg.Hierarchy(g, synth.Method(P=2, smoother="EA"), assemble=False, coarse=False)
    S = D.Solver(g, synth.Method(P=2, smoother="EA"))
    try:
        f = rng.standard_normal(g.n_dof(1))
        u = to_lex(S.coarse_solve(torch.tensor(to_elem(f, g, 1), device="cuda")).cpu().numpy(), g, 1)
        if periodic:
            f = f - f.mean()
            assert abs(u.mean()) <= 1e-12 * np.abs(u).max()
        scale = max(np.abs(L).sum(axis=1).max() * np.abs(M).max() ** (g.dim - 1) for M, L in H.levels[0].ops)
        bound = 1e-12 * (g.dim * scale * np.abs(u).max() + np.abs(f).max())
        assert np.abs(H.apply(0, u) - f).max() <= bound
    finally:
        S.close()
