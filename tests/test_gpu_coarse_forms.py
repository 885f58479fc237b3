"""Exact coarse solve at the sizes where its form changes (one block in LDS, planes and
columns, one launch per pass), 2D and 3D, Dirichlet, mixed and periodic, against the
defining equation with the oracle's operator: A_0 u = f (f less its mean and u
mean-free on fully periodic grids).

Tolerance: backward error of sums of at most G terms in six passes, 1e-12 of
||A|| ||u|| + ||f|| per entry norm."""
import numpy as np
import pytest

import synth
from gpu_util import to_elem, to_lex
from oracle import multigrid as mg

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    ((1, 1, 1), False), ((7, 5, 6), False), ((9, 9, 10), False), ((3, 4, 3), True), ((8, 11, 9), True),
    ((13, 11, 7), False), ((12, 13, 11), False), ((40, 3, 4), False), ((3, 2, 60), False), ((12, 12, 13), True),
    ((11, 14, 12), (True, False, True)), ((1, 2), False), ((16, 16), True), ((45, 44), False), ((61, 50), False),
    ((52, 51), True),
]


@pytest.mark.parametrize("n, periodic", CASES)
def test_coarse_forms(n, periodic):
    print(f"[{n} periodic {periodic}]", flush=True)
    rng = np.random.default_rng(len(n) + n[0])
    per = periodic if isinstance(periodic, tuple) else (periodic,) * len(n)
    g = synth.Grid(len(n), tuple(rng.uniform(0.5, 1.5, k) for k in n), per)
    H = mg.Hierarchy(g, synth.Method(P=2, smoother="EA"), assemble=False, coarse=False)
    S = D.Solver(g, synth.Method(P=2, smoother="EA"))
    try:
        f = rng.standard_normal(g.n_dof(1))
        u = to_lex(S.coarse_solve(torch.tensor(to_elem(f, g, 1), device="cuda")).cpu().numpy(), g, 1)
        if all(per):
            f = f - f.mean()
            assert abs(u.mean()) <= 1e-12 * np.abs(u).max()
        scale = max(np.abs(L).sum(axis=1).max() * np.abs(M).max() ** (g.dim - 1) for M, L in H.levels[0].ops)
        bound = 1e-12 * (g.dim * scale * np.abs(u).max() + np.abs(f).max())
        assert np.abs(H.apply(0, u) - f).max() <= bound
        u32 = S.coarse_solve(torch.tensor(to_elem(f, g, 1), dtype=torch.float32, device="cuda"))
        assert np.abs(to_lex(u32.double().cpu().numpy(), g, 1) - u).max() <= 1e-5 * np.abs(u).max()
    finally:
        S.close()
