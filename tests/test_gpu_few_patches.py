"""2D patch solves of few patches (a thread per node) on both sides of the line to the form
on the matrix cores, every order's tile, each sweep normal, Dirichlet and periodic ends,
against the separable sweep built from the oracle's 1D patches; and in a batch of grids
that take both forms, bitwise the sweeps' results alone.

Tolerances as for the 3D strips: FP64 1e-11, FP32 5e-4 of the largest value."""
import numpy as np
import pytest

import synth
from gpu_util import to_elem, to_lex
from oracle import multigrid as mg
from test_gpu_strips import _separable_sweep

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    ((1, 1), 2, "level", False), ((5, 3), 2, "level", True), ((4, 3), 3, 1, False), ((3, 5), 4, "level", (True, False)),
    ((4, 4), 6, "level", False), ((3, 4), 8, "level", True), ((5, 2), 12, "level", False), ((3, 3), 16, "level", True),
    ((16, 16), 16, "level", False), ((23, 24), 16, "level", False), ((33, 36), 8, "level", True), ((1, 2), 32, "level", False),
]


@pytest.mark.parametrize("n, P, overlap, periodic", CASES)
def test_few_patches(n, P, overlap, periodic):
    print(f"[{n} P = {P} overlap {overlap} periodic {periodic}]", flush=True)
    rng = np.random.default_rng(P)
    per = periodic if isinstance(periodic, tuple) else (periodic,) * 2
    g = synth.Grid(2, tuple(rng.uniform(0.5, 1.5, k) for k in n), per)
    m = synth.Method(P=P, smoother="FA", overlap=overlap)
    H = mg.Hierarchy(g, m, assemble=False, coarse=False)
    S = D.Solver(g, m)
    try:
        u, f = rng.standard_normal((2, g.n_dof(P)))
        for normal in (-1, 0, 1):
            ref = _separable_sweep(H, u, f, normal)
            for dt, tol in ((torch.float64, 1e-11), (torch.float32, 5e-4)):
                ud = torch.tensor(to_elem(u, g, P), dtype=dt, device="cuda")
                S.sweep(H.L, ud, torch.tensor(to_elem(f, g, P), dtype=dt, device="cuda"), normal)
                got = to_lex(ud.double().cpu().numpy(), g, P)
                assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (normal, dt)
    finally:
        S.close()


def test_batch_takes_each_grids_form():
    rng = np.random.default_rng(4)
    probs = [(synth.Grid(2, tuple(rng.uniform(0.5, 1.5, k) for k in n), (False,) * 2), synth.Method(P=8, smoother="EA"))
             for n in ((4, 3), (40, 41), (16, 16), (33, 34))]
    B = D.BatchSolver(probs)
    try:
        assert B.plan_info()[0] is True
        f = torch.tensor(rng.uniform(-1, 1, B.n_dof), device="cuda")
        xb = torch.zeros_like(f)
        B.solve(f, xb)
        for i, (g, m) in enumerate(probs):
            sl = slice(int(B.offsets[i]), int(B.offsets[i + 1]))
            S = D.Solver(g, m)
            try:
                x = torch.zeros_like(f[sl])
                S.solve(f[sl].clone(), x)
                assert torch.equal(x, xb[sl]), i
            finally:
                S.close()
    finally:
        B.close()
