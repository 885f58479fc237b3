"""Overlap summation (lines of nodes along one direction, whole blocks of lines) at its
edges: one element, layers of exactly one block of lines, one line more and less, mixed
periodic directions, every overlap from none to half an element, tiles stored either
way (P = 32: direction 2 slowest), and three covering patches (the general form), against
the separable sweep built from the oracle's 1D patches.

Tolerances as for the strips: FP64 1e-11, FP32 5e-4 of the largest value; P = 32: the
transforms have 64 terms, 1e-10 and 5e-3."""
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
    ((1, 1, 1), 2, "level", False), ((1, 1, 1), 8, "level", False), ((4, 3, 4), 3, "level", False),
    ((4, 2, 5), 3, 2, False), ((5, 3, 3), 3, 1, False), ((4, 4, 3), 4, "zero", (True, False, True)),
    ((3, 3, 5), 6, "level", (False, True, False)), ((3, 5, 3), 8, "level", (True, False, True)),
    ((2, 1, 2), 12, "level", False), ((1, 3, 1), 16, "level", (False, True, False)), ((1, 2, 1), 32, "level", False),
]


@pytest.mark.parametrize("n, P, overlap, periodic", CASES)
def test_overlap_sums(n, P, overlap, periodic):
    print(f"[{n} P = {P} overlap {overlap} periodic {periodic}]", flush=True)
    rng = np.random.default_rng(P)
    per = periodic if isinstance(periodic, tuple) else (periodic,) * 3
    g = synth.Grid(3, tuple(rng.uniform(0.5, 1.5, k) for k in n), per)
    m = synth.Method(P=P, smoother="FA", overlap=overlap)
    H = mg.Hierarchy(g, m, assemble=False, coarse=False)
    S = D.Solver(g, m)
    f64, f32 = (1e-11, 5e-4) if P < 32 else (1e-10, 5e-3)
    try:
        u, f = rng.standard_normal((2, g.n_dof(P)))
        for normal in (-1, 0, 1, 2):
            ref = _separable_sweep(H, u, f, normal)
            for dt, tol in ((torch.float64, f64), (torch.float32, f32)):
                ud = torch.tensor(to_elem(u, g, P), dtype=dt, device="cuda")
                S.sweep(H.L, ud, torch.tensor(to_elem(f, g, P), dtype=dt, device="cuda"), normal)
                got = to_lex(ud.double().cpu().numpy(), g, P)
                assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (normal, dt)
    finally:
        S.close()
