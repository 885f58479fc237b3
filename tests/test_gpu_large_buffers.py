"""Overlap sums whose patch buffer passes 4 GiB, where the lines of nodes run along direction
2, over strips: vectors periodic with period 16 elements on a large periodic grid give the
tiled result of the 16-element grid, whose sums take the usual form.  Elements of equal size,
so both grids hold the same matrices up to rounding.

Tolerance: FP64 1e-11 of the largest value as for the other sweeps."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu


def test_sweeps_beyond_4_gib():
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    n, rep = 16, 4
    m = synth.Method(P=8, smoother="FA")
    S, B = (D.Solver(synth.Grid(3, (np.full(k, 1.0 / 64),) * 3, (True,) * 3), m) for k in (n, n * rep))
    try:
        gen = torch.Generator(device="cuda").manual_seed(1)
        u, f = torch.rand(2, S.n_dof(), generator=gen, device="cuda", dtype=torch.float64)

        def tiled(v):
            return v.view(n, n, n, -1).repeat(rep, rep, rep, 1).reshape(-1)

        fb = tiled(f)
        for normal in (0, 1, 2):
            a, b = u.clone(), tiled(u)
            S.sweep(S.num_levels - 1, a, f, normal)
            B.sweep(B.num_levels - 1, b, fb, normal)
            assert (b - tiled(a)).abs().max().item() <= 1e-11 * a.abs().max().item(), normal
    finally:
        S.close()
        B.close()
