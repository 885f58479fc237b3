"""The autotuner chooses among block shapes only where the patch solve's kernel takes more
than one; elsewhere it reports the shape that the kernel is built for, whatever the timer
says.  Where there is a choice, every imposed shape gives the same bits."""
import numpy as np
import pytest

import synth
from gpu_util import rand_grid

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu


# wavefronts: 3D strips 4, tiles of more than 50 KB 8 (P = 16), stages through global memory 4
# (P = 32); 2D, a thread per node of 5 x 5 (P = 2), 9 x 9 (4), 13 x 13 (8): 1, 2, 3
@pytest.mark.parametrize("n, P, smoother, waves", [
    ((3, 4, 2), 8, "FA", [4, 4, 4]), ((2, 1, 2), 16, "FA", [4, 4, 4, 8]), ((3, 3, 3), 6, "EA", [4, 4]),
    ((1, 1, 1), 32, "EA", [4, 4, 4, 8, 4]), ((5, 4), 8, "EA", [1, 2, 3]),
])
def test_one_shape(n, P, smoother, waves):
    S = D.Solver(rand_grid(len(n), n, seed=P), synth.Method(P=P, smoother=smoother))
    try:
        tune = S.autotune()
        kinds = [3] if smoother == "EA" else list(range(len(n)))
        assert {k: w for k, (w, ms) in tune.items()} == {(l + 1, k): w for l, w in enumerate(waves) for k in kinds}
        assert all(ms > 0 for _, ms in tune.values())
    finally:
        S.close()


@pytest.mark.parametrize("n, P", [((14, 12, 15), 3), ((40, 42), 8)])
def test_choice(n, P):
    g = rand_grid(len(n), n, seed=3)
    S = D.Solver(g, synth.Method(P=P, smoother="EA"), max_iter=2)
    try:
        f = torch.tensor(np.random.default_rng(1).uniform(-1, 1, S.n_dof()), device="cuda")
        ref = torch.zeros_like(f)
        S.solve(f, ref)
        top = (S.num_levels - 1, 3)
        assert S.autotune()[top][0] in (1, 2, 4, 8)
        for w in (0, 1, 2, 4, 8):
            S.set_tuning(*top, w)
            x = torch.zeros_like(f)
            S.solve(f, x)
            assert torch.equal(x, ref), w
    finally:
        S.close()
