"""The PCG vector kernels at the edges of their block counts: grids below one block,
one unknown past a block, more unknowns than blocks x threads, more partial sums of p.q
than the update adds up itself, a zero right-hand side; alone (eager and replayed) and
in a batch, which must agree bitwise, and the true residual by the FP64 operator.

Tolerance: the solver confirms ||f - A x|| <= tol ||f|| with the same operator; another
order of the norm's sum moves it by at most n eps, 1e-9 relative here."""
import numpy as np
import pytest

import synth
from gpu_util import rand_grid

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu

# unknowns: 27, 225, 257 elements of 9, 343, 287500, 2100 elements of 27 with a zero rhs
GRIDS = [((1, 1, 1), 2), ((5, 5), 2), ((257, 1), 2), ((1, 1, 1), 6), ((100, 115), 4), ((15, 14, 10), 2)]
ZERO = 5


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_pcg_vectors(precision):
    probs = [(rand_grid(len(n), n, seed=60 + i), synth.Method(P=P, smoother="FA", precision=precision))
             for i, (n, P) in enumerate(GRIDS)]
    B = D.BatchSolver(probs)
    try:
        assert B.plan_info()[0] is True
        f_all = np.random.default_rng(8).uniform(-1, 1, B.n_dof)
        f_all[B.offsets[ZERO]:B.offsets[ZERO + 1]] = 0.0
        f_dev = torch.tensor(f_all, device="cuda")
        outs = []
        for rep in range(2):  # the second solve replays recorded phases
            B.use_graphs(rep == 1)
            x_all = torch.zeros(B.n_dof, dtype=torch.float64, device="cuda")
            stats = B.solve(f_dev, x_all)
            assert all(s["converged"] for s in stats)
            outs.append(x_all)
        assert torch.equal(outs[0], outs[1])
        for i, (g, m) in enumerate(probs):
            print(f"[{precision} {GRIDS[i]}]", flush=True)
            sl = slice(int(B.offsets[i]), int(B.offsets[i + 1]))
            fi, xb = f_dev[sl].clone(), outs[0][sl]
            S = D.Solver(g, m)
            try:
                for graphs in (False, True):
                    S.use_graphs(graphs)
                    x = torch.zeros_like(fi)
                    st = S.solve(fi, x)
                    assert st["converged"] and st["iterations"] == stats[i]["iterations"]
                    assert torch.equal(x, xb)
                if i == ZERO:
                    assert not x.any()
                    continue
                r = fi - S.apply(S.num_levels - 1, x)
                assert r.norm() <= st["r_true"] * (1 + 1e-6) + 1e-13 * fi.norm()
            finally:
                S.close()
    finally:
        B.close()
