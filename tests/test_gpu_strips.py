"""3D patch solves in strips of several patches (kernels_fdm3.hpp): one sweep at
grids whose patch counts give strips of 1, 2, 4 and 8 patches, with a ragged last
strip, every sweep normal, Dirichlet and periodic, against a separable sweep built
from the oracle's 1D patches (the same sum over patches, direction by direction).

Tolerances: FP64 1e-11 of the largest value (transforms of at most 16 terms in six
passes on a residual about 1e3 times the vector: a few hundred ulps), FP32 5e-4 as for
the smoothing steps of the other parity tests."""
import numpy as np
import pytest

import synth
from gpu_util import to_elem, to_lex
from oracle import multigrid as mg

torch = pytest.importorskip("torch")
from paper_1603_02524_amd import dgmg as D  # noqa: E402

pytestmark = pytest.mark.gpu


def _separable_sweep(H, u, f, normal):
    sm = H.levels[-1].smoother
    dim, shape = sm.grid.dim, sm.shape
    t = (f - H.apply(H.L, u)).reshape(shape)
    kinds = [("fc" if d == normal else "ec") for d in range(dim)]
    den = 0.0
    for d in range(dim):  # nodes -> (patch, mode), patch after patch
        patches = getattr(sm, kinds[d])[d]
        v = np.moveaxis(t, dim - 1 - d, 0)
        eig = [sm.eig1d(d, kinds[d], k) for k in range(len(patches))]
        v = np.concatenate([np.tensordot(S.T, v[p.idx], axes=(1, 0)) for p, (S, _) in zip(patches, eig)])
        t = np.moveaxis(v, 0, dim - 1 - d)
        sh = [1] * dim
        sh[dim - 1 - d] = -1
        den = den + np.concatenate([lam for _, lam in eig]).reshape(sh)
    t = t / den
    for d in range(dim):  # and back, weighted, summed over the patches of a node
        patches = getattr(sm, kinds[d])[d]
        v = np.moveaxis(t, dim - 1 - d, 0)
        out = np.zeros((shape[dim - 1 - d],) + v.shape[1:])
        at = 0
        for k, p in enumerate(patches):
            S, lam = sm.eig1d(d, kinds[d], k)
            out[p.idx] += p.w.reshape((-1,) + (1,) * (v.ndim - 1)) * np.tensordot(S, v[at:at + len(lam)], axes=(1, 0))
            at += len(lam)
        t = np.moveaxis(out, 0, dim - 1 - d)
    return u + t.reshape(-1)


# (elements, order, overlap, periodic): strips of 8 / 4 / 2 / 1 patches and ragged ends
CASES = [
    ((16, 17, 64), 2, "level", False), ((12, 9, 48), 2, "level", True),
    ((24, 9, 24), 4, "level", False), ((20, 10, 11), 4, "zero", True),
    ((24, 9, 28), 6, "level", False), ((12, 9, 16), 8, "level", False), ((13, 7, 17), 8, "level", True),
    ((5, 4, 3), 8, "level", False), ((3, 4, 3), 12, "level", True), ((2, 3, 2), 16, "level", False),
    ((9, 5, 31), 3, 2, False),
]


@pytest.mark.parametrize("n, P, overlap, periodic", CASES)
def test_sweep_matches_separable_oracle(n, P, overlap, periodic):
    print(f"[{n} P = {P} overlap {overlap} periodic {periodic}]", flush=True)
    rng = np.random.default_rng(P)
    g = synth.Grid(3, tuple(rng.uniform(0.5, 1.5, k) for k in n), (periodic,) * 3)
    m = synth.Method(P=P, smoother="FA", overlap=overlap)
    H = mg.Hierarchy(g, m, assemble=False, coarse=False)
    S = D.Solver(g, m)
    try:
        u, f = rng.standard_normal((2, g.n_dof(P)))
        for normal in (-1, 0, 1, 2):
            ref = _separable_sweep(H, u, f, normal)
            for dt, tol in ((torch.float64, 1e-11), (torch.float32, 5e-4)):
                ud = torch.tensor(to_elem(u, g, P), dtype=dt, device="cuda")
                S.sweep(H.L, ud, torch.tensor(to_elem(f, g, P), dtype=dt, device="cuda"), normal)
                got = to_lex(ud.double().cpu().numpy(), g, P)
                assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (normal, dt)
    finally:
        S.close()
