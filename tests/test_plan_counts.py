"""Launches per iteration that a planned batch reports (host only): the launches of the two
phases of an MGCG iteration, counted from the algorithm, without the ones of the solve's
start."""
import ctypes

import numpy as np
import pytest

import synth
from paper_1603_02524_amd import dgmg as D
from test_abi import _batch, _plan


# phase a: operator, x and r update, norm; phase b: V-cycle, z.r, direction update
@pytest.mark.parametrize("P, vcycle", [
    (1, 1),              # the coarse solve alone
    (2, 2 + 1 + 1 + 1 + 3),  # patch solve and sum; residual with restriction; coarse; prolongation; residual, solve, sum
])
@pytest.mark.parametrize("count", [1, 3])
def test_launches_per_iteration(P, vcycle, count):
    lib = D.load_library()
    rng = np.random.default_rng(count)
    g = synth.Grid(3, tuple(rng.uniform(0.5, 1.5, 3) for _ in range(3)), (False,) * 3)
    b, keep = _batch(lib, [(g, synth.Method(P=P, smoother="EA"))] * count)
    try:
        assert _plan(lib, b) == (1, 3 + vcycle + 2, 0)
    finally:
        lib.dgmg_batch_destroy(ctypes.c_void_p(b.value))
