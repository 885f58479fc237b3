"""Operator on 3D grids on both sides of the sizes where the lines of all directions at once
give way to the directions in turn, and beyond them at element counts whose blocks cut, fill
and span rows, FP64 and FP32: the checks of the forms."""
import pytest

torch = pytest.importorskip("torch")
from test_gpu_apply_forms import test_apply_forms as _check  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    ((6, 6, 7), False, 8), ((8, 8, 8), True, 8), ((8, 8, 9), (False, True, False), 8),
    ((3, 13, 14), True, 8), ((4, 12, 12), (True, False, True), 8), ((5, 10, 11), False, 8), ((1, 24, 24), False, 8),
    ((2, 16, 17), (False, True, True), 8), ((7, 9, 9), True, 8), ((8, 8, 9), False, 6), ((9, 8, 9), True, 6),
    ((11, 11, 10), False, 4), ((13, 13, 13), True, 3), ((14, 13, 14), False, 3), ((18, 18, 18), True, 2),
]


@pytest.mark.parametrize("n, periodic, P", CASES)
def test_sizes(n, periodic, P, monkeypatch):
    _check(n, periodic, P, monkeypatch)
