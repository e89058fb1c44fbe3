"""One-workgroup levels at the edges of their launch forms: three cells of a colour per
thread (more than 2048 pairs), pairs along every axis (rows of one or three cells pair along
the longest axis instead of x), the largest count of pairs; bars as for the other levels."""
import numpy as np
import pytest

from test_gpu_levels import _transport

pytestmark = pytest.mark.gpu

GRIDS = [(7, 23, 25), (5, 27, 30), (3, 36, 37), (3, 131, 9), (3, 5, 41), (1, 90, 45), (1, 45, 90), (1, 3500, 1),
         (3, 1, 31), (1, 1, 64), (12, 148, 72)]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-8), ("fp32", 1e-6)])
def test_potential_matches_oracle(orc, grid, precision, tol):
    a, b = _transport(orc, grid, precision)
    assert np.abs(a - b).max() <= tol * np.abs(b).max()
