"""Restriction from a level in segments whose count of coarse segments is no multiple of a
wavefront: a tiled coarse level, a coarse level in segments itself, split and natural
order; bars as for the other levels."""
import numpy as np
import pytest

from test_gpu_levels import _transport

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,precision,tol", [((72, 88, 56), "fp32", 1e-6), ((72, 104, 88), "fp64", 1e-8)])
def test_ragged_segment_restriction(orc, grid, precision, tol):
    a, b = _transport(orc, grid, precision)
    assert np.abs(a - b).max() <= tol * np.abs(b).max()


def test_two_levels_in_segments():
    a = _transport(None, (176, 208, 80), "fp32")
    b = _transport(None, (176, 208, 80), "fp32", fine_layout=1)
    assert np.abs(a - b).max() <= 1e-6 * np.abs(b).max()
