"""Merging of cells some of whose offsets are negative zeros, which set_particles takes
(they are not below zero): a negative zero is a zero in the extents that choose the split
axis and in the order along it.  Zeros of both signs in a third of the coordinates and in
every coordinate of one axis; against the oracle, bars as for the other ties."""
import numpy as np
import pytest

from test_gpu_merge_ties import COUNTS, _react
from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ppc", [32, 64])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["scattered", "one axis"])
def test_negative_zero(orc, kind, precision, n_ppc):
    rng = np.random.default_rng(29)
    counts = np.array(COUNTS + [700, 900])
    cfg = workloads.preset("avalanche_32", grid=(6, 6, 4), n_ppc=n_ppc, precision=precision)
    cfg["coeffs"].update(alpha_A=0.0, eta=0.0)
    cell = np.repeat(np.arange(len(counts)) * 6 + 1, counts)
    n = len(cell)
    off = rng.random((n, 3)).astype(np.float32).astype(np.float64)
    zero = rng.random((n, 3)) < 0.3
    if kind == "one axis":
        zero = np.zeros((n, 3), dtype=bool)
        zero[np.arange(n), cell // 6 % 3] = True
    off[zero] = np.where(rng.random(int(zero.sum())) < 0.5, 0.0, -0.0)
    assert np.signbit(off).any()
    w = np.where(rng.random(n) < 0.5, 1, rng.integers(1, 300, n)).astype(np.uint32)
    d = _react(orc, cfg, cell, off, w, rng.permutation(n).astype(np.uint64), precision)
    assert d["merged_cells"] > 0
