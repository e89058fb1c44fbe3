"""The two forms of the particle move (scatter; place and gather above 2^24 particles) give
the same particles: a seed just above the line and one just below it share their ids, and
with no reactions a particle's state after two steps depends on its id alone (bit for
bit).  Counts that leave a ragged last chunk, and dead slots from outflow."""
import numpy as np
import pytest

from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu


def _run(n0, precision, steps):
    from paper_2307_01797_amd import itokmc
    g = (96, 80, 72)
    cfg = workloads.preset("avalanche_32", grid=g, dx=4e-6, seed_n0=n0, seed_sigma=90e-6,
                           seed_centre=tuple(0.5 * a * 4e-6 for a in g), precision=precision)
    cfg["coeffs"].update(alpha_A=0.0, eta=0.0)
    sim = itokmc.Sim(cfg, max_particles=21_000_000)
    sim.seed()
    live = sim.diagnostics()["n_particles"]
    sim.step(steps)
    d = sim.diagnostics()
    assert d["n_particles"] + d["outflow_weight"] == live and d["outflow_weight"] > 0
    cell, off, w, ids = sim.particles()
    assert np.all(w == 1) and np.array_equal(np.bincount(cell, minlength=sim.ncell).astype(np.uint32),
                                             sim.deposit("ngp"))
    i = ids.astype(np.int64) - (1 << 61)
    full = np.full((n0, 4), -1.0)
    full[i, 0] = cell
    full[i, 1:] = off
    assert (full[:, 0] >= 0).sum() == len(ids)  # ids unique
    return live, full


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_gather_equals_scatter(precision):
    above, a = _run(22_400_123, precision, 2)  # about 17.8e6 inside the box
    below, b = _run(14_000_001, precision, 2)
    assert above > (1 << 24) + 100_000 and below < (1 << 24)
    assert np.array_equal(a[:len(b)], b)
