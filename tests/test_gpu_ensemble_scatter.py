"""An ensemble's pool on both sides of the line where its scatter takes two particles per
thread (two passes of 2048 workgroups, 2^20 particles): every realization equals its plain
single context bit for bit."""
import numpy as np
import pytest

from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n0", [262_000, 264_001])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_pool_around_two_passes(precision, n0):
    from paper_2307_01797_amd import itokmc
    L = 40 * 5e-6
    cfgs = [workloads.preset("avalanche_32", grid=(40, 40, 40), dx=5e-6, E=(0.0, 0.0, 4e6), seed=3, realization=r,
                             precision=precision, seed_n0=n0, seed_centre=(L / 2, L / 2, L / 2),
                             seed_sigma=0.12 * L, steps=3, max_particles=2 * n0, stop_particles=0) for r in range(4)]
    ens = itokmc.Ensemble(4, 4 * 16 * 4096, 8 * n0, precision=precision)
    slots = [ens.admit(c, tag=i) for i, c in enumerate(cfgs)]
    ens.step(4)
    for c, slot in zip(cfgs, slots):
        sim = itokmc.Sim(c, precision=precision, max_particles=2 * n0)
        sim.seed()
        sim.step(3)
        a, b = ens.particles(slot), sim.particles()
        oa, ob = np.argsort(a[3]), np.argsort(b[3])
        for x, y in zip(a, b):
            assert np.array_equal(x[oa], y[ob])
        assert np.array_equal(ens.counts(slot, "plus"), sim.counts("plus"))
        sim.close()
