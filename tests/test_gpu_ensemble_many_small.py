"""Realizations of a few electrons: wavefronts of the push that hold up to 64 of them.  Each
equals its plain single context bit for bit, and a step of 1024 realizations of one electron
costs about what one of sixteen times the particles costs (both are launches of a few
microseconds; a push that takes a wavefront's realizations one after another needs twice
the time)."""
import time

import numpy as np
import pytest

from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu


def _cfg(r, n0, E, steps, precision="fp32"):
    L = 16 * 5e-6
    return workloads.preset("avalanche_32", grid=(16, 16, 16), dx=5e-6, E=(0.0, 0.0, E), seed=5, realization=r,
                            precision=precision, seed_n0=n0, seed_centre=(L / 2, L / 2, L / 2),
                            seed_sigma=0.4 * L, steps=steps, max_particles=64 + 4 * n0, stop_particles=0)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_few_electrons_match_plain(precision):
    from paper_2307_01797_amd import itokmc
    # a realization's electrons leave the grid, multiply, or both; every fourth stops early
    cfgs = [_cfg(r, 1 + r % 3, 9e6 + 1e4 * r, 8 if r % 4 == 3 else 20, precision) for r in range(200)]
    ens = itokmc.Ensemble(256, 256 * 4096, 256 * 128, precision=precision)
    slots = [ens.admit(c, tag=i) for i, c in enumerate(cfgs)]
    ens.step(25)
    left = 0
    for i, c in enumerate(cfgs):
        sim = itokmc.Sim(c, precision=precision, max_particles=256)
        sim.seed()
        sim.step(c["steps"])
        de, ds = ens.result(slots[i]), sim.diagnostics()
        for k in ("n_particles", "weight", "charge", "outflow_weight", "fires", "created", "removed_weight",
                  "particle_steps"):
            assert de[k] == ds[k], (i, k)
        left += ds["outflow_weight"]
        a, b = ens.particles(slots[i]), sim.particles()
        oa, ob = np.argsort(a[3]), np.argsort(b[3])
        for x, y in zip(a, b):
            assert np.array_equal(x[oa], y[ob]), i
        sim.close()
    assert left > 0


def test_a_step_does_not_go_realization_by_realization():
    import torch
    from paper_2307_01797_amd import itokmc
    best = {}
    for n0 in (1, 16):
        ens = itokmc.Ensemble(1024, 1024 * 4096, 1024 * 256)
        for r in range(1024):
            ens.admit(_cfg(r, n0, 3e6, 100000), tag=r)
        ens.step(10)
        torch.cuda.synchronize()
        t = []
        for _ in range(5):
            t0 = time.perf_counter()
            ens.step(50)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        best[n0] = min(t)
        ens.close()
    assert best[1] < 1.5 * best[16], best
