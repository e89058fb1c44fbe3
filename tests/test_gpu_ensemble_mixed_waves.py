"""Many small realizations in one ensemble: wavefronts of the push and spans of the KMC pass
that hold several realizations, a realization released among them, one that exceeds its
quota, workgroups of every size.  Every other realization equals the plain single context
bit for bit; the capped one keeps its charge."""
import numpy as np
import pytest

from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu


def _cfg(r):
    n0 = [3, 17, 64, 65, 200, 700, 1, 33][r % 8]
    e = [8, 12, 16, 20][r % 4]
    L = e * 5e-6
    return workloads.preset("avalanche_32", grid=(e, e + 1, e + 2), dx=5e-6, E=(0.0, 0.0, 1.1e7 + 2e5 * r),
                            seed=9, realization=r, precision="fp32", seed_n0=n0,
                            seed_centre=(L / 2, L / 2, L / 2), seed_sigma=0.2 * L, steps=14 + r % 5,
                            max_particles=4000, stop_particles=0)


@pytest.mark.parametrize("shape", [dict(), dict(push_block=64, kmc_block=64), dict(push_block=1024, kmc_block=128),
                                   dict(fused_per_cu=1)])
def test_mixed_wavefronts_match_plain(shape):
    from paper_2307_01797_amd import itokmc
    cfgs = [_cfg(r) for r in range(24)]
    cfgs[7].update(seed_n0=400, max_particles=430, steps=30)     # exceeds its quota
    ens = itokmc.Ensemble(32, 32 * 4 * 4096, 32 * 4000)
    if shape:
        ens.set_tuning(**shape)
    slots = [ens.admit(c, tag=i) for i, c in enumerate(cfgs)]
    ens.step(5)
    ens.release(slots[10])
    ens.step(40)
    ev = {e[2]: e for e in ens.poll()}
    assert ev[7][1] == itokmc.SLOT_CAPPED
    d7 = ens.result(slots[7])
    # every reaction conserves charge: sum(n+ - n_e - n-) = outflow - seeded electrons
    seeded = itokmc.Sim(cfgs[7], max_particles=4000)
    seeded.seed()
    assert d7["charge"] == d7["outflow_weight"] - seeded.diagnostics()["weight"]
    assert d7["n_particles"] <= 430
    for i, c in enumerate(cfgs):
        if i in (7, 10):
            continue
        assert ev[i][1] == itokmc.SLOT_DONE and ev[i][3] == c["steps"]
        sim = itokmc.Sim(c, max_particles=4000)
        sim.seed()
        sim.step(c["steps"])
        a, b = ens.particles(slots[i]), sim.particles()
        oa, ob = np.argsort(a[3]), np.argsort(b[3])
        for x, y in zip(a, b):
            assert np.array_equal(x[oa], y[ob]), i
        assert np.array_equal(ens.counts(slots[i], "plus"), sim.counts("plus"))
        assert np.array_equal(ens.counts(slots[i], "minus"), sim.counts("minus"))
        de, ds = ens.result(slots[i]), sim.diagnostics()
        for k in ("n_particles", "weight", "charge", "outflow_weight", "fires", "created", "removed_weight",
                  "particle_steps"):
            assert de[k] == ds[k], (i, k)
