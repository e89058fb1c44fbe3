"""The KMC's early exit of a quiet step (the hardware logarithm of the first word compared
with a widened threshold) against the oracle, where it can go wrong: rates chosen so that
the first waiting time ends within 1e-12 to 1e-3 of the end of the step on either side,
step counts around the batch of first words, and reactors of every kind in one wavefront.
All results are integers and must be equal.  (A relative distance of 1e-12 is far above
the 1e-15 by which two correctly working double logarithms and divisions may differ.)
"""
import numpy as np
import pytest

from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu

DT = 1e-12


def _sim(**over):
    from paper_2307_01797_amd import itokmc
    return itokmc.Sim(dict(workloads.REACTOR_A, **over), max_particles=1024)


def test_waiting_time_near_the_end_of_the_step(orc):
    cfg = dict(workloads.REACTOR_A)
    n, step = 4096, 3
    ids = np.arange(n, dtype=np.uint32)
    TAG_KMC = 3
    x = orc.philox_many(np.stack([ids, 0 * ids, np.full_like(ids, step), np.full_like(ids, TAG_KMC << 24)], 1),
                        (cfg["seed"], cfg["realization"]))[:, 0]
    L = -np.log((x.astype(np.float64) + 1.0) * 2.0 ** -32)
    d = np.array([1e-12, 1e-9, 1e-7, 1e-6, 1e-5, 5e-5, 1e-4, 2e-4, 1e-3])
    delta = np.concatenate([d, -d])[np.arange(n) % 18]
    A = L / DT * (1.0 + delta)
    use = A * DT <= 1.0
    k = np.zeros((n, 3))
    k[:, 0] = np.where(use, 0.7 * A, 1e9)
    k[:, 1] = np.where(use, 0.3 * A, 1e8)
    X = np.zeros((n, 4), dtype=np.int64)
    X[:, 0] = 1
    Xo, Fo = orc.kmc_cells(cfg, X, k, DT, step)
    assert use.sum() > 2000 and 0.3 < (Fo[use].sum(1) > 0).mean() < 0.7
    sim = _sim()
    Xg, Fg = sim.kmc_cells(X, k, DT, step)
    assert np.array_equal(Xg, Xo) and np.array_equal(Fg, Fo)
    Xr, Fr = sim.kmc_run(X, k, DT, step, 1)
    assert np.array_equal(Xr, Xo) and np.array_equal(Fr, Fo)


@pytest.mark.parametrize("steps", [1, 7, 8, 9, 25])
@pytest.mark.parametrize("over", [{}, dict(kmc_eps=0.05), dict(kmc="pure_tau")])
def test_reactor_batches_match_oracle_step_by_step(orc, steps, over):
    cfg = dict(workloads.REACTOR_A, **over)
    rng = np.random.default_rng(5)
    n = 257
    X = np.zeros((n, 4), dtype=np.int64)
    X[:, 0] = rng.choice([0, 1, 3, 20, 70, 400, 5000], n)
    X[:, 1] = rng.integers(0, 50, n)
    X[:, 2] = rng.integers(0, 50, n)
    k = np.zeros((n, 5))
    k[:, 0] = rng.choice([0.0, 1e9, 1.3e10, 1e12], n)
    k[:, 1] = rng.choice([0.0, 4e8, 3e11], n)
    k[:, 2] = rng.choice([0.0, 8e8], n)
    five = rng.random(n) < 0.2
    k[five, 3] = 1e7
    k[five, 4] = 1e6
    Xo, Fo = X.copy(), np.zeros((n, 5), dtype=np.int64)
    for s in range(steps):
        Xo, f = orc.kmc_cells(cfg, Xo, k, DT, 11 + s)
        Fo += f
    Xg, Fg = _sim(**over).kmc_run(X, k, DT, 11, steps)
    assert np.array_equal(Xg, Xo) and np.array_equal(Fg, Fo)
