"""Seeding, per-cell queries and reductions at the sizes where their workgroup and wavefront
forms can go wrong: counts around a wavefront, a workgroup's draws and a bank's capacity;
density and weights of sorted, scattered and mixed particles, against plain numpy sums
(double sums of at most a few thousand terms per cell: 1e-12 of the cell's value) and
against the oracle's seeds (integers exact, offsets 1e-12)."""
import numpy as np
import pytest

from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu


def _axis(x, n, tsc):
    if tsc:
        j = np.floor(x).astype(np.int64)
        d = x - j - 0.5
        return [(np.clip(j - 1, 0, n - 1), 0.5 * (0.5 - d) ** 2), (j, 0.75 - d * d),
                (np.clip(j + 1, 0, n - 1), 0.5 * (0.5 + d) ** 2)]
    lo = np.floor(x - 0.5)
    f = x - 0.5 - lo
    lo = lo.astype(np.int64)
    return [(np.clip(lo, 0, n - 1), 1.0 - f), (np.clip(lo + 1, 0, n - 1), f)]


def _density(g, ijk, off, w, dV, tsc):
    out = np.zeros(np.prod(g))
    ax = [_axis(ijk[:, a] + off[:, a], g[a], tsc) for a in range(3)]
    for ix, wx in ax[0]:
        for iy, wy in ax[1]:
            for iz, wz in ax[2]:
                out += np.bincount(ix + g[0] * (iy + g[1] * iz), weights=w * wx * wy * wz / dV, minlength=len(out))
    return out


@pytest.mark.parametrize("shape", ["cic", "tsc"])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,spread", [(1, "sorted"), (63, "scattered"), (257, "sorted"), (6000, "sorted"),
                                      (6000, "scattered"), (6000, "mixed"), (5000, "one cell")])
def test_density_and_weights_match_numpy(n, spread, precision, shape):
    from paper_2307_01797_amd import itokmc
    rng = np.random.default_rng(n)
    g = (13, 11, 9)
    nc = int(np.prod(g))
    cell = rng.integers(0, nc, n)
    if spread == "sorted":
        cell = np.sort(cell)
    elif spread == "mixed":
        cell[: n // 2] = np.sort(cell[: n // 2])
    elif spread == "one cell":
        cell[:] = nc - 1
    off = rng.random((n, 3)).astype(np.float32).astype(np.float64)
    w = rng.integers(1, 5000, n).astype(np.uint32)
    cfg = workloads.preset("avalanche_32", grid=g, precision=precision, shape=shape)
    sim = itokmc.Sim(cfg, max_particles=2 * n + 10)
    sim.set_particles(cell.astype(np.uint32), off, w, np.arange(n, dtype=np.uint64))
    ijk = np.stack([cell % g[0], (cell // g[0]) % g[1], cell // (g[0] * g[1])], 1)
    ref = _density(g, ijk, off, w.astype(np.float64), cfg["dx"] ** 3, shape == "tsc")
    got = sim.deposit("cic")
    assert np.abs(got - ref).max() <= 1e-12 * ref.max()
    assert np.array_equal(sim.deposit("ngp"), np.bincount(cell, weights=w, minlength=nc).astype(np.uint32))
    d = sim.diagnostics()
    assert d["n_particles"] == n and d["weight"] == int(w.sum())


@pytest.mark.parametrize("n0", [1, 63, 65, 1023, 1025, 4097])
def test_gaussian_seed_matches_oracle(orc, n0):
    from paper_2307_01797_amd import itokmc
    cfg = workloads.preset("avalanche_32", grid=(9, 14, 11), seed_n0=n0, seed_sigma=60e-6,
                           seed_centre=(30e-6, 70e-6, 55e-6))
    sim = itokmc.Sim(cfg, max_particles=6000)
    sim.seed()
    o = orc.Sim(cfg)
    o.seed_gaussian(n0, cfg["seed_centre"], cfg["seed_sigma"])
    cell, off, w, ids = sim.particles()
    xi, wo, io = o.particles()
    a, b = np.argsort(ids), np.argsort(io)
    assert np.array_equal(ids[a], io[b]) and np.all(w == 1)
    ijk = np.stack([cell % 9, (cell // 9) % 14, cell // (9 * 14)], 1)
    assert len(ids) == 0 or np.abs(ijk[a] + off[a] - xi[b]).max() <= 1e-12 * 14


@pytest.mark.parametrize("kind", ["gaussian", "neutral"])
def test_seed_past_the_capacity_fills_the_bank_and_is_reported(kind):
    from paper_2307_01797_amd import itokmc
    cap = 1500
    cfg = workloads.preset("avalanche_32", grid=(16, 16, 16), seed_n0=5000, seed_sigma=20e-6,
                           seed_centre=(80e-6,) * 3, seed_kind=kind, seed_peak=1e17)
    sim = itokmc.Sim(cfg, max_particles=cap)
    sim.seed()
    d = sim.diagnostics(check=False)
    assert d["overflow"] & itokmc.OVF_PARTICLES and d["n_particles"] == cap
    cell, off, w, ids = sim.particles()
    assert len(np.unique(ids)) == cap and cell.max() < 16 ** 3 and off.min() >= 0 and off.max() < 1


def test_neutral_seed_weights_and_ions(orc):
    from paper_2307_01797_amd import itokmc
    cfg = workloads.preset("streamer_64", grid=(16, 12, 20), dx=10e-6, seed_peak=2e17, seed_sigma=25e-6,
                           seed_centre=(80e-6, 60e-6, 100e-6), precision="fp64")
    sim = itokmc.Sim(cfg, max_particles=200_000)
    sim.seed()
    o = orc.Sim(cfg)
    o.seed_neutral(cfg["seed_peak"], cfg["seed_centre"], cfg["seed_sigma"])
    cell, off, w, ids = sim.particles()
    xi, wo, io = o.particles()
    a, b = np.argsort(ids), np.argsort(io)
    assert len(ids) > 5000 and np.array_equal(ids[a], io[b]) and np.array_equal(w[a].astype(np.uint64), wo[b])
    assert np.array_equal(np.bincount(cell, weights=w, minlength=16 * 12 * 20).astype(np.uint32), sim.counts("plus"))
