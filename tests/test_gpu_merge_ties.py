"""Merging of cells whose pieces share coordinates: the small stagings order by coordinate
alone and fetch the ids only when two pieces take one slot.  All pieces at one point, two
or three distinct values per axis, one tied pair, signed zeros, cells around every
staging's capacity, and cells most of whose particles were just removed (more slots than
pieces); against the oracle (weights, ids and cells exact, offsets to the precision's
rounding of a weighted mean of values in [0, 1): 1e-6 and 1e-12)."""
import numpy as np
import pytest

from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 31, 32, 33, 44, 63, 64, 65, 96, 127, 128, 129, 160, 255, 256, 257, 400]


def _react(orc, cfg, cell, off, w, ids, precision):
    from paper_2307_01797_amd import itokmc
    g = cfg["grid"]
    sim = itokmc.Sim(cfg, precision=precision, max_particles=8 * len(w) + 70_000)
    sim.set_particles(cell.astype(np.uint32), off, w, ids)
    sim.react()
    ijk = np.stack([cell % g[0], (cell // g[0]) % g[1], cell // (g[0] * g[1])], 1)
    o = orc.Sim(cfg)
    o.set_particles(ijk + off, w.astype(np.uint64), ids)
    o.react(cfg["dt"])
    cg, og, wg, ig = sim.particles()
    xo, wo, io = o.particles()
    a, b = np.argsort(ig), np.argsort(io)
    assert np.array_equal(ig[a], io[b]) and np.array_equal(wg[a].astype(np.uint64), wo[b])
    pos = np.stack([cg % g[0], (cg // g[0]) % g[1], cg // (g[0] * g[1])], 1) + og
    assert np.abs(pos[a] - xo[b]).max() <= (1e-6 if precision == "fp32" else 1e-12) * max(g)
    return sim.diagnostics()


@pytest.mark.parametrize("n_ppc", [32, 64, 5])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["one point", "few values", "one pair", "signed zero"])
def test_tied_coordinates(orc, kind, precision, n_ppc):
    rng = np.random.default_rng(11)
    counts = np.array(COUNTS * 2)
    nc = len(counts)
    g = (6, 6, 4)
    cfg = workloads.preset("avalanche_32", grid=g, n_ppc=n_ppc, precision=precision)
    cfg["coeffs"].update(alpha_A=0.0, eta=0.0)
    cell = np.repeat(np.arange(nc) * 3 + 1, counts)
    n = len(cell)
    off = rng.random((n, 3)).astype(np.float32).astype(np.float64)
    if kind == "one point":
        off[:] = 0.375
    elif kind == "few values":
        off = rng.integers(0, 3, (n, 3)) / 4.0
    elif kind == "one pair":
        first = np.concatenate([[0], np.cumsum(counts)[:-1]])
        two = first[counts >= 2]
        off[two] = off[two + 1]
    else:
        off[rng.random((n, 3)) < 0.3] = 0.0
    w = np.where(rng.random(n) < 0.5, 1, rng.integers(1, 300, n)).astype(np.uint32)
    ids = rng.permutation(n).astype(np.uint64) * np.uint64(1 << 33) + np.uint64(5)
    d = _react(orc, cfg, cell, off, w, ids, precision)
    assert d["merged_cells"] >= nc - 8


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_more_slots_than_pieces(orc, precision):
    rng = np.random.default_rng(4)
    counts = np.tile([300, 420, 700, 1000], 9)
    g = (6, 6, 1)
    # attachment takes about two thirds of a cell's electrons in the step
    cfg = workloads.preset("avalanche_32", grid=g, n_ppc=32, precision=precision, E=(0.0, 0.0, 5e6), dt=2e-10)
    cfg["coeffs"].update(alpha_A=0.0, eta=4.5e4)
    cell = np.repeat(np.arange(36), counts)
    n = len(cell)
    off = rng.integers(0, 64, (n, 3)) / 64.0
    d = _react(orc, cfg, cell, off, np.ones(n, dtype=np.uint32), rng.permutation(n).astype(np.uint64), precision)
    assert d["removed_weight"] > n // 3 and d["merged_cells"] >= 30
