"""Sizes on both sides of the lines of a step's launches, one step against the oracle (FP64,
every integer exact, positions to 1e-9 cells): the cell scan at and past 1024 tiles of 2048
cells, with the first and last cell occupied; KMC with one, two and four cells per thread
(131072 threads); the push with one and two particles per thread (2^20 threads)."""
import numpy as np
import pytest

from paper_2307_01797_amd import workloads
from test_gpu_parity import _compare, _compare_tallies, _oracle_from_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,occupied,n", [
    ((128, 128, 128), 131072, 131072),
    ((128, 128, 129), 131073, 131073),
    ((96, 96, 96), 524287, 1048576),
    ((95, 96, 97), 524288, 1048577),
    ((15, 14, 13), 257, 600),
])
def test_step_at_the_lines(orc, grid, occupied, n):
    from paper_2307_01797_amd import itokmc
    print(grid, occupied, n, flush=True)
    cfg = workloads.preset("avalanche_32", grid=grid, coeffs=dict(D=0.0))  # centred particles stay in their cells
    nc = int(np.prod(grid))
    rng = np.random.default_rng(n)
    cells = rng.choice(nc - 2, occupied - 2, replace=False) + 1
    cells = np.concatenate([[0, nc - 1], cells])
    cells = np.sort(np.concatenate([cells, rng.choice(cells, n - occupied)]))
    g = itokmc.Sim(cfg, max_particles=2 * n + 1000)
    g.set_particles(cells, np.full((n, 3), 0.5), rng.integers(1, 4, n).astype(np.uint32),
                    np.arange(1, n + 1, dtype=np.uint64))
    o = _oracle_from_gpu(orc, cfg, g)
    g.step(1)
    o.step(cfg["dt"], 1)
    assert _compare(g, o, cfg, 1e-9) == 0
    _compare_tallies(g, o)
    cell = g.particles()[0]
    assert np.array_equal(np.bincount(cell, weights=g.particles()[2], minlength=nc).astype(np.uint32), g.deposit("ngp"))
    assert len(np.unique(cell)) >= 0.9 * occupied
