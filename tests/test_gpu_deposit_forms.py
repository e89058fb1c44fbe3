"""The field deposit's two kernels from the same state: the one that sums blocks of nodes per
run of equal cells and the one that adds every particle to the table.  The device chooses by
particles and occupied cells of the last sort, so a fresh context (no sort yet) takes the
blocks and one that has sorted sparse cells takes the particles by themselves; cells of one
particle to some hundred, runs of 8 and 9 (and 4 and 5) cells a wavefront, clusters at the
walls, displacements inside and outside a block, weights on both sides of the short
fixed-point conversion.

One transport against the oracle's from the same state: FP64 within 1e-9 of the largest
potential; FP32 within 1e-5 of it (every charge may sit 1e-5 cells off, the bar of the
positions).  In FP32 the node sums are integers: both kernels give the potential bit for
bit."""
import numpy as np
import pytest

from test_gpu_parity import _oracle_from_gpu, _streamer_small

pytestmark = pytest.mark.gpu

# (cells, particles each): particles per occupied cell below 12, 5 and 2
MIXES = {
    "sparse 12": ((64, 60, 52), [(99_000, 1), (60_000, 4), (20_000, 16), (3_000, 7), (3_000, 8), (8_000, 80),
                                 (1_500, 520)]),
    "sparse 5": ((60, 52, 48), [(80_000, 1), (30_000, 4), (2_000, 7), (2_000, 8), (6_000, 16), (1_000, 200)]),
    "sparse 2": ((60, 52, 44), [(105_000, 1), (10_000, 3), (500, 13), (300, 16), (100, 70)]),
}
# precision, shape, mix, the smallest number of particles and the line of the per-particle form
CASES = [("fp32", "cic", "sparse 12", 1 << 21, 12), ("fp64", "cic", "sparse 5", 1 << 19, 5),
         ("fp32", "tsc", "sparse 5", 1 << 19, 5), ("fp32", "tsc", "sparse 2", 0, 3),
         ("fp64", "tsc", "sparse 2", 0, 2)]


@pytest.mark.parametrize("disp", [0.1, 1.3])
@pytest.mark.parametrize("prec,shape,mix,least,line", CASES)
def test_both_forms(orc, prec, shape, mix, least, line, disp):
    from paper_2307_01797_amd import itokmc
    grid, per = MIXES[mix]
    nx, ny, nz = grid
    cfg = _streamer_small(grid=grid, shape=shape, precision=prec, n_ppc=0, gmg_rtol=1e-12, gmg_max_cycles=500)
    cfg["coeffs"] = dict(cfg["coeffs"], alpha_A=0.0, eta=0.0, kgamma_ratio=0.0,
                         D=(disp * cfg["dx"]) ** 2 / (2 * cfg["dt"]))
    rng = np.random.default_rng(17)
    walls = [i + nx * (j + ny * k) for i in (0, nx - 1) for j in (0, ny - 1) for k in (0, nz - 1)]
    perm = rng.permutation(nx * ny * nz)
    cells, at = [np.repeat(walls, 21)], 0
    for count, size in per:
        cells.append(np.repeat(perm[at:at + count], size))
        at += count
    cells = np.sort(np.concatenate(cells)).astype(np.int64)
    n, occ = len(cells), len(np.unique(cells))
    assert n >= least and n // line < occ
    off = rng.random((n, 3))
    w = rng.integers(1, 2000, n).astype(np.uint32)
    w[rng.integers(0, n, 5)] = (1 << 24) + 12345
    ids = np.arange(1, n + 1, dtype=np.uint64) * 7919
    plus = np.bincount(cells, weights=w, minlength=nx * ny * nz).astype(np.uint32)

    phi = []
    for sort_first in (False, True):
        print(f"{prec} {shape} {mix} {disp} n={n} occ={occ} sorted={sort_first}", flush=True)
        g = itokmc.Sim(cfg, precision=prec, max_particles=n + 100_000)
        g.set_particles(cells, off, w, ids)
        if sort_first:
            g.react(cfg["dt"])  # no reaction has a rate: the sort alone
            g.set_step(0)
            assert g.diagnostics()["occupied_cells"] == occ
            g.set_particles(cells, off, w, ids)
        g.set_counts("plus", plus)
        if not sort_first:
            o = _oracle_from_gpu(orc, cfg, g)
            o.transport(cfg["dt"])
            phi_o = o.field()[0]
        g.transport(cfg["dt"])
        phi.append(g.field())
        g.close()
    scale = np.abs(phi_o).max()
    tol = 1e-9 if prec == "fp64" else 1e-5
    assert np.abs(phi[0] - phi_o).max() <= tol * scale
    assert np.abs(phi[1] - phi_o).max() <= tol * scale
    if prec == "fp32":
        assert np.array_equal(phi[0], phi[1])
