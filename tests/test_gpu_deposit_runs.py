"""The field deposit over every way a wavefront's particles can share cells: whole
wavefronts in one cell, runs at and past the lines of its two forms (8 and 9 runs; 4 and 5),
single particles, clusters at the walls, small and large diffusive displacements (inside and
outside a run's block of nodes), weights on both sides of the short fixed-point conversion.

One transport against the oracle from the same state: FP64 within 1e-9 of the largest
potential; FP32 within 1e-5 of it (every charge may sit 1e-5 cells off, the bar of the
positions).  In FP32 the node sums are integers, so the same particles in any order, which
shares cells differently, must give the potential bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import _oracle_from_gpu, _streamer_small

pytestmark = pytest.mark.gpu

GRID = (13, 11, 9)


@pytest.fixture(scope="module")
def itk():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2307_01797_amd import itokmc
    itokmc.lib()
    return itokmc


def _particles(rng):
    nx, ny, nz = GRID
    nc = nx * ny * nz
    walls = [i + nx * (j + ny * k) for i in (0, nx - 1) for j in (0, ny - 1) for k in (0, nz - 1)]
    per = [(12, 100), (6, 64), (24, 16), (20, 13), (32, 8), (27, 7), (16, 3), (150, 1)]
    perm = rng.permutation(nc)
    cells, at = [np.repeat(walls, 21)], 0
    for count, size in per:
        cells.append(np.repeat(np.sort(perm[at:at + count]), size))
        at += count
    cells = np.concatenate(cells).astype(np.int64)
    n = len(cells)
    w = rng.integers(1, 2000, n).astype(np.uint32)
    w[rng.integers(0, n, 5)] = (1 << 24) + 12345
    return cells, rng.random((n, 3)), w, np.arange(1, n + 1, dtype=np.uint64) * 7919


@pytest.mark.parametrize("disp", [0.1, 1.3])
@pytest.mark.parametrize("shape", ["cic", "tsc"])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("fp32", 1e-5)])
def test_runs(itk, orc, prec, tol, shape, disp):
    cfg = _streamer_small(grid=GRID, shape=shape, precision=prec, n_ppc=0, gmg_rtol=1e-12, gmg_max_cycles=500)
    cfg["coeffs"] = dict(cfg["coeffs"], D=(disp * cfg["dx"]) ** 2 / (2 * cfg["dt"]))
    rng = np.random.default_rng(83)
    cells, off, w, ids = _particles(rng)
    print(f"{prec} {shape} {disp} n={len(ids)}", flush=True)
    plus = np.bincount(cells, weights=w, minlength=int(np.prod(GRID))).astype(np.uint32)

    def potential(order):
        g = itk.Sim(cfg, precision=prec, max_particles=4 * len(ids))
        g.set_particles(cells[order], off[order], w[order], ids[order])
        g.set_counts("plus", plus)
        o = _oracle_from_gpu(orc, cfg, g) if order is every else None
        g.transport(cfg["dt"])
        return g.field(), o

    every = np.arange(len(ids))
    phi, o = potential(every)
    o.transport(cfg["dt"])
    phi_o = o.field()[0]
    assert np.abs(phi - phi_o).max() <= tol * np.abs(phi_o).max()
    for order in (rng.permutation(len(ids)), np.argsort(cells, kind="stable")):
        other, _ = potential(order)
        if prec == "fp32":
            assert np.array_equal(phi, other)
        else:
            assert np.abs(phi - other).max() <= tol * np.abs(phi_o).max()


@pytest.mark.parametrize("shape", ["cic", "tsc"])
def test_many_particles_in_any_order(itk, shape):
    """Past 2^21 particles (CIC's other line): grouped by cell and shuffled, bit for bit."""
    cfg = _streamer_small(grid=GRID, shape=shape, precision="fp32", n_ppc=0, gmg_rtol=1e-12, gmg_max_cycles=500)
    rng = np.random.default_rng(91)
    n, nc = (1 << 21) + 4321, int(np.prod(GRID))
    cells = np.sort(rng.integers(0, nc, n))
    off = rng.random((n, 3))
    w = rng.integers(1, 4, n).astype(np.uint32)
    ids = np.arange(1, n + 1, dtype=np.uint64)
    plus = np.bincount(cells, weights=w, minlength=nc).astype(np.uint32)
    phi = []
    for order in (np.arange(n), rng.permutation(n)):
        g = itk.Sim(cfg, precision="fp32", max_particles=2 * n)
        g.set_particles(cells[order], off[order], w[order], ids[order])
        g.set_counts("plus", plus)
        g.transport(cfg["dt"])
        phi.append(g.field())
    assert np.array_equal(phi[0], phi[1])
