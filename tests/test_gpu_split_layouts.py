"""The finest level in split red-black order and in natural order with sweep counts whose
colours do not fit a tile's halo (three and three, four and none, none and three): such
levels are smoothed colour by colour in both precisions, so that the two layouts run
different kernels (nx = 48: the 8-cell row segments, split or natural; nx = 44: one cell a
thread).  With up to two sweeps these grids run in tiles, in natural order under either
setting.

In FP32 three self-consistent steps are bit-identical in both layouts (every cell's
arithmetic and every reduction order are the same, and the charge sums are integers); in FP64
the potential of one transport from the same state agrees within 1e-9 (the deposit adds in
any order).  The layout is the only difference of the two runs."""
import numpy as np
import pytest

from helpers import by_id
from paper_2307_01797_amd import workloads

pytestmark = pytest.mark.gpu

SWEEPS = [(3, 3), (4, 0), (0, 3)]


def _runs(grid, precision, pre, post, steps, **kw):
    from paper_2307_01797_amd import itokmc
    nz = grid[2]
    cfg = workloads.preset("streamer_64", grid=grid, dx=1e-3 / nz, V_anode=18e3 * nz / 64, precision=precision,
                           seed_centre=tuple(0.5 * g * 1e-3 / nz for g in grid), **kw)
    for layout in (0, 1):
        sim = itokmc.Sim(cfg, precision=precision)
        sim.set_tuning(fine_layout=layout, mg_pre=pre, mg_post=post)
        sim.seed()
        if steps:
            sim.step(steps)
        else:
            sim.transport()
        yield sim
        sim.close()


@pytest.mark.parametrize("pre,post", SWEEPS)
@pytest.mark.parametrize("grid", [(48, 32, 40), (44, 24, 36)])
def test_layouts_are_bit_identical(grid, pre, post):
    out = []
    for sim in _runs(grid, "fp32", pre, post, 3):
        c, o, w, i = sim.particles()
        out.append((sim.field(), sim.deposit("ez"), *by_id(i, c, o, w), sim.diagnostics()["solver_cycles_total"]))
    assert out[0][-1] == out[1][-1] > 0
    for a, b in zip(out[0][:-1], out[1][:-1]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("pre,post", SWEEPS)
@pytest.mark.parametrize("grid", [(64, 32, 48), (44, 36, 52)])
def test_layouts_reach_the_same_potential(grid, pre, post):
    a, b = [sim.field() for sim in _runs(grid, "fp64", pre, post, 0, gmg_rtol=1e-12, gmg_max_cycles=500)]
    assert np.abs(a - b).max() <= 1e-9 * np.abs(a).max()


def test_a_tiled_finest_level_against_colour_by_colour():
    """Two sweeps each way in tiles, three colour by colour in either layout: one potential."""
    phi = []
    for pre, post in ((2, 2), (3, 3)):
        phi += [sim.field() for sim in _runs((44, 24, 36), "fp64", pre, post, 0, gmg_rtol=1e-12, gmg_max_cycles=500)]
    for p in phi[1:]:
        assert np.abs(p - phi[0]).max() <= 1e-9 * np.abs(phi[0]).max()
