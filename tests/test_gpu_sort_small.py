"""The one-workgroup counting sort and the line to the six launches: particle and cell
counts at the edges of both (6144 particles, 36864 cells), a thread's runs of cells, one
cell for all, dead and out-of-range particles, against the sort's definition."""
import numpy as np
import pytest

from test_gpu_sort import check_sorted, make_input

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,ncell", [(0, 1), (1, 1), (777, 1), (1024, 1023), (1025, 1025), (3001, 32768),
                                     (6143, 4097), (6144, 36864), (6145, 36864), (6144, 36865), (64, 36863)])
def test_small_sorts(prec, n, ncell):
    from paper_2307_01797_amd import itokmc
    rng = np.random.default_rng(7 * n + ncell)
    cell, off, w, ids = make_input(rng, n, ncell)
    print(n, ncell, prec, flush=True)
    out = itokmc.sort_by_cell(cell, off, w, ids, ncell, precision=prec)
    check_sorted(out, cell, off, w, ids, ncell, prec)


def test_every_particle_dead_or_outside():
    from paper_2307_01797_amd import itokmc
    n, ncell = 3000, 500
    rng = np.random.default_rng(5)
    cell, off, w, ids = make_input(rng, n, ncell)
    cell[::2] = 0xFFFFFFFF
    w[1::2] = 0
    check_sorted(itokmc.sort_by_cell(cell, off, w, ids, ncell, precision="fp32"), cell, off, w, ids, ncell, "fp32")
