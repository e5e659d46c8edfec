"""The cell-wise list build with 8, 4, 2 and 1 wavefronts per cell (by the
particle count), with cells at the wall, periodic axes and cells of many
particles, against the per-particle scan: the lists hold the same entries in
the same order, so two steps on them (one with the list as built, one later)
give the same bits."""
import numpy as np
import pytest

import lpgen
from cases import CASES
from test_gpu_parity import lp  # noqa: F401
from test_gpu_staging import _run

pytestmark = pytest.mark.gpu

_STATES = {
    "column_16384": lambda: _column(26, 26, 25, 16384),
    "column_16385": lambda: _column(26, 26, 25, 16385),
    "column_65537": lambda: _column(41, 41, 40, 65537),
    "column_262145": lambda: _column(65, 64, 64, 262145),
    "sheared_33k": lambda: lpgen.column_sheared(nx=37, ny=29, nz=31),
    "periodic_xy": CASES["periodic_xy"],
    "ensemble_3": CASES["ensemble_3"],
    "sparse_cloud": CASES["sparse_cloud"],
}


def _column(nx, ny, nz, n):
    wl = lpgen.column_bench(seed=37, nx=nx, ny=ny, nz=nz)
    wl.state = wl.state.take(np.arange(n))
    wl.offsets = np.array([0, n])
    return wl


@pytest.mark.parametrize("name", list(_STATES))
def test_split_cells_give_the_scan_lists(lp, name):
    wl = _STATES[name]()
    print(name, wl.n, flush=True)
    got, _ = _run(lp, wl, 2)
    ref, _ = _run(lp, wl, 2, debug_flags=lp.LP_DEBUG_PARTICLE_LIST)
    for a, b in zip(got.arrays(), ref.arrays()):
        assert np.array_equal(a, b)
