"""Stencil selection at the edges of its dispatch (lanes per particle, one
or two kernels), of the stencil cap and of its ties, against the oracle bit
for bit: particle counts on both sides of each size rule, caps below the
number of octants, equal distances decided by id (a lattice, coincident
points), lists longer than the chunks a group of lanes takes at once."""
import numpy as np
import pytest

import lpgen
from cases import CASES
from test_gpu_parity import _check_neighbours, _log, lp  # noqa: F401

pytestmark = pytest.mark.gpu


def _column(nx, ny, nz, drop=0, seed=91):
    wl = lpgen.column_bench(seed=seed, nx=nx, ny=ny, nz=nz)
    if drop:
        keep = np.sort(np.random.default_rng(7).choice(wl.n, wl.n - drop, replace=False))
        wl.state = wl.state.take(keep)
        wl.offsets = np.array([0, wl.n])
    return wl


# 8,192: 16 or 8 lanes per particle; 163,840: one kernel or two (the second
# pair without a tile map: lp_neighbors gathers)
@pytest.mark.parametrize("dims,drop", [((4, 4, 4), 0), ((21, 20, 20), 208), ((21, 20, 20), 207),
                                       ((55, 55, 55), 2535), ((55, 55, 55), 2534)])
@pytest.mark.parametrize("m_max", [60, 17])
def test_selection_on_both_sides_of_its_size_rules(lp, dims, drop, m_max):
    wl = _column(*dims, drop=drop)
    _log("n=%d m_max=%d" % (wl.n, m_max))
    import oracle
    cfg = oracle.CFG_DEFAULT
    saved = cfg["m_max"]
    try:
        cfg["m_max"] = m_max
        _check_neighbours(lp, wl, m_max=m_max)
    finally:
        cfg["m_max"] = saved


def _coincident(n_same):
    """A jittered column with n_same copies of one of its points."""
    wl = _column(9, 9, 9)
    st = wl.state
    j = 364
    wl.state = lpgen.State.concat([st, st.take(np.full(n_same, j))])
    wl.offsets = np.array([0, wl.n])
    return wl


_STATES = {
    "lattice": CASES["lattice_exact"],
    "sparse_cloud": CASES["sparse_cloud"],
    "periodic_xy": CASES["periodic_xy"],
    "ensemble_3": CASES["ensemble_3"],
    # 20 and 130 points at distance zero of each other: ties ranked from the
    # LDS list, and more than it holds
    "coincident_20": lambda: _coincident(20),
    "coincident_130": lambda: _coincident(130),
}


@pytest.mark.parametrize("case", list(_STATES))
@pytest.mark.parametrize("m_max", [1, 5, 8, 33, 64])
@pytest.mark.parametrize("second_kernel", [False, True])
def test_selection_ties_and_caps(lp, case, m_max, second_kernel):
    import oracle
    wl = _STATES[case]()
    _log("case %s n=%d m_max=%d second kernel %s" % (case, wl.n, m_max, second_kernel))
    cfg = oracle.CFG_DEFAULT
    saved = cfg["m_max"]
    try:
        cfg["m_max"] = m_max
        ctx = _check_neighbours(lp, wl, m_max=m_max,
                                debug_flags=lp.LP_DEBUG_SORTED_STENCIL if second_kernel else 0)
    finally:
        cfg["m_max"] = saved
    assert (ctx.stats()["sorted_stencils"] > 0) == second_kernel
