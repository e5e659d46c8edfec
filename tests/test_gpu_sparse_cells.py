"""The cell-wise list build where nearly every cell is empty (a wavefront looks
at 64 of its cells at once, several times over) against the per-particle scan:
lists with the same entries in the same order, so steps on them give the same
bits; eager, captured (a grid sized by the particles strides over the cells)
and without a skin, which builds the list in every step."""
import numpy as np
import pytest

import lpgen
from test_gpu_parity import lp  # noqa: F401

pytestmark = pytest.mark.gpu


def _spread(n, cells, clumps):
    """n particles in `clumps` dense clumps over a box of cells^3 list cells."""
    h = 1.0 / 16.0
    p = lpgen.default_params(h)
    u = lpgen.uniform01(101, np.arange(7 * n, dtype=np.uint64)).reshape(7, n)
    side = cells * 2.75 * h
    c = lpgen.uniform01(102, np.arange(3 * clumps, dtype=np.uint64)).reshape(3, clumps)
    which = np.arange(n) % clumps
    at = side * c[:, which] + 4.0 * h * u[:3]
    at[:, 0] = 0.0
    at[:, 1] = side
    st = lpgen.State(at[0], at[1], at[2] + 0.001, 0.2 * (u[3] - 0.5), 0.2 * (u[4] - 0.5),
                     0.2 * (u[5] - 0.5), 1.0 / (0.30 + 0.32 * u[6]))
    return lpgen.Workload("spread", st, np.array([0, n]), [p], 1e-4, 1)


@pytest.mark.parametrize("n,cells,clumps", [(700, 60, 40), (700, 60, 650), (17000, 60, 500)])
@pytest.mark.parametrize("captured,skin", [(False, 0.1), (False, 0.0), (True, 0.0)])
def test_sparse_cells_give_the_scan_lists(lp, n, cells, clumps, captured, skin):
    import torch
    wl = _spread(n, cells, clumps)
    print(n, cells, clumps, captured, skin, flush=True)
    out = []
    for flags in (0, lp.LP_DEBUG_PARTICLE_LIST):
        ctx = lp.make_context(wl, skin=skin, debug_flags=flags)
        st = lp.DeviceState.from_host(wl.state)
        if captured:
            for _ in range(2):
                ctx.lp_step_graph(st, wl.dt, 2)
        else:
            for _ in range(3):
                ctx.lp_step(st, wl.dt)
        ctx.sync_status()
        out.append(st.t)
    for a, b in zip(*out):
        assert torch.equal(a, b)
