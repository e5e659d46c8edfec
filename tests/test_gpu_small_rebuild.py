"""The captured re-sort in one block (up to 8,192 particles and 64 systems)
at its edges against eager steps, bit for bit: one particle, powers of two
and their neighbours, several systems, periodic axes, ids carried along, and
a skin of 0, which re-sorts in every step; 8,193 particles and 65 systems
take the general path."""
import numpy as np
import pytest

import lpgen
from cases import CASES
from test_gpu_parity import lp  # noqa: F401

pytestmark = pytest.mark.gpu


def _column(n):
    wl = lpgen.column_bench(seed=59, nx=21, ny=21, nz=21)
    wl.state = wl.state.take(np.arange(n))
    wl.offsets = np.array([0, n])
    return wl


_STATES = {"n%d" % n: (lambda n=n: _column(n)) for n in (1, 2, 3, 1024, 1025, 4097, 8192, 8193)}
_STATES["ensemble_3"] = CASES["ensemble_3"]
_STATES["periodic_xy"] = CASES["periodic_xy"]
_STATES["sparse_cloud"] = CASES["sparse_cloud"]
_STATES["systems_64"] = lambda: lpgen.ensemble(n_sys=64, n_lo=40, n_hi=120)
_STATES["systems_65"] = lambda: lpgen.ensemble(n_sys=65, n_lo=40, n_hi=120)


@pytest.mark.parametrize("name", list(_STATES))
@pytest.mark.parametrize("skin", [0.1, 0.0])
def test_small_rebuild(lp, name, skin):
    import torch
    wl = _STATES[name]()
    print(name, wl.n, skin, flush=True)
    steps = 3
    a = lp.make_context(wl, skin=skin)
    sa = lp.DeviceState.from_host(wl.state)
    ids_a = torch.arange(wl.n, dtype=torch.int32, device="cuda")
    for _ in range(2):
        a.lp_step_graph(sa, wl.dt, steps, ids=ids_a)
    a.sync_status()
    # eager steps: the graph's first call sorts the caller's arrays
    b = lp.make_context(wl, skin=skin)
    sb = lp.DeviceState.from_host(wl.state)
    perm = torch.empty(wl.n, dtype=torch.int32, device="cuda")
    ids_b = torch.arange(wl.n, dtype=torch.int32, device="cuda")
    for _ in range(2 * steps):
        b.lp_step(sb, wl.dt, perm)
        ids_b = ids_b[perm.long()]
    b.sync_status()
    assert torch.equal(ids_a, ids_b)
    for x, y in zip(sa.t, sb.t):
        assert torch.equal(x, y)
