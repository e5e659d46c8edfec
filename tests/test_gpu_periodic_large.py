"""Periodic layers above the size rules of the selection and the fits (16,384:
one lane per particle in the fits; 163,840: the selection in two kernels, from
staged positions in a step and gathering in lp_neighbors), with one and two
periodic axes, against the oracle: candidates, stencils and ghost masks equal,
one step and, with Gaussian weights, its fits within the parity bounds."""
import numpy as np
import pytest

import oracle
from cases import _periodic_layer
from test_gpu_parity import _check_neighbours, _incr_ok, _log, lp  # noqa: F401

pytestmark = pytest.mark.gpu

_DIMS = {16900: (26, 26, 25), 166375: (55, 55, 55)}
_AXES = {"xy": (True, True), "x": (True, False)}


@pytest.mark.parametrize("n", list(_DIMS))
@pytest.mark.parametrize("axes", list(_AXES))
@pytest.mark.parametrize("weight", [0, 1])
def test_step_on_a_large_periodic_layer(lp, n, axes, weight):
    import torch
    wl = _periodic_layer(*_DIMS[n], axes=_AXES[axes], seed=97)
    assert wl.n == n
    print("n", n, axes, "weight", weight, flush=True)
    ctx = lp.make_context(wl, weight=weight)
    st = lp.DeviceState.from_host(wl.state)
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    ctx.lp_step(st, wl.dt, perm)
    ctx.sync_status()
    stats = ctx.stats()
    _log("stats %s" % stats)
    assert stats["unstaged_tiles"] < stats["tiles"]
    ost, operm, _ = oracle.step(wl.state, wl.offsets, wl.params, wl.dt,
                                cfg=dict(weight=weight))
    assert np.array_equal(perm.cpu().numpy(), operm)
    old = wl.state.take(operm)
    for k, (a, b, c) in enumerate(zip(st.to_host().arrays(), ost.arrays(), old.arrays())):
        ok, e = _incr_ok(a, b, c)
        assert ok, (lp.DeviceState.NAMES[k], e)


@pytest.mark.parametrize("n", list(_DIMS))
@pytest.mark.parametrize("axes", list(_AXES))
def test_neighbours_of_a_large_periodic_layer(lp, n, axes):
    print("n", n, axes, flush=True)
    _check_neighbours(lp, _periodic_layer(*_DIMS[n], axes=_AXES[axes], seed=97))
