"""A system that turns non-finite leaves the other systems of its context as
they are: captured steps (whose re-sort bounds the systems in one block, a
wavefront of 64 particles across two systems included) against eager ones."""
import numpy as np
import pytest

import lpgen
from test_gpu_parity import lp  # noqa: F401

pytestmark = pytest.mark.gpu


def _two_columns():
    h = 1.0 / 16.0
    p = lpgen.default_params(h)
    a = lpgen.lattice_column(10, 10, 10, h, seed=73, params=p)
    b = lpgen.lattice_column(10, 10, 10, h, seed=74, params=p, x0=3.0)
    st = lpgen.State.concat([a, b])
    return lpgen.Workload("two", st, np.array([0, 1000, 2000]), [p, p], 1e-4, 1)


def _run(lp, wl, captured, steps):
    """State, ids and the error of the steps of the sorted state wl."""
    import torch
    ctx = lp.make_context(wl)
    st = lp.DeviceState.from_host(wl.state)
    ids = torch.arange(wl.n, dtype=torch.int32, device="cuda")
    if captured:
        ctx.lp_step_graph(st, wl.dt, steps, ids=ids)
    else:
        perm = torch.empty(wl.n, dtype=torch.int32, device="cuda")
        for _ in range(steps):
            ctx.lp_step(st, wl.dt, perm)
            ids = ids[perm.long()]
    try:
        ctx.sync_status()
        err = 0
    except lp.LPError as e:
        err = e.status
    return [a.cpu().numpy() for a in st.t], ids.cpu().numpy(), err


def test_the_other_system_is_untouched(lp):
    wl = _two_columns()
    ctx = lp.make_context(wl)
    st = lp.DeviceState.from_host(wl.state)
    ctx.lp_build_cells(st)
    wl.state = st.to_host()
    # the last particle of the first system: its position turns non-finite in
    # the first step, and the next one re-sorts
    wl.state.u[999] = np.nan
    got, ids, err = _run(lp, wl, True, 4)
    want, wids, werr = _run(lp, wl, False, 4)
    print("errors", err, werr, flush=True)
    assert np.isnan(got[0][:1000]).any()
    assert np.array_equal(ids[1000:], wids[1000:])
    for name, a, b in zip(lp.DeviceState.NAMES, got, want):
        assert np.isfinite(b[1000:]).all()
        assert np.array_equal(a[1000:], b[1000:]), name
    assert err == werr != 0
