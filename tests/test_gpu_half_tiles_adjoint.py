"""The reverse kernels on tiles staged in halves: the reverse of a recorded
step (whose list has a tile map) on a state whose launch mixes whole and half
tiles, against the adjoint oracle with the bounds of the other adjoint tests,
for one system and for two that meet inside a tile."""
import dataclasses

import numpy as np
import pytest

import lpgen
from cases import _with_flow
from oracle import adjoint
from test_gpu_adjoint import TOL, _dev, _lam
from test_gpu_parity import _log, _relerr, lp  # noqa: F401

pytestmark = pytest.mark.gpu


def _dense(systems):
    wl = lpgen.column_bench(seed=83, nx=27, ny=26, nz=25)      # 17,550
    h = wl.params[0].h * 1.25
    wl.params = [dataclasses.replace(p, h=h, R=2.5 * h) for p in wl.params]
    if systems == 2:
        st = wl.state
        far = dataclasses.replace(st, x=st.x + 3.0)
        wl.state = lpgen.State.concat([st, far])
        wl.params = wl.params + [dataclasses.replace(wl.params[0], mu_s=0.33, I0=0.25)]
        wl.offsets = np.array([0, st.n, 2 * st.n])
    return _with_flow(wl)


@pytest.mark.parametrize("systems", [1, 2])
def test_recorded_step_on_half_tiles(lp, systems):
    import torch
    wl = _dense(systems)
    lam = _lam(wl, 89)
    want, wth, operm = adjoint.step_vjp(wl.state, wl.offsets, wl.params, wl.dt, lam)
    ctx = lp.make_context(wl)
    st = lp.DeviceState.from_host(wl.state)
    before = st.clone()
    rec = lp.StepRecord(wl.n, force_sort=True)
    ctx.lp_step(st, wl.dt, rec=rec)
    ctx.sync_status()
    stats = ctx.stats()
    print("systems", systems, "n", wl.n, stats, flush=True)
    assert 0 < stats["unstaged_tiles"] < stats["tiles"]
    assert np.array_equal(rec.perm.cpu().numpy(), operm)
    dth = torch.zeros(systems, 3, dtype=torch.float64, device="cuda")
    got = ctx.lp_step_adjoint(before, wl.dt, _dev(lam), dth, rec=rec)
    ctx.sync_status()
    # (the list and its map are those of the recorded step still)
    assert ctx.stats()["unstaged_tiles"] == stats["unstaged_tiles"]
    for k, (a, b) in enumerate(zip(got.to_host().arrays(), want)):
        e = _relerr(a, b)
        _log("  d/d%s rel err %.3e" % (lp.DeviceState.NAMES[k], e))
        assert e <= TOL, (lp.DeviceState.NAMES[k], e)
    gth = dth.cpu().numpy()
    e = np.max(np.abs(gth - wth)) / np.max(np.abs(wth))
    _log("  d/dtheta rel err %.3e (max |dtheta| %.3e)" % (e, np.max(np.abs(wth))))
    assert np.all(np.max(np.abs(wth), axis=1) > 0.0) and e <= 1e-9
