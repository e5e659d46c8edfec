"""Tiles of which neither half can be staged (more than 1,664 sources each, on
a dense lattice) are one unit that gathers from memory: steps and reversed
steps on launches that mix them with staged ones against launches that gather
throughout, with the bounds of the tests that compare those paths."""
import dataclasses

import numpy as np
import pytest

import lpgen
from test_gpu_adjoint import _dev, _lam
from test_gpu_parity import _log, lp  # noqa: F401
from test_gpu_staging import _compare, _run

pytestmark = pytest.mark.gpu


def _denser(nx, ny, nz):
    # 235 list entries per particle at most; 2,000 sources per half tile inside
    wl = lpgen.column_bench(seed=107, nx=nx, ny=ny, nz=nz)
    h = wl.params[0].h * 1.36
    wl.params = [dataclasses.replace(p, h=h, R=2.5 * h) for p in wl.params]
    return wl


@pytest.mark.parametrize("dims", [(20, 20, 22), (27, 26, 25)])     # eight lanes, one
@pytest.mark.parametrize("order", [1, 2])
def test_steps_on_unstaged_tiles(lp, dims, order):
    wl = _denser(*dims)
    print(dims, order, flush=True)
    got, st = _run(lp, wl, 2, order)
    ref, sg = _run(lp, wl, 2, order, debug_flags=lp.LP_DEBUG_GLOBAL_GATHER)
    _log("stats %s" % st)
    assert 0 < st["unstaged_tiles"] < st["tiles"] == sg["unstaged_tiles"]
    _compare(got, ref, "unstaged")


def test_reversed_steps_on_unstaged_tiles(lp):
    wl = _denser(20, 20, 22)
    wl = lpgen.with_shear_velocity(wl)
    lam = _dev(_lam(wl, 109))
    out = []
    for flags in (0, lp.LP_DEBUG_GLOBAL_GATHER):
        ctx = lp.make_context(wl, debug_flags=flags)
        st = lp.DeviceState.from_host(wl.state)
        before = st.clone()
        rec = lp.StepRecord(wl.n, force_sort=True)
        ctx.lp_step(st, wl.dt, rec=rec)
        got = ctx.lp_step_adjoint(before, wl.dt, lam, rec=rec)
        ctx.sync_status()
        out.append(got.to_host().arrays())
    for name, a, b in zip(lp.DeviceState.NAMES, *out):
        assert float(np.max(np.abs(a - b))) <= 1e-10 * float(np.max(np.abs(b))), name
