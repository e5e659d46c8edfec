"""Small states with ill-conditioned stencils: the fits refit their own
particles until they have met some, then a launch after each fit does.  Both
give the same bits: steps, second-order steps and reversed steps on a context
that has changed against one that has not, and captured sequences, captured
anew at the change, against eager steps."""
import dataclasses

import numpy as np
import pytest

import lpgen
from test_gpu_adjoint import _dev, _lam
from test_gpu_parity import _log, lp  # noqa: F401

pytestmark = pytest.mark.gpu


def _spray(n, dens):
    """n particles, dens per h^3, in a cube on the wall: hundreds of refits."""
    h = 1.0 / 16.0
    p = lpgen.default_params(h)
    u = lpgen.uniform01(11, np.arange(7 * n, dtype=np.uint64)).reshape(7, n)
    side = (n / dens) ** (1.0 / 3.0) * h
    st = lpgen.State(side * u[0], side * u[1], side * u[2] + 0.001, 0.2 * (u[3] - 0.5),
                     0.2 * (u[4] - 0.5), 0.2 * (u[5] - 0.5), 1.0 / (0.47 + 0.1 * u[6]))
    return lpgen.Workload("spray", st, np.array([0, n]), [p], 1e-5, 1)


def _changed(lp, wl, **cfg):
    """A context that has met refits, and the state again."""
    ctx = lp.make_context(wl, **cfg)
    st = lp.DeviceState.from_host(wl.state)
    ctx.lp_step(st, wl.dt)
    ctx.sync_status()
    ctx.stats()
    for a, b in zip(st.t, lp.DeviceState.from_host(wl.state).t):
        a.copy_(b)
    return ctx, st


# (16,384 particles: the most that the fits refit themselves)
@pytest.mark.parametrize("n,weight,periodic", [(1000, 0, False), (10000, 0, False),
                                               (16384, 0, False), (10000, 1, False),
                                               (10000, 0, True), (10000, 1, True)])
def test_steps_on_both_sides_of_the_change(lp, n, weight, periodic):
    import torch
    wl = _spray(n, 0.1)
    if periodic:
        side = (n / 0.1) ** (1.0 / 3.0) * wl.params[0].h
        wl.params = [dataclasses.replace(p, box_len=(side, side)) for p in wl.params]
    print("n", n, weight, periodic, flush=True)
    a, sa = lp.make_context(wl, weight=weight), lp.DeviceState.from_host(wl.state)
    b, sb = _changed(lp, wl, weight=weight)
    refits = []
    for k in range(3):
        for ctx, st in ((a, sa), (b, sb)):
            ctx.lp_step(st, wl.dt, rec=lp.StepRecord(n, force_sort=k == 0))
            ctx.sync_status()
            refits.append(ctx.stats()["qr_refits"])
        for name, x, y in zip(lp.DeviceState.NAMES, sa.t, sb.t):
            assert torch.equal(x, y), (k, name)
    _log("refits %s" % refits)
    assert refits[0] > n // 50 and refits[1::2] == refits[::2]


def test_captured_steps(lp):
    import torch
    wl = _spray(10000, 0.1)
    a, sa = lp.make_context(wl), lp.DeviceState.from_host(wl.state)
    b, sb = lp.make_context(wl), lp.DeviceState.from_host(wl.state)
    for k in range(3):
        a.lp_step_graph(sa, wl.dt, 3)
        a.sync_status()
        for _ in range(3):
            b.lp_step(sb, wl.dt)
        b.sync_status()
        assert a.stats()["qr_refits"] == b.stats()["qr_refits"] > 500
        for name, x, y in zip(lp.DeviceState.NAMES, sa.t, sb.t):
            assert torch.equal(x, y), (k, name)


def test_second_order_steps(lp):
    import torch
    wl = _spray(10000, 0.1)
    a, sa = lp.make_context(wl), lp.DeviceState.from_host(wl.state)
    b, sb = _changed(lp, wl)
    for ctx, st in ((a, sa), (b, sb)):
        ctx.lp_step2(st, wl.dt, rec=lp.StepRecord(wl.n, force_sort=True))
        ctx.sync_status()
    for name, x, y in zip(lp.DeviceState.NAMES, sa.t, sb.t):
        assert torch.equal(x, y), name


@pytest.mark.parametrize("second", [False, True])
def test_reversed_steps(lp, second):
    wl = _spray(10000, 0.1)
    lam = _dev(_lam(wl, 103))
    out = []
    for ctx, st in ((lp.make_context(wl), lp.DeviceState.from_host(wl.state)),
                    _changed(lp, wl)):
        got = (ctx.lp_step2_adjoint if second else ctx.lp_step_adjoint)(st, wl.dt, lam)
        ctx.sync_status()
        out.append(got.to_host().arrays())
    # (the reverse kernels add their receivers' shares in no fixed order)
    for name, a, b in zip(lp.DeviceState.NAMES, *out):
        assert float(np.max(np.abs(a - b))) <= 1e-12 * float(np.max(np.abs(b))), name
