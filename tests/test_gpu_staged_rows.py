"""The staged fits at the edges of their dispatch: eight lanes per particle
up to 16,384 particles and one above, stencils of every remainder of a row
chunk, with each kind of weights and with periodic axes, against the oracle;
and tiles staged in halves (more than 1,664 sources) in every kernel that
reads staged rows, against the same pass gathering from global memory, with
the bounds of the tests that compare those two paths on whole tiles."""
import dataclasses

import numpy as np
import pytest

import lpgen
import oracle
from cases import CASES
from test_gpu_adjoint import _dev, _lam
from test_gpu_parity import _incr_ok, _log, lp  # noqa: F401
from test_gpu_staging import _compare, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16384, 16385])
def test_rows_on_both_sides_of_the_lane_rule(lp, n):
    import torch
    wl = lpgen.column_bench(seed=29, nx=26, ny=26, nz=25)
    wl.state = wl.state.take(np.arange(n))
    wl.offsets = np.array([0, n])
    print("n", n, flush=True)
    ctx = lp.make_context(wl)
    st = lp.DeviceState.from_host(wl.state)
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    ctx.lp_step(st, wl.dt, perm)
    ctx.sync_status()
    ost, operm, _ = oracle.step(wl.state, wl.offsets, wl.params, wl.dt)
    assert np.array_equal(perm.cpu().numpy(), operm)
    old = wl.state.take(operm)
    for k, (a, b, c) in enumerate(zip(st.to_host().arrays(), ost.arrays(), old.arrays())):
        ok, e = _incr_ok(a, b, c)
        assert ok, (lp.DeviceState.NAMES[k], e)


@pytest.mark.parametrize("case", ["column16", "periodic_xy"])
@pytest.mark.parametrize("weight", [0, 1])
@pytest.mark.parametrize("m_max", [57, 58, 59, 64, 9, 3])
def test_rows_of_every_remainder(lp, case, weight, m_max):
    wl = CASES[case]()
    print("case", case, "weight", weight, "m_max", m_max, flush=True)
    cfg = dict(weight=weight, m_max=m_max)
    got, _ = _run(lp, wl, 1, **cfg)
    ref, _ = _run(lp, wl, 1, debug_flags=lp.LP_DEBUG_GLOBAL_GATHER, **cfg)
    _compare(got, ref, "m_max %d" % m_max)


def _dense():
    wl = lpgen.column_bench(seed=31, nx=27, ny=26, nz=25)      # 17,550
    h = wl.params[0].h * 1.25
    wl.params = [dataclasses.replace(p, h=h, R=2.5 * h) for p in wl.params]
    return wl


@pytest.mark.parametrize("n", [17550, 13001])          # one lane, eight
@pytest.mark.parametrize("kind", ["step", "step2", "refined", "gauss"])
def test_half_tiles(lp, n, kind):
    wl = _dense()
    wl.state = wl.state.take(np.arange(n))
    wl.offsets = np.array([0, n])
    print("n", n, kind, flush=True)
    cfg = {"refined": dict(precision=lp.LP_FP32_REFINED), "gauss": dict(weight=1)}.get(kind, {})
    order = 2 if kind == "step2" else 1
    got, st = _run(lp, wl, 1, order, **cfg)
    ref, _ = _run(lp, wl, 1, order, debug_flags=lp.LP_DEBUG_GLOBAL_GATHER, **cfg)
    _log("stats %s" % st)
    assert 0 < st["unstaged_tiles"] < st["tiles"]
    _compare(got, ref, kind, rtol=1e-10 if kind == "refined" else 1e-12)


def test_half_tiles_adjoint(lp):
    import torch
    wl = _dense()
    lam = _lam(wl, 47)
    out = []
    for flags in (0, lp.LP_DEBUG_GLOBAL_GATHER):
        ctx = lp.make_context(wl, debug_flags=flags)
        st = lp.DeviceState.from_host(wl.state)
        dth = torch.zeros(len(wl.params), 3, dtype=torch.float64, device="cuda")
        got, _ = ctx.lp_step_adjoint(st, wl.dt, _dev(lam), dth, want_perm=True)
        ctx.sync_status()
        out.append(got.to_host().arrays())
    for k, (a, b) in enumerate(zip(*out)):
        scale = max(float(np.max(np.abs(b))), 1e-300)
        assert float(np.max(np.abs(a - b))) <= 1e-10 * scale, lp.DeviceState.NAMES[k]
