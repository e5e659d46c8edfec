"""Passes with fewer launches, at the sizes where they begin and end: the
mirrors numbered in one launch up to 32,768 particles against the scanned
numbering, bit for bit; ill-conditioned stencils refitted inside the staged
fits against refits from the global list (other summation order: the bound
of the tests that compare those two paths); and the displacement check whose
result the device writes to the host up to 131,072 particles, which has to
find one particle moved by a little more than half the skin."""
import numpy as np
import pytest

import lpgen
from cases import CASES
from test_gpu_parity import _log, lp  # noqa: F401
from test_gpu_staging import _run

pytestmark = pytest.mark.gpu


def _column(nx, ny, nz, n, seed=53):
    wl = lpgen.column_bench(seed=seed, nx=nx, ny=ny, nz=nz)
    wl.state = wl.state.take(np.arange(n))
    wl.offsets = np.array([0, n])
    return wl


@pytest.mark.parametrize("n", [1, 4096, 4097, 32768, 32769])
def test_mirrors_in_one_launch(lp, n):
    wl = _column(33, 32, 32, n)
    print("n", n, flush=True)
    got, a = _run(lp, wl, 2)
    ref, b = _run(lp, wl, 2, debug_flags=lp.LP_DEBUG_MIRROR_SCAN)
    assert a["mirrors"] == b["mirrors"]
    for x, y in zip(got.arrays(), ref.arrays()):
        assert np.array_equal(x, y)


def test_mirrors_in_one_launch_ensemble(lp):
    wl = CASES["ensemble_3"]()
    got, a = _run(lp, wl, 2)
    ref, b = _run(lp, wl, 2, debug_flags=lp.LP_DEBUG_MIRROR_SCAN)
    assert a["mirrors"] == b["mirrors"]
    for x, y in zip(got.arrays(), ref.arrays()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("order", [1, 2])
def test_refits_in_the_fits(lp, order):
    wl = CASES["sparse_cloud"]()
    got, a = _run(lp, wl, 1, order)
    ref, b = _run(lp, wl, 1, order, debug_flags=lp.LP_DEBUG_LANES2)
    _log("refits %d and %d" % (a["qr_refits"], b["qr_refits"]))
    assert a["qr_refits"] == b["qr_refits"] > 0
    for k, (x, y) in enumerate(zip(got.arrays(), ref.arrays())):
        scale = max(float(np.max(np.abs(y))), 1e-300)
        assert float(np.max(np.abs(x - y))) <= 1e-10 * scale, lp.DeviceState.NAMES[k]


@pytest.mark.parametrize("n", [63, 4097, 131072, 131073])
@pytest.mark.parametrize("far", [False, True])
def test_check_result_reaches_the_host(lp, n, far):
    wl = _column(51, 51, 51, n)
    print("n", n, far, flush=True)
    ctx = lp.make_context(wl)
    st = lp.DeviceState.from_host(wl.state)
    ctx.lp_step(st, wl.dt)
    assert ctx.stats()["rebuilds"] == 1
    # half the skin is 0.05 R = 0.125 h; a step moves a particle far less
    # (the check counts from 0.49 skins)
    h = wl.params[0].h
    st.t[2][n // 2] += (0.2 if far else 0.02) * h
    ctx.lp_step(st, wl.dt)
    ctx.sync_status()
    assert ctx.stats()["rebuilds"] == (1 if far else 0)
