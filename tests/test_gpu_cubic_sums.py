"""The cubic fits take their reflectors' sums four columns and right-hand
sides at a time: every number of fields (each remainder of four, in each
column step) against the same fields fitted one by one.  The two differ only
in the order of sums over the rows, some 1e-15 of the data amplified by the
condition of the 19-column fit (up to 1e6): 1e-8 of the largest coefficient."""
import numpy as np
import pytest

from cases import CASES
from test_gpu_parity import _log, lp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("case", ["column16_flow_ragged", "sparse_cloud"])
def test_fields_together_and_alone(lp, case, k):
    import torch
    wl = CASES[case]()
    ctx = lp.make_context(wl, fit_order=3, m_max=56)
    st = lp.DeviceState.from_host(wl.state)
    ctx.lp_build_cells(st, want_perm=False)
    ctx.lp_neighbors(st, candidates=False)
    g = torch.Generator(device="cuda").manual_seed(61)
    f = torch.rand(k, wl.n, dtype=torch.float64, device="cuda", generator=g)
    signs, zero = [1] * k, [0] * k
    both, flags = ctx.lp_fit_derivs(st, f, signs, zero)
    for q in range(k):
        one, fl = ctx.lp_fit_derivs(st, f[q:q + 1], signs[q:q + 1], zero[q:q + 1])
        assert torch.equal(flags, fl)
        d = float((both[q] - one[0]).abs().amax(1).div(one[0].abs().amax(1)).max())
        _log("case %s k %d field %d: %.2e" % (case, k, q, d))
        assert d <= 1e-8
    assert np.isfinite(both.cpu().numpy()).all()
