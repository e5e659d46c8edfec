"""A captured step sequence belongs to the kind of system it was captured
for: a context that goes from open to periodic systems (or back) with the
same sizes, arrays and step captures anew, and steps as a fresh context
does, bit for bit."""
import dataclasses

import pytest

import lpgen
from cases import _periodic_layer
from test_gpu_parity import lp  # noqa: F401

pytestmark = pytest.mark.gpu


def _params(wl, periodic):
    return wl.params if periodic else [dataclasses.replace(p, box_len=(0.0, 0.0))
                                       for p in wl.params]


@pytest.mark.parametrize("first", [False, True])
def test_captured_steps_follow_the_periodic_axes(lp, first):
    import torch
    # (the open y axis is the longest either way: the sort keys keep their width)
    wl = _periodic_layer(12, 20, 9, axes=(True, False), seed=71)
    print("periodic first:", first, flush=True)
    ctx = lp.Context()
    ctx.reserve(wl.n)
    st = lp.DeviceState.from_host(wl.state)
    for periodic in (first, not first, first):
        for a, b in zip(st.t, wl.state.arrays()):
            a.copy_(torch.from_numpy(b))
        ctx.set_systems(list(wl.offsets), _params(wl, periodic))
        ref = lp.make_context(lpgen.Workload("ref", wl.state, wl.offsets,
                                             _params(wl, periodic), wl.dt, 1))
        want = lp.DeviceState.from_host(wl.state)
        for c, s in ((ctx, st), (ref, want)):
            c.lp_step_graph(s, wl.dt, 3)
            c.sync_status()
        for name, a, b in zip(lp.DeviceState.NAMES, st.t, want.t):
            assert torch.equal(a, b), (periodic, name)
