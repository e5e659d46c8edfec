"""Candidate and stencil exports at the edges of their kernels: particle
counts around a block of the offset sums (4,096) and around 16 particles,
and periodic boxes; against the oracle, entry for entry."""
import numpy as np
import pytest

import lpgen
from cases import _periodic_layer
from test_gpu_parity import _check_neighbours, lp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 17, 4095, 4096, 4097, 8193])
def test_export_counts(lp, n):
    wl = lpgen.column_bench(seed=41, nx=21, ny=20, nz=20)
    wl.state = wl.state.take(np.arange(n))
    wl.offsets = np.array([0, n])
    print("n", n, flush=True)
    _check_neighbours(lp, wl)


@pytest.mark.parametrize("dims,axes", [((9, 9, 5), (True, True)), ((14, 9, 9), (False, True)),
                                       ((23, 11, 19), (True, False))])
def test_export_periodic(lp, dims, axes):
    _check_neighbours(lp, _periodic_layer(*dims, axes=axes, seed=43))
