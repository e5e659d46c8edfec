"""The tile map (distinct list sources of each 256-particle tile, by
granules of 16 ids) at its edges: particle counts around one and two tiles
and around a granule, and columns whose tiles have fewer and more sources
than are staged, in one launch.  The staged fits number their rows by it, so
a wrong slot, a missing source or a word past a list that is taken for a
source shows against the global-gather step, which reads ids.  Same rows,
same order, same arithmetic: 1e-12 relative leaves room for the compiler's
different scheduling of the two paths only."""
import dataclasses

import numpy as np
import pytest

import lpgen
from test_gpu_parity import _log, lp  # noqa: F401
from test_gpu_staging import _compare, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 17, 255, 256, 257, 513, 1000])
def test_tile_map_counts(lp, n):
    wl = lpgen.column_bench(seed=17, nx=10, ny=10, nz=10)
    wl.state = wl.state.take(np.arange(n))
    wl.offsets = np.array([0, n])
    print("n", n, flush=True)
    got, st = _run(lp, wl, 2)
    ref, _ = _run(lp, wl, 2, debug_flags=lp.LP_DEBUG_GLOBAL_GATHER)
    _log("stats %s" % st)
    assert st["tiles"] == (n + 255) // 256 and st["unstaged_tiles"] == 0
    _compare(got, ref, "n %d" % n)


@pytest.mark.parametrize("scale", [1.1, 1.2, 1.3])
def test_tile_map_around_the_staged_size(lp, scale):
    wl = lpgen.column_bench(seed=18, nx=20, ny=20, nz=20)
    h = wl.params[0].h * scale
    wl.params = [dataclasses.replace(p, h=h, R=2.5 * h) for p in wl.params]
    print("scale", scale, flush=True)
    got, st = _run(lp, wl, 1)
    ref, _ = _run(lp, wl, 1, debug_flags=lp.LP_DEBUG_GLOBAL_GATHER)
    _log("stats %s" % st)
    _compare(got, ref, "scale %g" % scale)
