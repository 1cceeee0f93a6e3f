"""A shell between an inner and an outer wall keeps the order of its pair sums in FP64, whatever its size:
its tiles and the order of its neighbour lists are the cell grid's, as in FP32.  (The slab fit of the
oscillation record amplifies the rounding of the sums by many orders where all particles lie in one layer.)"""
import numpy as np
import pytest

from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


def _lists(w, precision, lanes):
    from paper_2107_07315_amd import sph
    ctx = sph.Context(w.params.replace(precision=precision), capacity=w.n, skin=0.1, lanes=lanes)
    st = sph.DeviceState(w.arrays)
    ctx.evaluate(st)
    ctx.sph_sync()
    off, ids = ctx.sph_export_neighbours(w.n)
    out = off, ids, st.numpy(["id"])["id"], ctx.sph_neighbour_stats()["tiles"]
    ctx.close()
    return out


@pytest.mark.parametrize("n,solid,lanes", [(3000, True, 4), (21_000, True, 4), (21_000, False, 2), (40_000, True, 4)])
def test_shell_lists_keep_the_grids_order(n, solid, lanes):
    w = W.crust_shell(n, solid=solid)
    a, b = _lists(w, "FP64", lanes), _lists(w, "FP32", lanes)
    print(n, solid, lanes, "tiles", a[3], b[3], "pairs", a[0][-1], flush=True)
    assert a[3] == b[3]
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)
