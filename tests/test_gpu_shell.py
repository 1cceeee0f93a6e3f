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


@pytest.mark.parametrize("cell_div", [2, 4])
def test_cell_size_leaves_the_fp64_sets(cell_div):
    # where an FP64 build has cells (shells, wide skins), finer ones leave the exact sets
    from paper_2107_07315_amd import sph
    w = W.crust_shell(5000)
    star = W.star(3000, seed=3)
    for v, skin in ((w, 0.08), (star, 0.6)):
        out = []
        for div in (1, cell_div):
            ctx = sph.Context(v.params, capacity=v.n, skin=skin, cell_div=div)
            st = sph.DeviceState(v.arrays)
            ctx.evaluate(st)
            ctx.sph_sync()
            off, ids = ctx.sph_export_neighbours(v.n)
            order = st.numpy(["id"])["id"]
            rows = np.repeat(order, np.diff(off)).astype(np.int64)
            out.append((np.sort(rows * v.n + order[ids]), ids))
            ctx.close()
        assert np.array_equal(out[0][0], out[1][0])
        assert not np.array_equal(out[0][1], out[1][1])   # in another order: the cells did change
