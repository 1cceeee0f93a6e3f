"""FP64 lists on both sides of the size from which the build takes the cell grid: the neighbour counts are
those of the FP32 build (whose sets are the exact ones too), and above the size its tiles."""
import numpy as np
import pytest

from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,grid", [(2 ** 23, False), (2 ** 23 + 1, True)])
def test_neighbours_of_a_large_set(n, grid):
    from paper_2107_07315_amd import sph
    x = np.random.Generator(np.random.PCG64(3)).random((3, n))
    arrays = dict(x=x[0], y=x[1], z=x[2], vx=np.zeros(n), vy=np.zeros(n), vz=np.zeros(n), u=np.full(n, 1.5),
                  h=np.full(n, 0.0045), S=np.zeros((6, n)), type=np.zeros(n, np.int8), broken=np.zeros(n, np.uint8),
                  id=np.arange(n, dtype=np.int32))
    out = []
    for precision in ("FP64", "FP32"):
        p = W.lattice(n_side=8).params.replace(precision=precision, periodic=False)
        ctx = sph.Context(p, capacity=n, skin=0.05, max_neighbours=100)
        st = sph.DeviceState(arrays)
        ctx.evaluate(st)
        ctx.sph_sync()
        out.append(ctx.sph_neighbour_stats())
        print(n, precision, out[-1], flush=True)
        ctx.close()
        del st
    assert out[0]["pairs"] == out[1]["pairs"] and out[0]["max_count"] == out[1]["max_count"]
    assert (out[0]["tiles"] == out[1]["tiles"] and out[0]["candidates"] == out[1]["candidates"]) == grid
