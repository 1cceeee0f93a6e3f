"""FP64 lists of a cluster whose particles come in no order, in a set with one particle so far away that the
whole cluster lies in a cell or two of the sort's curve: a tile of such particles has the candidates of
many places, and has to stay within what a union takes."""
import numpy as np
import pytest

from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


def _pairs(n, h, far, **kw):
    from paper_2107_07315_amd import sph
    rng = np.random.Generator(np.random.PCG64(2))
    x = rng.uniform(0.0, 1.0, (3, n))
    if far:
        x[:, n // 2] = far
    n1 = n if far else n - 1
    x = x if far else np.delete(x, n // 2, axis=1)
    arrays = dict(x=x[0].copy(), y=x[1].copy(), z=x[2].copy(), vx=np.zeros(n1), vy=np.zeros(n1), vz=np.zeros(n1),
                  u=np.full(n1, 1.5), h=np.full(n1, h), S=np.zeros((6, n1)), type=np.zeros(n1, np.int8),
                  broken=np.zeros(n1, np.uint8), id=np.arange(n1, dtype=np.int32))
    ctx = sph.Context(W.lattice(n_side=8).params.replace(periodic=False), capacity=n1, **kw)
    st = sph.DeviceState(arrays)
    ctx.evaluate(st)
    ctx.sph_sync()   # (a union or list that overflowed raises)
    s = ctx.sph_neighbour_stats()
    ctx.close()
    return s


@pytest.mark.parametrize("n,h,cap", [(20_000, 0.08, 512), (30_000, 0.069, 512), (70_000, 0.053, 512)])
@pytest.mark.parametrize("lanes", [1, 4])
def test_cluster_with_a_particle_far_away(n, h, cap, lanes):
    kw = dict(lanes=lanes, max_neighbours=cap, skin=0.08)
    a, b = _pairs(n, h, 1e5, **kw), _pairs(n, h, 0.0, **kw)
    print(n, h, lanes, a, b, flush=True)
    assert a["pairs"] == b["pairs"]
