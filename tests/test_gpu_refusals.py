"""What a list build refuses, with a reason that names it: smoothing lengths that are not positive, a box too
small for them, a set too wide for them (beyond what an int counts in cells, and infinite).  A set within
the limit is taken."""
import numpy as np
import pytest

from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


def _sync(box, h, far, precision):
    from paper_2107_07315_amd import sph
    n = 200
    x = np.random.default_rng(1).uniform(0.0, 1.0, (3, n))
    x[0, 0] = far
    arrays = dict(x=x[0].copy(), y=x[1].copy(), z=x[2].copy(), vx=np.zeros(n), vy=np.zeros(n), vz=np.zeros(n),
                  u=np.full(n, 1.5), h=np.full(n, h), S=np.zeros((6, n)), type=np.zeros(n, np.int8),
                  broken=np.zeros(n, np.uint8), id=np.arange(n, dtype=np.int32))
    ctx = sph.Context(W.lattice(n_side=8).params.replace(precision=precision, periodic=box), capacity=n)
    st = sph.DeviceState(arrays)
    ctx.sph_build_cells(st)
    ctx.sph_sync()
    ctx.close()


@pytest.mark.parametrize("precision", ["FP64", "FP32"])
@pytest.mark.parametrize("box,h,far", [(True, 0.3, 0.5), (False, 0.1, 1e12), (False, 0.1, np.inf), (False, -0.1, 0.5),
                                       (False, 0.0, 0.5)])
def test_refused(box, h, far, precision):
    from paper_2107_07315_amd import sph
    print(box, h, far, precision, flush=True)
    with pytest.raises(sph.SphError) as e:
        _sync(box, h, far, precision)
    assert e.value.code == 1
    assert all(w in e.value.detail for w in ("box too small", "not positive", "too wide")), e.value.detail


@pytest.mark.parametrize("precision", ["FP64", "FP32"])
@pytest.mark.parametrize("far", [5e3, 5e7])
def test_wide_sets_are_taken(far, precision):
    _sync(False, 0.1, far, precision)
