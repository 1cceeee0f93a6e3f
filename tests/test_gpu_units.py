"""FP64 results do not depend on the caller's unit of length: with lengths, and masses as their cubes, scaled
by a power of two every operation scales exactly, so lists and fields are the unit's bit for bit."""
import numpy as np
import pytest

from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


def _run(scale, shell, box):
    from paper_2107_07315_amd import sph
    rng = np.random.Generator(np.random.PCG64(4))
    n = 3000
    x = np.round(rng.uniform(0.0, 1.0, (3, n)) * 2.0 ** 20) * 2.0 ** -20
    h = 0.04 * rng.uniform(0.7, 1.0, n) ** (3 if box else 12)
    typ = (x[0] < 0.5).astype(np.int8)
    S = rng.normal(scale=0.01, size=(6, n)) * (typ == 1)
    X = x * scale
    arrays = dict(x=X[0].copy(), y=X[1].copy(), z=X[2].copy(), vx=rng.normal(scale=0.1, size=n),
                  vy=rng.normal(scale=0.1, size=n), vz=rng.normal(scale=0.1, size=n), u=np.full(n, 1.5), h=h * scale,
                  S=S, type=typ, broken=np.zeros(n, np.uint8), id=np.arange(n, dtype=np.int32))
    p = W.lattice(n_side=8).params.replace(periodic=box, box=scale, m=scale ** 3 / n, wall_in=1e-6 * scale if shell else 0.0)
    ctx = sph.Context(p, capacity=n, skin=0.08)
    st = sph.DeviceState(arrays)
    ctx.evaluate(st)
    ctx.sph_sync()
    off, ids = ctx.sph_export_neighbours(n)
    g = st.numpy()
    ctx.close()
    return off, ids, {k: g[k] for k in ("D", "P", "ax", "ay", "az", "dudt", "dSdt", "id")}


@pytest.mark.parametrize("bits", [-90, -70, -40, 33, 66, 90])
@pytest.mark.parametrize("shell,box", [(False, False), (False, True), (True, False)])
def test_unit_of_length(bits, shell, box):
    scale = 2.0 ** bits
    a, b = _run(1.0, shell, box), _run(scale, shell, box)
    print(bits, shell, box, "pairs", a[0][-1], b[0][-1], flush=True)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    for k, v in a[2].items():   # accelerations and the rates go with the velocities over the length
        w = b[2][k] * (scale if k in ("ax", "ay", "az", "dudt", "dSdt") else 1.0)
        assert np.array_equal(v, w), (k, np.abs(v - w).max())
