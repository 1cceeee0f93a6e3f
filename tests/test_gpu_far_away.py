"""FP64 passes far from the origin: the records that pad a walk lie nowhere near a particle, wherever the
particles are."""
import numpy as np
import pytest

from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


def _run(shift, lanes, n):
    from paper_2107_07315_amd import sph
    rng = np.random.Generator(np.random.PCG64(4))
    x = np.round(rng.uniform(0.0, 1.0, (3, n)) * 2.0 ** 15) * 2.0 ** -15 + shift   # exact at 2e10 too
    typ = (x[0] < shift + 0.5).astype(np.int8)
    arrays = dict(x=x[0].copy(), y=x[1].copy(), z=x[2].copy(), vx=rng.normal(scale=0.1, size=n),
                  vy=rng.normal(scale=0.1, size=n), vz=rng.normal(scale=0.1, size=n), u=np.full(n, 1.5),
                  h=0.06 * rng.uniform(0.7, 1.0, n), S=rng.normal(scale=0.01, size=(6, n)) * (typ == 1), type=typ,
                  broken=np.zeros(n, np.uint8), id=np.arange(n, dtype=np.int32))
    p = W.lattice(n_side=8).params.replace(periodic=False, m=1.0 / n)
    ctx = sph.Context(p, capacity=n, lanes=lanes)
    st = sph.DeviceState(arrays)
    ctx.evaluate(st)
    ctx.sph_sync()
    pairs = ctx.sph_neighbour_stats()["pairs"]
    g = st.numpy()
    ctx.close()
    return pairs, {k: g[k] for k in ("D", "ax", "ay", "az", "dudt", "dSdt", "id")}


@pytest.mark.parametrize("lanes,n", [(4, 2500), (1, 2500), (4, 30_000)])
def test_around_1e10(lanes, n):
    a, b = _run(1e10 - 0.5, lanes, n), _run(2e10 - 0.5, lanes, n)
    print(lanes, n, "pairs", a[0], b[0], flush=True)
    assert a[0] == b[0]
    for k, v in a[1].items():   # the same sums but for the order of a few terms
        assert np.abs(v - b[1][k]).max() <= 1e-12 * np.abs(b[1][k]).max(), k
