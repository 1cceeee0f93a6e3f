"""Candidate lists at the edge of the support: pairs a relative 1e-8 to 1e-3 inside and outside of it, in
tiles that mix smoothing lengths up to a factor of 1e6 apart, against a brute-force FP64 search."""
import numpy as np
import pytest

from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


def edge_pairs(ratio, n=640, seed=0):
    """A cloud of n particles of one h, some placed just inside and just outside another's support, and
    one particle in each corner of it whose h is ratio times theirs: positions (3, n + 8), h."""
    rng = np.random.Generator(np.random.PCG64(seed))
    h = rng.uniform(0.7, 1.0, n)
    x = rng.uniform(0.0, 14.0, (3, n))
    k = n // 2
    u = rng.normal(size=(3, k))
    u /= np.sqrt((u * u).sum(0))
    off = 10.0 ** rng.uniform(-8.0, -3.0, k) * np.where(rng.uniform(size=k) < 0.8, -1.0, 1.0)
    x[:, k:] = x[:, :k] + u * ((h[:k] + h[k:]) * (1.0 + off))
    c = 3.0 + 8.0 * np.array([[i >> d & 1 for i in range(8)] for d in range(3)])
    return np.concatenate([x, c], axis=1), np.concatenate([h, np.full(8, ratio)])


def lists(x, h, precision, lanes, skin):
    from paper_2107_07315_amd import sph
    n = h.size
    arrays = dict(x=x[0].copy(), y=x[1].copy(), z=x[2].copy(), vx=np.zeros(n), vy=np.zeros(n), vz=np.zeros(n),
                  u=np.full(n, 1.5), h=h.copy(), S=np.zeros((6, n)), type=np.zeros(n, np.int8),
                  broken=np.zeros(n, np.uint8), id=np.arange(n, dtype=np.int32))
    p = W.lattice(n_side=8).params.replace(precision=precision, periodic=False)
    ctx = sph.Context(p, capacity=n, skin=skin, lanes=lanes, max_neighbours=2048)
    st = sph.DeviceState(arrays)
    ctx.evaluate(st)
    ctx.sph_sync()
    off, ids = ctx.sph_export_neighbours(n)
    order = st.numpy(["id"])["id"]
    out = [None] * n
    for k in range(n):
        out[order[k]] = np.sort(order[ids[off[k]:off[k + 1]]])
    ctx.close()
    return out


def brute(x, h):
    out = []
    for a in range(h.size):
        d = x[:, a, None] - x
        H = h[a] + h
        hit = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2] < H * H
        hit[a] = False
        out.append(np.nonzero(hit)[0])
    return out


@pytest.mark.parametrize("ratio", [1.0, 20.0, 150.0, 300.0, 3e3, 1e4, 1e6])
@pytest.mark.parametrize("precision,lanes,skin", [("FP64", 4, 0.0), ("FP64", 1, 0.08), ("FP32", 4, 0.0)])
def test_pairs_at_the_edge_of_the_support(ratio, precision, lanes, skin):
    for seed in range(4):
        x, h = edge_pairs(ratio, seed=seed)
        got, want = lists(x, h, precision, lanes, skin), brute(x, h)
        print(ratio, precision, lanes, skin, seed, sum(v.size for v in want), flush=True)
        for a in range(h.size):
            assert np.array_equal(got[a], want[a]), (seed, a, np.setxor1d(got[a], want[a]))
