"""Candidate-list build: the exact neighbour sets of the evaluation equal a brute-force FP64 search on
inputs at the edges of the build: single particles and ragged tiles, smoothing lengths a factor of 100
apart (beyond the range of the matrix-core test, which then tests pair by pair), particles far
outside a cluster, many particles in one place, periodic boxes down to a few supports across, 1, 2 and
4 lanes per target, both precisions, no skin and a large one."""
import numpy as np
import pytest

from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


def _cloud(name, rng):
    """positions (3, n), h (n), periodic box or 0"""
    def box(n, h, L=1.0):
        return rng.uniform(0.0, L, (3, n)), np.full(n, h), 0.0
    if name == "one":
        return box(1, 0.1)
    if name == "ragged":            # 2 x 64 + 1 particles
        return box(129, 0.15)
    if name == "tiles":             # many tiles, several runs of 64 of them
        return box(9001, 0.045)
    if name == "wide_h":            # h over a factor of 100 in one place
        x, h, _ = box(3000, 0.02)
        h = 0.02 * 100.0 ** (rng.uniform(0.0, 1.0, 3000) ** 8)
        return x, np.minimum(h, 0.25), 0.0
    if name == "outliers":          # a cluster, a few particles 1e4 of its sizes away
        x, h, _ = box(1500, 0.08)
        x[:, :5] = 1e4 * rng.normal(size=(3, 5))
        return x, h, 0.0
    if name == "pile":              # coincident particles and a line of large h across them
        x, h, _ = box(700, 0.06)
        x[:, 100:140] = x[:, 100:101]
        h[140:150] = 0.4
        return x, h, 0.0
    if name == "periodic":
        x = rng.uniform(0.0, 1.0, (3, 2500))
        return x, rng.uniform(0.03, 0.07, 2500), 1.0
    x = rng.uniform(0.0, 1.0, (3, 400))   # periodic_small: the support is just below a quarter box
    return x, np.full(400, 0.12), 1.0


def _brute(x, h, box, s1=1.0):
    n = h.size
    out = []
    for a in range(n):
        d = x[:, a, None] - x
        if box > 0:
            d = np.where(d > 0.5 * box, d - box, np.where(d < -0.5 * box, d + box, d))
        r2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
        H = (h[a] + h) * s1
        hit = r2 < H * H
        hit[a] = False
        out.append(np.nonzero(hit)[0])
    return out


def _evaluate(name, precision, lanes, skin):
    from paper_2107_07315_amd import sph
    x, h, box = _cloud(name, np.random.Generator(np.random.PCG64(7)))
    n = h.size
    w = W.lattice(n_side=8)
    arrays = dict(x=x[0].copy(), y=x[1].copy(), z=x[2].copy(), vx=np.zeros(n), vy=np.zeros(n), vz=np.zeros(n),
                  u=np.full(n, 1.5), h=h.copy(), S=np.zeros((6, n)), type=np.zeros(n, np.int8),
                  broken=np.zeros(n, np.uint8), id=np.arange(n, dtype=np.int32))
    p = w.params.replace(precision=precision, periodic=box > 0, box=box)
    ctx = sph.Context(p, capacity=n, skin=skin, lanes=lanes, max_neighbours=2048)
    st = sph.DeviceState(arrays)
    ctx.evaluate(st)
    ctx.sph_sync()
    return ctx, st, x, h, box


@pytest.mark.parametrize("name", ["one", "ragged", "tiles", "wide_h", "outliers", "pile", "periodic", "periodic_small"])
@pytest.mark.parametrize("precision,lanes,skin", [("FP64", 4, 0.08), ("FP32", 4, 0.14), ("FP64", 1, 0.0), ("FP32", 2, 0.3)])
def test_lists_equal_brute_force(name, precision, lanes, skin):
    ctx, st, x, h, box = _evaluate(name, precision, lanes, skin)
    n = h.size
    off, ids = ctx.sph_export_neighbours(n)
    order = st.numpy(["id"])["id"]
    want = _brute(x, h, box)
    print(name, precision, lanes, skin, "pairs", off[n], flush=True)
    for k in range(n):
        got = np.sort(order[ids[off[k]:off[k + 1]]])
        assert np.array_equal(got, want[order[k]]), (name, k, got.size, want[order[k]].size)
    s = ctx.sph_neighbour_stats()
    assert s["pairs"] == sum(v.size for v in want)
    assert s["candidates"] >= s["pairs"]
    ctx.close()


@pytest.mark.parametrize("name", ["ragged", "tiles", "wide_h", "outliers", "pile", "periodic", "periodic_small"])
def test_fp32_candidates_are_the_fp64_decision(name):
    """The FP32 lists decide the order of the FP32 sums, so they hold the candidates of the FP64 test at
    the skin-widened support and no others (the matrix-core test leaves the close pairs to it)."""
    skin = 0.14
    ctx, _, x, h, box = _evaluate(name, "FP32", 4, skin)
    want = sum(v.size for v in _brute(x, h, box, 1.0 + skin))
    assert ctx.sph_neighbour_stats()["candidates"] == want
    ctx.close()
