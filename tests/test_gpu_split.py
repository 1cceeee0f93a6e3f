"""FP64 pair passes of small sets, with 2 and 4 lanes to a slot list and tiles of 32: particle and tile counts
on both sides of the limits, and unions wider than one LDS chunk, against the same evaluation with 2 lanes
per target (tiles of 64, one lane to a slot list)."""
import numpy as np
import pytest

from sph_inputs import workloads as W

from parity import gpu_run

pytestmark = pytest.mark.gpu

# sums of at most 1000 terms in another order: 1000 2^-53 of the sum of their sizes, which the jitter
# keeps below 100 times the largest result
TOL = 1000 * 2.0 ** -53 * 100


@pytest.mark.parametrize("n_side,widen", [(3, 1.0), (12, 1.0), (12, 2.2), (16, 1.0), (17, 1.0), (20, 1.0), (20, 2.2),
                                          (24, 1.0), (29, 1.0), (30, 1.0)])
def test_split_tiles_give_the_same_sums(n_side, widen):
    w = W.lattice(n_side=n_side)
    rng = np.random.default_rng(n_side)
    n = w.n
    dx = 1.0 / n_side
    for k in "xyz":
        w.arrays[k] = (w.arrays[k] + rng.uniform(-0.2, 0.2, n) * dx) % 1.0
    w.arrays["h"] = np.minimum(w.arrays["h"] * widen * rng.uniform(0.95, 1.0, n), 0.124)
    w.arrays["type"] = (w.arrays["x"] < 0.6).astype(w.arrays["type"].dtype)
    w.arrays["S"] = 0.01 * rng.normal(size=w.arrays["S"].shape)
    got = gpu_run(w, ctx_kw={"max_neighbours": 2048})
    ref = gpu_run(w, ctx_kw={"max_neighbours": 2048, "lanes": 2})
    print(n_side, widen, got["_stats"], flush=True)
    assert got["_stats"]["pairs"] == ref["_stats"]["pairs"]
    for k in ("D", "ax", "ay", "az", "dudt", "dSdt"):
        err = np.abs(got[k] - ref[k]).max() / np.abs(ref[k]).max()
        assert err < TOL, (k, err)
