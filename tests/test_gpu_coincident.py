"""Forces on coincident particles without the viscosity's eps term (visc_eps = 0): the pair's terms are
zero, in every form of the force pass, and the others are those of the oracle."""
import numpy as np
import pytest

import oracle
from parity import eval_errors, gpu_run, oracle_run
from sph_inputs import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,lanes,tol", [("FP64", 4, 1e-12), ("FP64", 2, 1e-12), ("FP64", 1, 1e-12),
                                                 ("FP32", 4, 1e-4)])
@pytest.mark.parametrize("solid", [True, False])
def test_coincident_particles_without_eps(precision, lanes, tol, solid):
    w = W.lattice(n_side=9)
    rng = np.random.default_rng(3)
    for k in "xyz":
        w.arrays[k] = (w.arrays[k] + rng.uniform(-0.2, 0.2, w.n) / 9.0) % 1.0
        w.arrays[k][[7, 300, 301]] = w.arrays[k][[6, 299, 299]]
    if not solid:
        w.arrays["type"][:] = 0
    p = w.params.replace(visc_eps=0.0)
    g = gpu_run(w, precision=precision, params=p, ctx_kw={"lanes": lanes})   # (a latched NaN raises)
    e = eval_errors(g, oracle_run(w, mode=oracle.BRUTE, params=p))
    print(precision, lanes, solid, {k: f"{v:.1e}" for k, v in e.items()}, flush=True)
    for k, v in e.items():
        assert v <= tol, (k, v)
