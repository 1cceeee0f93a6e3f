"""EoS network training kernels over the range of batch sizes: the gradient against the oracle where the
sum over the workgroups' partials has one, several and incomplete chunks, and the operand packs that an
Adam step leaves against those that loading the same weights makes."""
import numpy as np
import pytest

import oracle
from sph_inputs import eos_table as E
from test_gpu_mlp import BLOCKS, TOL_GRAD, _ctx, _domain, _to_dev

pytestmark = pytest.mark.gpu


def _batch(n):
    rng = np.random.default_rng(n)
    return rng.uniform(-1, 1, (n, 2)).astype(np.float32), rng.uniform(-1, 1, (n, 2)).astype(np.float32)


@pytest.mark.parametrize("n", [4032, 4096, 4160, 8192])
def test_gradient_sums_every_partial(n):
    _, ctx, _ = _ctx()
    ctx.mlp_set_params(E.mlp_init(4))
    wr = ctx.mlp_get_params(rounded=True).astype(np.float64)
    x, t = _batch(n)
    g, loss = ctx.mlp_grad(_to_dev(x, np.float32), _to_dev(t, np.float32))
    lo, go = oracle.mlp_loss_grad(wr, x.astype(np.float64), t.astype(np.float64))
    assert abs(loss - lo) <= TOL_GRAD * lo
    for k, (a, b) in BLOCKS.items():
        err = float(np.linalg.norm(g[a:b] - go[a:b]) / np.linalg.norm(go[a:b]))
        print(f"n={n} {k} {err:.2e}", flush=True)
        assert err < TOL_GRAD, (k, err)
    ctx.close()


@pytest.mark.parametrize("batch", [64, 4160])
def test_adam_step_leaves_the_packs_of_its_weights(batch):
    _, ctx, _ = _ctx()
    pp, lo, hi, wd, dom = _domain()
    ctx.mlp_set_domain(*dom)
    ctx.mlp_set_params(E.mlp_init(4))
    s = E.mlp_band_samples(pp, lo, hi, wd, 2 * batch, 4)
    ctx.mlp_train(_to_dev(s, np.float64), 0, 1, batch, 1e-3)
    x, t = (_to_dev(v, np.float32) for v in _batch(320))
    g, loss = ctx.mlp_grad(x, t)
    _, other, _ = _ctx()
    other.mlp_set_domain(*dom)
    other.mlp_set_params(ctx.mlp_get_params(rounded=False))
    assert np.array_equal(other.mlp_get_params(rounded=True), ctx.mlp_get_params(rounded=True))
    g2, loss2 = other.mlp_grad(x, t)
    assert loss == loss2 and np.array_equal(g, g2)
    ctx.close()
    other.close()
