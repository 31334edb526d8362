"""The training kernels at the edges of their split: minibatches below, at
and above the samples one wavefront, one workgroup and one load-ahead batch
take, and one larger than the forward kernel's grid.

The gradient is the mean of the per-sample gradients.  Both sides round
every product and sum to float32; the longest sum has 64 terms, so their
difference is at most about 66 * 2^-24 = 4e-6 of the sum of the moduli, and
1e-5 of the mean per-sample norm bounds it.
"""
import numpy as np
import pytest

from oracle.mlp import N_PARAMS
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


def _f32(x):
    import torch
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.float32)).to("cuda:0")


@pytest.fixture(scope="module")
def pred(lx):
    c = lx.context(n_max=1 << 10, k_max=1)
    p = c.predictor(seed=3)
    s = p.get_state()
    s[:N_PARAMS] = np.random.default_rng(0).standard_normal(N_PARAMS).astype(np.float32) * 0.2
    p.set_state(s)
    yield p
    p.close()
    c.close()


@pytest.mark.parametrize("n", [1, 2, 4, 5, 31, 32, 33, 65])
def test_gradient_is_the_mean_of_the_samples(pred, n):
    rng = np.random.default_rng(n)
    X, T = rng.standard_normal((n, 8)), rng.standard_normal((n, 2))
    say("mlp gradient of", n)
    loss, g = pred.gradient(_f32(X), _f32(T))
    each = [pred.gradient(_f32(X[i:i + 1]), _f32(T[i:i + 1])) for i in range(n)]
    assert abs(loss - np.mean([e[0] for e in each])) <= 1e-5 * loss
    d = g.astype(np.float64) - np.mean([e[1].astype(np.float64) for e in each], axis=0)
    assert np.linalg.norm(d) <= 1e-5 * np.mean([np.linalg.norm(e[1]) for e in each])


def test_gradient_of_more_samples_than_one_grid(pred):
    rng = np.random.default_rng(9)
    X, T = rng.standard_normal((5, 8)), rng.standard_normal((5, 2))
    say("mlp gradient of 4100")
    loss5, g5 = pred.gradient(_f32(X), _f32(T))
    loss, g = pred.gradient(_f32(np.tile(X, (820, 1))), _f32(np.tile(T, (820, 1))))
    assert abs(loss - loss5) <= 1e-5 * loss5
    assert np.linalg.norm(g.astype(np.float64) - g5) <= 1e-5 * np.linalg.norm(g5)
