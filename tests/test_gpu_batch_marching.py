"""Batches by register marching (the default where every side is even and at
least 10): at the edges of strips (116 output columns of a window of six, 120
of four, 108 of a power launch) and bands, down to the smallest grids, against
the oracle, against one iteration per launch, and the power iteration at the
edges of its launches of ten sweeps.

Outputs are the one-iteration loop's bit for bit when the counts agree (the
same terms in the same order); parity with the oracle 1e-10 and the spectral
estimate 1e-12, as in the other batch tests.
"""
import numpy as np
import pytest

from oracle.phi_action import leja_phi, power_iteration, shift_scale
from paper_2310_08344_amd import binding as B
from tests.gpu_helpers import dev, host, oracle_parity, rel, say
from tests.test_gpu_batch import _mixed_batch, _run, splitmix_vector

pytestmark = pytest.mark.gpu

PARITY = 1e-10

DA = [(10, 10, "da"), (12, 11, "da"), (116, 24, "da"), (118, 40, "da"), (128, 17, "da"), (232, 33, "da"),
      (234, 10, "da"), (64, 96, "da"), (16, 130, "da"), (348, 20, "da")]
BOTH = DA[:6] + [(10, 12, "bu"), (120, 24, "bu"), (122, 40, "bu"), (240, 16, "bu"), (66, 34, "bu")]


@pytest.fixture(scope="module")
def ctx(lx):
    c = lx.context(n_max=1 << 16, k_max=1)
    yield c
    c.close()


@pytest.mark.parametrize("specs,depth", [(DA, 6), (BOTH, 4), (DA[:1], 6), (BOTH[6:7], 4)])
def test_marching_batch_matches_oracle_and_single_iterations(ctx, specs, depth):
    inst = _mixed_batch(21, specs)
    say("marching batch", len(specs), depth)
    st, res, outs = _run(ctx, inst, rtol=1e-9, max_iters=250)
    assert st == B.LX_OK and ctx.stats()["marching"] == 1 and ctx.stats()["depth"] == depth
    ctx.set_depth(1)
    try:
        st1, res1, outs1 = _run(ctx, inst, rtol=1e-9, max_iters=250)
    finally:
        ctx.set_depth(0)
    for q, r, r1, o, o1 in zip(inst, res, res1, outs, outs1):
        oracle_parity([o], [r["iters"]],
                      lambda f, q=q: leja_phi(q["A"], q["v"], [(q["l"], 1.0, 1.0)], q["h"], q["c"], q["gamma"],
                                              1e-9, 0.0, 250, f), PARITY)
        if r["iters"] == r1["iters"]:
            assert np.array_equal(o, o1)


def test_marching_batch_budgets(ctx):
    """Budgets that end at every position of a window of six and of four."""
    inst = _mixed_batch(22, BOTH)
    budgets = [1, 2, 3, 4, 5, 6, 1, 3, 4, 5, 8]
    say("marching budgets")
    st, res, outs = _run(ctx, inst, budgets=budgets, rtol=1e-13, max_iters=250)
    assert st == B.LX_ENOTCONV and ctx.stats()["marching"] == 1
    for q, b, r, o in zip(inst, budgets, res, outs):
        assert r["status"] == B.LX_ENOTCONV and r["iters"] == b
        ref = leja_phi(q["A"], q["v"], [(q["l"], 1.0, 1.0)], q["h"], q["c"], q["gamma"], 1e-13, 0.0, b)
        assert rel(o, ref.p[0]) <= PARITY


@pytest.mark.parametrize("iters", [1, 2, 9, 10, 11, 20, 21])
def test_marching_batch_power_iteration(ctx, iters):
    """Given and own start vectors in one batch, twice (the second call
    replays the captured pipeline)."""
    inst = _mixed_batch(23, BOTH)
    rng = np.random.default_rng(iters)
    x0s = [rng.standard_normal((q["ny"], q["nx"])) * 1e3 if i % 2 else None for i, q in enumerate(inst)]
    say("marching power", iters)
    for _ in range(2):
        st, res, outs = _run(ctx, inst, power_iters=iters, x0s=x0s, rtol=1e-6, max_iters=400, raise_on_error=False)
        assert ctx.stats()["marching"] == 1
        for i, (q, r) in enumerate(zip(inst, res)):
            x0 = x0s[i] if x0s[i] is not None else splitmix_vector(i, q["nx"] * q["ny"]).reshape(q["ny"], q["nx"])
            rho, _ = power_iteration(q["A"], x0, iters)
            assert abs(r["rho_hat"] - rho) <= 1e-12 * rho
            c, g = shift_scale(r["rho_hat"])
            assert r["c"] == c and r["gamma"] == g


def test_marching_batch_beyond_the_cache(ctx):
    """More than 2^23 points: Burgers windows of six; bit for bit one
    iteration per launch on a sample of the batch."""
    specs = [(512, 420, "bu" if i % 2 else "da") for i in range(40)]
    inst = _mixed_batch(24, specs[:4])
    inst = [inst[i % 4] for i in range(40)]
    say("marching deep")
    st, res, outs = _run(ctx, inst, rtol=1e-9, max_iters=250)
    assert st == B.LX_OK and ctx.stats()["marching"] == 1 and ctx.stats()["depth"] == 6
    ctx.set_depth(1)
    try:
        st1, res1, outs1 = _run(ctx, inst[:4], rtol=1e-9, max_iters=250)
    finally:
        ctx.set_depth(0)
    for i in range(40):
        assert res[i]["iters"] == res[i % 4]["iters"] and np.array_equal(outs[i], outs[i % 4])
    for i in range(4):
        if res[i]["iters"] == res1[i]["iters"]:
            assert np.array_equal(outs[i], outs1[i])
        else:
            assert abs(res[i]["iters"] - res1[i]["iters"]) == 1 and rel(outs[i], outs1[i]) <= 1e-8
