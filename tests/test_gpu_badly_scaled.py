"""Power iteration of operators far from 1 in size: several sweeps without a
normalisation between them must not leave the range of a double."""
import numpy as np
import pytest

from oracle.operators import diffadv_apply
from oracle.phi_action import leja_phi, power_iteration, shift_scale
from paper_2310_08344_amd import binding as B
from tests.gpu_helpers import dev, diffadv_setup, oracle_parity, say
from tests.test_gpu_batch import _mixed_batch, _run, splitmix_vector

pytestmark = pytest.mark.gpu

PARITY = 1e-10


@pytest.fixture(scope="module")
def ctx(lx):
    c = lx.context(n_max=1 << 16, k_max=1)
    yield c
    c.close()


@pytest.mark.parametrize("scale", [1e-120, 1e-56, 1e-20, 1e-17, 1e20, 1e100])
def test_marching_batch_of_badly_scaled_operators(ctx, scale):
    """Operators of 1e-113 to 1e105 beside one of ordinary size, with given and
    own start vectors: estimates to 1e-12, outputs as the other batch tests."""
    inst = _mixed_batch(31, [(64, 64, "da"), (64, 48, "da"), (118, 40, "da"), (12, 11, "da")])
    for q in inst[:3]:
        q["op"].D, q["op"].vx, q["op"].vy = q["op"].D * scale, q["op"].vx * scale, q["op"].vy * scale
        q["A"] = (lambda A: lambda y: scale * A(y))(q["A"])
        q["h"] /= scale
    rng = np.random.default_rng(9)
    x0s = [rng.standard_normal((q["ny"], q["nx"])) if i == 1 else None for i, q in enumerate(inst)]
    say("badly scaled batch", scale)
    st, res, outs = _run(ctx, inst, power_iters=20, x0s=x0s, rtol=1e-9, max_iters=400)
    assert st == B.LX_OK and ctx.stats()["marching"] == 1
    for i, (q, r, o) in enumerate(zip(inst, res, outs)):
        x0 = x0s[i] if x0s[i] is not None else splitmix_vector(i, q["nx"] * q["ny"]).reshape(q["ny"], q["nx"])
        rho, _ = power_iteration(q["A"], x0, 20)
        assert abs(r["rho_hat"] - rho) <= 1e-12 * rho
        c, g = shift_scale(r["rho_hat"])
        assert r["c"] == c and r["gamma"] == g
        oracle_parity([o], [r["iters"]],
                      lambda f, q=q: leja_phi(q["A"], q["v"], [(q["l"], 1.0, 1.0)], q["h"], c, g, 1e-9, 0.0, 400, f),
                      PARITY)


@pytest.mark.parametrize("scale", [1e-150, 1e-56, 1e-20, 1e30, 1e100])
@pytest.mark.parametrize("nx,ny,march", [(64, 48, False), (65, 48, False), (64, 48, True), (2048, 700, False)])
@pytest.mark.parametrize("given", [True, False])
def test_spectrum_of_badly_scaled_operators(lx, nx, ny, march, scale, given):
    """Even and odd grids, on register tiles and by marching (forced, and the
    automatic choice of a grid this large)."""
    rng = np.random.default_rng(11)
    prm, _ = diffadv_setup(nx, ny, vx=0.7 * nx, vy=-0.4 * ny)
    op = B.make_operator(kind=B.LX_OP_DIFFADV2D, nx=nx, ny=ny, dx=prm["dx"], dy=prm["dy"], D=prm["D"] * scale,
                         vx=prm["vx"] * scale, vy=prm["vy"] * scale)
    x0 = rng.standard_normal((ny, nx)) if given else splitmix_vector(0, nx * ny).reshape(ny, nx)
    rho_o, _ = power_iteration(lambda y: diffadv_apply(y, prm["D"], prm["vx"], prm["vy"], prm["dx"], prm["dy"]), x0, 20)
    say("badly scaled spectrum", nx, ny, march, scale, given)
    with lx.context(n_max=nx * ny, k_max=1) as c:
        if march:
            c.set_window_kernel(2)
        rho, _, _ = c.spectrum(op, x0=dev(x0) if given else None, iters=20)
        assert c.stats()["marching"] == int(march or nx == 2048)
    assert abs(rho - rho_o * scale) <= 1e-12 * rho_o * scale
