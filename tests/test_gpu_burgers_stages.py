"""The right-hand side and the remainder of the Burgers steps, on columns of
four points per thread: at the edges of the 64 x 16 blocks and on the smallest
grids, against the oracle's steps (1e-10, as the other step tests); and with
spacings whose squares leave the range of the reciprocals, against the same
step scaled by a power of two, which differs by the rounding of the quotients.
"""
import numpy as np
import pytest

from oracle.phi_action import exprb32_step, exprb42_step
from paper_2310_08344_amd import binding as B
from paper_2310_08344_amd import workloads as W
from tests.gpu_helpers import dev, host, oracle_step_parity, rel, say

pytestmark = pytest.mark.gpu

PARITY = 1e-10


@pytest.fixture(scope="module")
def ctx(lx):
    c = lx.context(n_max=300 * 300, k_max=3)
    yield c
    c.close()


def _problem(nx, ny):
    dx, dy = 1.0 / nx, 1.0 / ny
    u = W.fourier_modes(max(nx, ny), seed=nx + ny)[:ny, :nx] + 0.2
    umax = float(np.max(np.abs(u)))
    nu = umax * max(dx, dy) / 2.0
    hc = W.burgers_cfl_step(nu, umax, dx, dy)
    return u, nu, dx, dy, 4.0 * hc, -1.05 / hc, 1.05 / (2.0 * hc)


@pytest.mark.parametrize("nx,ny", [(3, 3), (4, 19), (63, 5), (64, 16), (65, 17), (130, 48), (129, 33), (250, 290)])
@pytest.mark.parametrize("scheme", [32, 42])
def test_burgers_steps_match_oracle(ctx, scheme, nx, ny):
    u, nu, dx, dy, h, c, g = _problem(nx, ny)
    op = B.make_operator(kind=B.LX_OP_BURGERS2D, nx=nx, ny=ny, dx=dx, dy=dy, nu=nu)
    code, step = (B.LX_EXPRB32, exprb32_step) if scheme == 32 else (B.LX_EXPRB42, exprb42_step)
    say("burgers stages", scheme, nx, ny)
    out = dev(np.full(u.shape, np.nan))
    r = ctx.exprb_step(op, dev(u), out, h, c, g, rtol=1e-9, max_iters=300, scheme=code)
    assert r.status == B.LX_OK
    oracle_step_parity(host(out), r.iters, lambda f: step(u, nu, dx, dy, h, c, g, 1e-9, 0.0, 300, force_iters=f),
                       PARITY)


@pytest.mark.parametrize("scheme", [32, 42])
def test_burgers_steps_with_spacings_beyond_the_reciprocals(ctx, scheme):
    u, nu, dx, dy, h, c, g = _problem(96, 50)
    say("burgers stages scaled", scheme)
    code = B.LX_EXPRB32 if scheme == 32 else B.LX_EXPRB42
    got = []
    for s in (1.0, 2.0**-270):
        op = B.make_operator(kind=B.LX_OP_BURGERS2D, nx=96, ny=50, dx=dx * s, dy=dy * s, nu=nu * s)
        out = dev(np.full(u.shape, np.nan))
        r = ctx.exprb_step(op, dev(u), out, h * s, c / s, g / s, rtol=1e-9, max_iters=300, scheme=code)
        assert r.status == B.LX_OK
        got.append(host(out))
    assert rel(got[1], got[0]) <= 1e-12
