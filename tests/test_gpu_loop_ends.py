"""The end of a loop on register tiles: the launches past it, and the
workgroups beside the tiles that form coefficients no launch will read."""
import numpy as np
import pytest

from paper_2310_08344_amd import binding as B
from tests.gpu_helpers import closed_form_shift, dev, diffadv_setup, host, rel, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lx):
    c = lx.context(n_max=256 * 256, k_max=3)
    yield c
    c.close()


def _problem(nx, ny, cfl):
    prm, h = diffadv_setup(nx, ny, cfl=cfl)
    c, g = closed_form_shift(prm["D"], prm["vx"], prm["vy"], prm["dx"], prm["dy"])
    op = B.make_operator(kind=B.LX_OP_DIFFADV2D, nx=nx, ny=ny, dx=prm["dx"], dy=prm["dy"], D=prm["D"], vx=prm["vx"],
                         vy=prm["vy"])
    return op, np.random.default_rng(nx + ny).standard_normal((ny, nx)), h, c, g


@pytest.mark.parametrize("nx,ny", [(64, 64), (113, 50)])
def test_loops_that_end_while_coefficients_are_formed_beside_them(ctx, nx, ny):
    """Back-to-back solves whose loops end after two to five windows, each
    with a launch or more past its end whose extra workgroups meet at barriers:
    every repetition has the bits of one iteration per launch."""
    op, v, h, c, g = _problem(nx, ny, 20.0)
    d = dev(v)
    for rtol in (1e-2, 1e-4, 1e-6, 1e-9, 1e-12):
        say("loop ends", nx, ny, rtol)
        outs = [dev(np.full(v.shape, np.nan)) for _ in range(2)]
        ctx.set_depth(1)
        try:
            r1 = ctx.phi_leja(op, d, outs, [0, 2], h, c, g, rtol=rtol, max_iters=300)
        finally:
            ctx.set_depth(0)
        ref = [host(o) for o in outs]
        for _ in range(8):
            r = ctx.phi_leja(op, d, outs, [0, 2], h, c, g, rtol=rtol, max_iters=300)
            assert r.status == B.LX_OK and r.stats["depth"] == 8
            if r.iters == r1.iters:
                assert all(np.array_equal(host(o), q) for o, q in zip(outs, ref))
            else:
                assert max(rel(host(o), q) for o, q in zip(outs, ref)) <= 10 * rtol
