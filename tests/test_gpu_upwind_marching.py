"""Register-marching windows of the third-order upwind operator (radius 2):
at the edges of strips (112 output columns at depth 4, 104 at depth 6), on the
smallest grids (sides of twice the depth), one and several bands, with stops
and iteration caps at every place of a window; against the oracle (1e-10, as
the other window tests) and bit for bit against one iteration per launch when
the counts agree.
"""
import numpy as np
import pytest

from oracle.phi_action import leja_phi
from paper_2310_08344_amd import binding as B
from tests.gpu_helpers import oracle_parity, rel, say
from tests.test_gpu_register_tiles import _case, _solve

pytestmark = pytest.mark.gpu

PARITY = 1e-10


@pytest.fixture(scope="module")
def ctx(lx):
    c = lx.context(n_max=2048 * 1100, k_max=1)
    yield c
    c.close()


def _march(ctx, case, l, depth, bands=0, nb=0, **kw):
    ctx.set_window_kernel(2, bands, nb)
    try:
        return _solve(ctx, case, [l], depth, **kw)
    finally:
        ctx.set_window_kernel(0)


@pytest.mark.parametrize("depth", [4, 6])
@pytest.mark.parametrize("nx,ny,bands,nb", [(12, 12, 0, 0), (14, 13, 0, 0), (104, 17, 0, 0), (106, 64, 3, 1),
                                            (112, 100, 0, 0), (114, 101, 7, 2), (208, 40, 40, 0), (226, 250, 0, 0),
                                            (336, 64, 2, 3), (1000, 300, 0, 0)])
def test_upwind_marching_matches_oracle_and_single_iterations(ctx, depth, nx, ny, bands, nb):
    case = _case("up3", nx, ny, nx + ny)
    op, A, u, v, h, c, g = case
    say("upwind marching", depth, nx, ny, bands, nb)
    r, o = _march(ctx, case, 1, depth, bands, nb, rtol=1e-9, max_iters=300)
    assert r.status == B.LX_OK and r.stats["depth"] == depth and r.stats["marching"] == 1
    r1, o1 = _solve(ctx, case, [1], 1, rtol=1e-9, max_iters=300)
    assert r1.stats["depth"] == 1
    if r.iters == r1.iters:
        assert np.array_equal(o[0], o1[0])
    oracle_parity(o, r.iters, lambda f: leja_phi(A, v, [(1, 1.0, 1.0)], h, c, g, 1e-9, 0.0, 300, f), PARITY)


@pytest.mark.parametrize("max_iters", list(range(1, 14)))
@pytest.mark.parametrize("depth", [4, 6])
def test_upwind_marching_at_max_iters(ctx, depth, max_iters):
    case = _case("up3", 62, 45, 5)
    op, A, u, v, h, c, g = case
    say("upwind marching notconv", depth, max_iters)
    r, o = _march(ctx, case, 2, depth, rtol=1e-15, max_iters=max_iters, raise_on_error=False)
    assert r.status == B.LX_ENOTCONV and r.iters == [max_iters] and r.stats["marching"] == 1
    ref = leja_phi(A, v, [(2, 1.0, 1.0)], h, c, g, 1e-15, 0.0, max_iters)
    assert rel(o[0], ref.p[0]) <= PARITY
