"""FP32 sweeps on register tiles go over to FP32 after the same iteration as
one iteration per launch, whichever place of a window it falls on, and form
every level in the same precision: the same bits when the counts agree."""
import numpy as np
import pytest

from oracle.operators import diffadv_apply
from oracle.phi_action import leja_phi
from paper_2310_08344_amd import binding as B
from paper_2310_08344_amd import workloads as W
from tests.gpu_helpers import closed_form_shift, dev, diffadv_setup, host, rel, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lx):
    c = lx.context(n_max=2048 * 1100, k_max=3)
    yield c
    c.close()


def _case(kind, nx, ny, cfl=20.0):
    rng = np.random.default_rng(5 * nx + ny)
    v = rng.standard_normal((ny, nx))
    if kind == "da":
        prm, h = diffadv_setup(nx, ny, vx=0.7 * nx, vy=-0.4 * ny, cfl=cfl)
        c, g = closed_form_shift(prm["D"], prm["vx"], prm["vy"], prm["dx"], prm["dy"])
        op = B.make_operator(kind=B.LX_OP_DIFFADV2D, nx=nx, ny=ny, dx=prm["dx"], dy=prm["dy"], D=prm["D"],
                             vx=prm["vx"], vy=prm["vy"], prec=B.LX_FP32_SWEEP)
        return op, v, None, h, c, g
    dx, dy = 1.0 / nx, 1.0 / ny
    u = W.fourier_modes(max(nx, ny), seed=nx)[:ny, :nx] + 0.2
    umax = float(np.max(np.abs(u)))
    nu = umax * max(dx, dy) / 2.0
    h = 8.0 * W.burgers_cfl_step(nu, umax, dx, dy)
    op = B.make_operator(kind=B.LX_OP_BURGERS2D, nx=nx, ny=ny, dx=dx, dy=dy, nu=nu, prec=B.LX_FP32_SWEEP)
    rho = 2.0 / W.burgers_cfl_step(nu, umax, dx, dy)
    return op, v, u, h, -1.05 * rho / 2.0, 1.05 * rho / 4.0


def _solve(ctx, case, ls, depth, **kw):
    op, v, u, h, c, g = case
    outs = [dev(np.full(v.shape, np.nan)) for _ in ls]
    ctx.set_depth(depth)
    try:
        r = ctx.phi_leja(op, dev(v), outs, ls, h, c, g, u=dev(u) if u is not None else None, **kw)
    finally:
        ctx.set_depth(0)
    return r, [host(o) for o in outs]


SWITCHES = [0.0, 3.0, 30.0, 300.0, 1e3, 1e4, 1e5, 1e6, 1e7, 1e9, 1e300]


@pytest.mark.parametrize("kind,nx,ny,ls", [("da", 9, 10, [1]), ("da", 83, 85, [0]), ("da", 83, 85, [0, 2]),
                                           ("da", 96, 64, [1, 2, 3]), ("da", 640, 700, [0, 1, 3]),
                                           ("da", 2048, 1100, [0, 2]), ("bu", 11, 9, [1]), ("bu", 120, 113, [0]),
                                           ("bu", 96, 64, [1, 3]), ("bu", 701, 640, [0, 2])])
def test_fp32_sweeps_start_after_the_iteration_one_per_launch_finds(ctx, kind, nx, ny, ls):
    case = _case(kind, nx, ny)
    counts = set()
    for switch in SWITCHES:
        say("fp32 switch", kind, nx, ny, ls, switch)
        kw = dict(rtol=1e-7, max_iters=300, fp32_switch=switch)
        r, o = _solve(ctx, case, ls, 0, **kw)
        r1, o1 = _solve(ctx, case, ls, 1, **kw)
        assert r.status == r1.status == B.LX_OK
        assert r.stats["depth"] == 8 and r.stats["marching"] == 0 and r1.stats["depth"] == 1
        say("iterations", r.iters, r1.iters, "fp32", r.stats["n_fp32"], r1.stats["n_fp32"])
        counts.add((max(r1.iters) - r1.stats["n_fp32"]) % 8)   # the place of the switch in a window
        if r.iters == r1.iters:
            assert all(np.array_equal(a, b) for a, b in zip(o, o1)), [rel(a, b) for a, b in zip(o, o1)]
        else:
            assert max(rel(a, b) for a, b in zip(o, o1)) <= 1e-6
    assert len(counts) >= 3


@pytest.mark.parametrize("max_iters", [3, 8, 9, 13, 16, 20])
@pytest.mark.parametrize("switch", [1e300, 1e8])
def test_fp32_switch_before_the_iteration_limit(ctx, switch, max_iters):
    """The limit before, at and after the switch, inside a window and at its end."""
    case = _case("da", 61, 45)
    say("fp32 switch notconv", switch, max_iters)
    kw = dict(rtol=1e-12, max_iters=max_iters, fp32_switch=switch, raise_on_error=False)
    r, o = _solve(ctx, case, [0, 1], 0, **kw)
    r1, o1 = _solve(ctx, case, [0, 1], 1, **kw)
    assert r.status == r1.status == B.LX_ENOTCONV and r.iters == r1.iters == [max_iters] * 2
    assert all(np.array_equal(a, b) for a, b in zip(o, o1))


@pytest.mark.parametrize("nx,tiles", [(256, False), (255, True)])
def test_tuned_fp32_sweeps_have_one_switch_rule_per_shape(lx, nx, tiles):
    """Even grids march (or sweep one by one) as tuned; odd ones, which cannot,
    run on register tiles."""
    case = _case("da", nx, 128)
    say("fp32 tuned", nx)
    with lx.context(n_max=nx * 128, k_max=1) as c:
        rows = c.tune(case[0], K=1, sweeps=8)
        assert any(q[0] == 108 and q[1:3] == (64, 8) for q in rows) == tiles
        r, o = _solve(c, case, [1], 0, rtol=1e-8, max_iters=300)
        assert r.status == B.LX_OK
    op, v, _, h, cc, g = case
    A = lambda y: diffadv_apply(y, op.D, op.vx, op.vy, op.dx, op.dy)
    ref = leja_phi(A, v, [(1, 1.0, 1.0)], h, cc, g, 1e-8, 0.0, 300)
    assert rel(o[0], ref.p[0]) <= 1e-8
