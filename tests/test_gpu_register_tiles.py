"""Windows and power iteration on register tiles, the automatic choice for
small grids and for every odd one: at the edges of tiles (112 output columns;
16 or 48 output rows; windows of six at radius 2: 104 and 8 or 40),
on the smallest grids they take, with stops and iteration caps at every place
of a window, against the oracle (1e-10, as the other window tests) and bit for
bit against one iteration per launch when the counts agree (the same terms in
the same order).
"""
import numpy as np
import pytest

from oracle.operators import burgers_J, diffadv3_apply, diffadv_apply
from oracle.phi_action import leja_phi, power_iteration
from paper_2310_08344_amd import binding as B
from paper_2310_08344_amd import workloads as W
from tests.gpu_helpers import closed_form_shift, dev, diffadv_setup, host, oracle_parity, rel, say

pytestmark = pytest.mark.gpu

PARITY = 1e-10


@pytest.fixture(scope="module")
def ctx(lx):
    c = lx.context(n_max=2402 * 2401, k_max=3)
    yield c
    c.close()


def _case(kind, nx, ny, seed, cfl=20.0):
    rng = np.random.default_rng(seed)
    v = rng.standard_normal((ny, nx))
    if kind == "da":
        prm, h = diffadv_setup(nx, ny, vx=0.7 * nx, vy=-0.4 * ny, cfl=cfl)
        c, g = closed_form_shift(prm["D"], prm["vx"], prm["vy"], prm["dx"], prm["dy"])
        op = B.make_operator(kind=B.LX_OP_DIFFADV2D, nx=nx, ny=ny, dx=prm["dx"], dy=prm["dy"], D=prm["D"],
                             vx=prm["vx"], vy=prm["vy"])
        return op, (lambda y: diffadv_apply(y, prm["D"], prm["vx"], prm["vy"], prm["dx"], prm["dy"])), None, v, h, c, g
    dx, dy = 1.0 / nx, 1.0 / ny
    if kind == "up3":
        vx, vy = -2.0 * nx, 1.5 * ny
        h = cfl * 2.0 / sum(2.0 / d**2 + abs(q) / (2 * d) + abs(1.0 / d**2 - abs(q) / (3 * d)) + 1.0 / d**2
                            + abs(q) / d + abs(q) / (6 * d) for q, d in ((vx, dx), (vy, dy)))
        op = B.make_operator(kind=B.LX_OP_DIFFADV2D_UP3, nx=nx, ny=ny, dx=dx, dy=dy, D=1.0, vx=vx, vy=vy)
        A = lambda y: diffadv3_apply(y, 1.0, vx, vy, dx, dy)
        rho = 2.0 * cfl / h
    else:
        u = W.fourier_modes(max(nx, ny), seed=seed)[:ny, :nx] + 0.2
        umax = float(np.max(np.abs(u)))
        nu = umax * max(dx, dy) / 2.0
        h = 8.0 * W.burgers_cfl_step(nu, umax, dx, dy)
        op = B.make_operator(kind=B.LX_OP_BURGERS2D, nx=nx, ny=ny, dx=dx, dy=dy, nu=nu)
        A = lambda w: burgers_J(u, w, nu, dx, dy)
        rho = 2.0 / W.burgers_cfl_step(nu, umax, dx, dy)
        return op, A, u, v, h, -1.05 * rho / 2.0, 1.05 * rho / 4.0
    return op, A, None, v, h, -1.05 * rho / 2.0, 1.05 * rho / 4.0


def _solve(ctx, case, ls, depth, **kw):
    op, A, u, v, h, c, g = case
    outs = [dev(np.full(v.shape, np.nan)) for _ in ls]
    ctx.set_depth(depth)
    try:
        r = ctx.phi_leja(op, dev(v), outs, ls, h, c, g, u=dev(u) if u is not None else None, **kw)
    finally:
        ctx.set_depth(0)
    return r, [host(o) for o in outs]


DEPTH = {"da": 8, "bu": 8, "up3": 6}
CASES = [("da", nx, ny, ls) for (nx, ny), ls in zip(
    [(9, 9), (10, 12), (64, 64), (111, 17), (112, 16), (113, 33), (224, 49), (225, 48), (127, 130), (333, 250),
     (1000, 600), (1023, 601)],
    [[1], [0, 2], [0], [1, 2, 3], [3], [0, 1], [0, 1, 2], [2], [0, 3], [1, 2], [1, 2, 3], [1, 2, 3]])] + \
    [("bu", nx, ny, ls) for (nx, ny), ls in zip([(9, 10), (112, 16), (113, 35), (96, 64), (130, 131), (700, 620)],
                                                [[1], [1, 3], [2], [0], [0, 1], [1, 2]])] + \
    [("up3", nx, ny, [l]) for (nx, ny), l in zip([(13, 13), (104, 16), (105, 41), (250, 250), (75, 49), (901, 700)],
                                                 [1, 0, 2, 1, 0, 1])]


@pytest.mark.parametrize("kind,nx,ny,ls", CASES)
def test_register_tiles_match_oracle_and_single_iterations(ctx, kind, nx, ny, ls):
    case = _case(kind, nx, ny, nx + ny)
    op, A, u, v, h, c, g = case
    say("register tiles", kind, nx, ny, ls)
    r, o = _solve(ctx, case, ls, 0, rtol=1e-9, max_iters=300)
    assert r.status == B.LX_OK and r.stats["depth"] == DEPTH[kind] and r.stats["marching"] == 0
    r1, o1 = _solve(ctx, case, ls, 1, rtol=1e-9, max_iters=300)
    assert r1.stats["depth"] == 1
    if r.iters == r1.iters:
        assert all(np.array_equal(a, b) for a, b in zip(o, o1))
    oracle_parity(o, r.iters, lambda f: leja_phi(A, v, [(l, 1.0, 1.0) for l in ls], h, c, g, 1e-9, 0.0, 300, f), PARITY)


@pytest.mark.parametrize("max_iters", [1, 2, 4, 7, 8, 9, 16, 17])
@pytest.mark.parametrize("kind", ["da", "bu", "up3"])
def test_register_tiles_at_max_iters(ctx, kind, max_iters):
    case = _case(kind, 61, 45, 5)
    op, A, u, v, h, c, g = case
    ls = [1] if kind == "up3" else [1, 2]
    say("register tiles notconv", kind, max_iters)
    r, o = _solve(ctx, case, ls, 0, rtol=1e-15, max_iters=max_iters, raise_on_error=False)
    assert r.status == B.LX_ENOTCONV and r.iters == [max_iters] * len(ls)
    ref = leja_phi(A, v, [(l, 1.0, 1.0) for l in ls], h, c, g, 1e-15, 0.0, max_iters)
    assert max(rel(a, b) for a, b in zip(o, ref.p)) <= PARITY


def test_register_tiles_more_tiles_than_workgroups(ctx):
    """An odd grid of more tiles than the launch has workgroups, bit for bit
    one iteration per launch; and its power iteration."""
    case = _case("da", 2401, 2399, 3, cfl=4.0)
    say("register tiles 2401 x 2399")
    r, o = _solve(ctx, case, [0, 1], 0, rtol=1e-8, max_iters=100)
    r1, o1 = _solve(ctx, case, [0, 1], 1, rtol=1e-8, max_iters=100)
    assert r.stats["depth"] == 8 and r1.stats["depth"] == 1
    if r.iters == r1.iters:
        assert all(np.array_equal(a, b) for a, b in zip(o, o1))
    else:
        assert max(rel(a, b) for a, b in zip(o, o1)) <= 1e-7
    op, A, u, v = case[:4]
    rho, _, _ = ctx.spectrum(op, x0=dev(v), iters=9)
    rho_o, _ = power_iteration(A, v, 9)
    assert abs(rho - rho_o) <= 1e-12 * rho_o


@pytest.mark.parametrize("kind,nx,ny", [("da", 9, 9), ("da", 112, 17), ("da", 113, 64), ("da", 640, 700), ("bu", 6, 5),
                                        ("bu", 120, 25), ("bu", 242, 56), ("up3", 9, 9), ("up3", 113, 33)])
@pytest.mark.parametrize("iters", [1, 2, 7, 8, 9, 20])
def test_register_tile_power_iteration(ctx, kind, nx, ny, iters):
    op, A, u, v, h, c, g = _case(kind, nx, ny, nx * 3 + ny)
    say("register tile power", kind, nx, ny, iters)
    rho, _, _ = ctx.spectrum(op, u=dev(u) if u is not None else None, x0=dev(v), iters=iters)
    rho_o, _ = power_iteration(A, v, iters)
    assert abs(rho - rho_o) <= 1e-12 * rho_o


@pytest.mark.parametrize("scale", [1e-150, 1e-60, 1e12, 1e60, 1e140])
@pytest.mark.parametrize("nx", [64, 65])
def test_power_iteration_of_badly_scaled_vectors_and_operators(ctx, scale, nx):
    """Start vectors outside the range a launch may take unscaled, and
    operators whose powers would leave the range of a launch's levels: the
    estimate comes from the paths that normalise more often.  (Even grids fall
    back on launches of up to ten sweeps, whose levels of an operator of 1e-56
    underflow: such an operator is refused there.)"""
    op, A, u, v, h, c, g = _case("da", nx, 48, 11)
    say("power scale", scale, nx)
    rho_o, _ = power_iteration(A, v, 20)
    rho, _, _ = ctx.spectrum(op, x0=dev(v * scale), iters=20)
    assert abs(rho - rho_o) <= 1e-12 * rho_o
    s = scale if 1e-70 < scale < 1e70 else 1.0
    if s < 1.0 and nx % 2 == 0:
        return
    op.D, op.vx, op.vy = op.D * s, op.vx * s, op.vy * s
    rho, _, _ = ctx.spectrum(op, x0=dev(v), iters=20)
    assert abs(rho - rho_o * s) <= 1e-12 * rho_o * s


@pytest.mark.parametrize("switch", [1e4, 0.0])
@pytest.mark.parametrize("kind,nx,ny,ls", [("da", 10, 12, [1]), ("da", 113, 33, [0, 2]), ("da", 256, 192, [1, 2, 3]),
                                           ("da", 1001, 640, [0, 1, 3]), ("bu", 11, 9, [1]), ("bu", 112, 50, [0, 3]),
                                           ("bu", 900, 701, [1, 2])])
def test_register_tiles_fp32_levels(ctx, kind, nx, ny, ls, switch):
    """FP32 sweeps on register tiles: the basis and the stencil in FP32 once
    every term is small (0: from the first window), everything else in FP64;
    within the solve's tolerance of the FP64 oracle with the default switch,
    1e-5 with FP32 throughout (the bounds of the other FP32 window kernels)."""
    case = _case(kind, nx, ny, 2 * nx + ny)
    op, A, u, v, h, c, g = case
    op.prec = B.LX_FP32_SWEEP
    say("register tiles fp32", kind, nx, ny, ls, switch)
    r, o = _solve(ctx, case, ls, 0, rtol=1e-8, max_iters=300, fp32_switch=switch)
    assert r.status == B.LX_OK and r.stats["depth"] == 8 and r.stats["marching"] == 0
    assert r.stats["n_fp32"] % 8 == 0 and (switch > 0 or r.stats["n_fp32"] > 0)
    ref = leja_phi(A, v, [(l, 1.0, 1.0) for l in ls], h, c, g, 1e-8, 0.0, 300)
    errs = [rel(a, b) for a, b in zip(o, ref.p)]
    say("fp32 register tile errors", errs, r.iters, ref.iters, r.stats["n_fp32"])
    assert max(errs) <= (1e-8 if switch > 0 else 1e-5)


@pytest.mark.parametrize("kind,ls,cfl", [("da", [0], 20.0), ("da", [0, 1, 3], 60.0), ("da", [1], 120.0),
                                         ("up3", [1], 60.0)])
def test_register_tile_windows_form_the_coefficients_they_need(ctx, kind, ls, cfl):
    """Coefficients formed beside the tiles: bit for bit one iteration per
    launch, whose coefficients come from launches of their own.  (The last
    case needs coefficients below 1e-33, what a double-double table of values
    up to 1 resolves: its loop diverges, in every kernel.)"""
    case = _case(kind, 47, 53, 7, cfl=cfl)
    say("register tile coefficients", kind, ls, cfl)
    if kind == "up3":
        for depth in (0, 1):
            with pytest.raises(B.LxError, match="nonfinite"):
                _solve(ctx, case, ls, depth, rtol=1e-9, max_iters=900)
        return
    r, o = _solve(ctx, case, ls, 0, rtol=1e-9, max_iters=900)
    r1, o1 = _solve(ctx, case, ls, 1, rtol=1e-9, max_iters=900)
    say("iterations", r.iters, r1.iters)
    assert r.status == B.LX_OK and r.stats["depth"] == DEPTH[kind] and r1.stats["depth"] == 1
    if r.iters == r1.iters:
        assert all(np.array_equal(a, b) for a, b in zip(o, o1))
    else:
        assert max(rel(a, b) for a, b in zip(o, o1)) <= 1e-8


@pytest.mark.parametrize("max_iters", [120, 121, 128, 130, 256, 300, 513, 700])
def test_register_tile_loops_past_the_first_coefficient_table(ctx, max_iters):
    """Loops that never converge, so that the tables grow to 256 rows and past
    the 512 that a window launch forms beside its tiles."""
    case = _case("da", 47, 53, 7, cfl=4.0)
    say("register tile long loops", max_iters)
    r, o = _solve(ctx, case, [0, 2], 0, rtol=1e-300, max_iters=max_iters, raise_on_error=False)
    r1, o1 = _solve(ctx, case, [0, 2], 1, rtol=1e-300, max_iters=max_iters, raise_on_error=False)
    assert r.status == r1.status == B.LX_ENOTCONV and r.iters == r1.iters == [max_iters] * 2
    assert all(np.array_equal(a, b) for a, b in zip(o, o1))


@pytest.mark.parametrize("kind,nx,ny", [("bu", 1400, 1300), ("up3", 1301, 1201), ("up3", 1302, 1200),
                                        ("da", 1601, 1300)])
def test_power_iteration_on_more_than_one_round_of_tiles(ctx, kind, nx, ny):
    op, A, u, v, h, c, g = _case(kind, nx, ny, nx + 2 * ny)
    say("register tile power, two workgroups per CU", kind, nx, ny)
    rho, _, _ = ctx.spectrum(op, u=dev(u) if u is not None else None, x0=dev(v), iters=10)
    rho_o, _ = power_iteration(A, v, 10)
    assert abs(rho - rho_o) <= 1e-12 * rho_o


@pytest.mark.parametrize("nx,ny", [(1201, 1100), (2049, 1040)])
def test_upwind_windows_on_more_than_one_round_of_tiles(ctx, nx, ny):
    case = _case("up3", nx, ny, 8, cfl=4.0)
    say("upwind register tiles, two workgroups per CU", nx, ny)
    r, o = _solve(ctx, case, [1], 0, rtol=1e-9, max_iters=100)
    r1, o1 = _solve(ctx, case, [1], 1, rtol=1e-9, max_iters=100)
    assert r.stats["depth"] == 6 and r1.stats["depth"] == 1
    if r.iters == r1.iters:
        assert np.array_equal(o[0], o1[0])
    else:
        assert rel(o[0], o1[0]) <= 1e-8
