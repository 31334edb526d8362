"""Windows need a second buffer per output.  Where it cannot be allocated, the
automatic choice and the tuner do without (odd grids never needed one before
they had windows)."""
import numpy as np
import pytest
import torch

from paper_2310_08344_amd import binding as B
from tests.gpu_helpers import closed_form_shift, dev, diffadv_setup, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def full(lx):
    """A context whose own vectors (20 bytes per point of n_max) leave no room
    for one more of n_max doubles."""
    torch.cuda.empty_cache()
    c = lx.context(n_max=int(0.8 * torch.cuda.mem_get_info()[0] / 20), k_max=1)
    yield c
    c.close()


@pytest.mark.parametrize("nx", [65, 64])
@pytest.mark.parametrize("prec", [B.LX_FP64, B.LX_FP32_SWEEP])
def test_solves_and_tuning_without_memory_for_windows(full, nx, prec):
    ny = 48
    prm, h = diffadv_setup(nx, ny, cfl=10.0)
    c, g = closed_form_shift(prm["D"], prm["vx"], prm["vy"], prm["dx"], prm["dy"])
    op = B.make_operator(kind=B.LX_OP_DIFFADV2D, nx=nx, ny=ny, dx=prm["dx"], dy=prm["dy"], D=prm["D"], vx=prm["vx"],
                         vy=prm["vy"], prec=prec)
    v = dev(np.random.default_rng(1).standard_normal((ny, nx)))
    say("no memory for windows", nx, prec)
    outs = [torch.empty_like(v) for _ in range(3)]

    def solve(o):
        return full.phi_leja(op, v, [o], [1], h, c, g, rtol=1e-9, max_iters=200)

    r = solve(outs[0])
    assert r.status == B.LX_OK and r.stats["depth"] <= 2
    full.set_depth(1)
    try:
        r1 = solve(outs[1])
    finally:
        full.set_depth(0)
    assert r.iters == r1.iters and np.array_equal(host(outs[0]), host(outs[1]))
    if nx % 2:
        # even grids time windows on other kernels, which report LX_ENOMEM
        rows = full.tune(op, K=1, sweeps=4)
        assert rows and all(q[0] == 1 for q in rows)
        assert solve(outs[2]).stats["depth"] == 1 and np.array_equal(host(outs[2]), host(outs[1]))
    else:
        with pytest.raises(B.LxError):
            full.tune(op, K=1, sweeps=4)
        assert solve(outs[2]).status == B.LX_OK     # the failure is not left to later launches
