"""Newton coefficients as the device forms them, span of columns after span,
against the host's correctly rounded ones (lx_newton_coeffs): the launcher is
called as the loops call it, on tables that end inside and beyond a wavefront
and that start over with more rows."""
import ctypes

import numpy as np
import pytest
import torch

from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

K_MAX = 4


class Series(ctypes.Structure):
    _fields_ = [(n, ctypes.c_double) for n in ("alpha", "sigma", "h", "c", "gamma")] + [("l", ctypes.c_int)]


class Args(ctypes.Structure):
    _fields_ = [("s", Series * K_MAX), ("K", ctypes.c_int), ("rtol", ctypes.c_double), ("atol", ctypes.c_double),
                ("fp32_switch", ctypes.c_double), ("max_iters", ctypes.c_int), ("out32", ctypes.c_int)]


LAUNCH = "_ZN2lx13launch_coeffsERKNS_8CoefArgsEPKdPdS5_iiiiPNS_7LoopCtlEP12ihipStream_t"


def _device_coeffs(lx, series, ld, spans):
    """spans: [(rows, j0, j1), ...]; returns [K][ld] coefficients."""
    f = getattr(ctypes.CDLL(lx.path), LAUNCH)
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.POINTER(Args)] + [ctypes.c_void_p] * 3 + [ctypes.c_int] * 4 + [ctypes.c_void_p] * 2
    a = Args(K=len(series))
    for k, q in enumerate(series):
        a.s[k] = Series(*q)
    xi = torch.as_tensor(np.asarray(lx.leja_points(ld))).to("cuda:0")
    state = torch.full((len(series), 2, ld), float("nan"), dtype=torch.float64, device="cuda:0")
    coef = torch.full((len(series), ld), float("nan"), dtype=torch.float64, device="cuda:0")
    for rows, j0, j1 in spans:
        assert f(ctypes.byref(a), xi.data_ptr(), state.data_ptr(), coef.data_ptr(), ld, rows, j0, j1, None,
                 torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return coef.cpu().numpy()


def _check(lx, series, d, upto):
    """Correctly rounded down to the floor of a double-double table, as the
    host's own test (1e-30 of the largest; 2^-52 for one rounding each)."""
    for k, (alpha, sigma, h, c, gamma, l) in enumerate(series):
        ref = lx.newton_coeffs(l, h, c, gamma, upto, alpha=alpha, sigma=sigma)
        err = np.abs(d[k, :upto] - ref)
        assert np.all(err <= 2.3e-16 * np.abs(ref) + 1e-30 * np.max(np.abs(ref))), (k, int(np.argmax(err)))


def _series(*spec):
    h = 2.0e-3
    return [(alpha, sigma, h, -2.0 * hg / h, hg / h, l) for l, hg, alpha, sigma in spec]


@pytest.mark.parametrize("ld,spans", [
    (60, [(60, 0, 9), (60, 9, 17), (60, 17, 60)]),
    (64, [(64, 0, 64)]),
    (65, [(65, 0, 1), (65, 1, 2), (65, 2, 64), (65, 64, 65)]),
    (200, [(128, 0, 9), (128, 9, 25), (128, 25, 128), (200, 0, 129), (200, 129, 200)]),
    (320, [(128, 0, 17), (256, 0, 160), (320, 0, 300), (320, 300, 320)]),
    (700, [(700, 0, 513), (700, 513, 700)]),
    (1001, [(1001, 0, 600), (1001, 600, 1001)])])
def test_device_coefficients_match_the_host_ones(lx, ld, spans):
    series = _series((0, 5.1, 1.0, 1.0), (1, 25.6, 1.0, 1.0), (3, 25.6, 1.0, 32.0 / 9.0), (2, 150.0, 0.75, 0.75))
    say("device coefficients", ld, spans)
    d = _device_coeffs(lx, series, ld, spans)
    _check(lx, series, d, spans[-1][2])
    assert np.all(np.isnan(d[:, spans[-1][2]:]))


@pytest.mark.parametrize("l", range(9))
def test_device_coefficients_of_every_order(lx, l):
    series = _series((l, 0.3, 1.0, 1.0), (l, 40.0, 0.5, 2.0), (l, 200.0, 1.0, 1.0))
    say("device coefficients of order", l)
    _check(lx, series, _device_coeffs(lx, series, 160, [(128, 0, 9), (128, 9, 100), (160, 0, 160)]), 160)
