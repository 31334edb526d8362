"""CPU tests of the plain arithmetic that host and device share (headers under
csrc that a C++ compiler takes as they are): built into a small library here."""
import ctypes
import math
import os
import shutil
import subprocess

import mpmath as mp
import numpy as np
import pytest

from oracle.leja import phi_mp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "dd_math.h"
#include "planner.h"
#include "quotient.h"
extern "C" int started(unsigned word, unsigned base) { return lx::launches_started(word, base); }
extern "C" int exponent(double g) { return lx::power_exponent(g); }
extern "C" void inv_fact(int k, double* o) { const lx::dd r = lx::dd_inv_fact(k); o[0] = r.hi; o[1] = r.lo; }
extern "C" void phi(int fast, int l, double hi, double lo, double* o) {
    const lx::dd r = fast ? lx::dd_phi_fast(l, lx::dd{hi, lo}) : lx::dd_phi(l, lx::dd{hi, lo});
    o[0] = r.hi;
    o[1] = r.lo;
}
extern "C" void div_rcp(double xh, double xl, double yh, double yl, double ulps, double* o) {
    const lx::dd r = lx::dd_div_rcp(lx::dd{xh, xl}, lx::dd{yh, yl}, 1.0 / yh * (1.0 + ulps * 0x1p-53));
    o[0] = r.hi;
    o[1] = r.lo;
}
extern "C" int fp32_taken(double a, int da, double b, int db) { return lx::fp32_marching_taken(a, da, b, db); }
extern "C" int windows_faster(double a, int da, double b, int db) { return lx::windows_faster(a, da, b, db); }
extern "C" double quotient(double x, double d) { return lx::quotient_rcp(x, d, 1.0 / d); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("shim")
    (d / "shim.cpp").write_text(SOURCE)
    subprocess.run([cxx, "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2310_08344_amd", "csrc"), str(d / "shim.cpp"), "-o", str(d / "shim.so")],
                   check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.exponent.argtypes = [ctypes.c_double]
    lib.quotient.argtypes = [ctypes.c_double, ctypes.c_double]
    lib.quotient.restype = ctypes.c_double
    d, p = ctypes.c_double, ctypes.c_void_p
    lib.inv_fact.argtypes = [ctypes.c_int, p]
    lib.phi.argtypes = [ctypes.c_int, ctypes.c_int, d, d, p]
    lib.div_rcp.argtypes = [d, d, d, d, d, p]
    lib.fp32_taken.argtypes = [d, ctypes.c_int, d, ctypes.c_int]
    lib.windows_faster.argtypes = [ctypes.c_double, ctypes.c_int, ctypes.c_double, ctypes.c_int]
    lib.started.argtypes = [ctypes.c_uint, ctypes.c_uint]
    return lib


def test_progress_of_an_earlier_loop_counts_as_none(shim):
    """A loop of 40 launches (base 0), then one with base 42: a late store of
    the first loop must not let the second enqueue 40 launches at once.  The
    counter may wrap."""
    for base in (0, 42, 2**32 - 42, 2**32 - 1):
        nxt = (base + 42) % 2**32
        for launch in range(40):
            assert shim.started((base + launch + 1) % 2**32, base) == launch + 1
            assert shim.started((base + launch + 1) % 2**32, nxt) == 0
        assert shim.started(base, base) == 0
        assert shim.started((nxt + 1) % 2**32, nxt) == 1


@pytest.mark.parametrize("g", [5e-324, 1e-310, 2.3e-308, 1e-120, 1e-17, 0.49, 0.5, 0.75, 1.0, 3.0, 4.0, 1e17, 1e300])
def test_power_exponent_brings_the_bound_below_one(shim, g):
    e = shim.exponent(g)
    assert 0.5 <= g * 2.0 ** (e // 2) * 2.0 ** (e - e // 2) < 1.0


def test_power_exponent_of_degenerate_bounds(shim):
    for g in (0.0, float("inf"), float("nan")):
        assert shim.exponent(g) == 0


def test_quotient_is_the_division(shim):
    rng = np.random.default_rng(3)
    xs = np.concatenate([rng.standard_normal(2000) * 10.0 ** rng.uniform(-130, 130, 2000), [0.0, -0.0, 1.0, -7.0]])
    for d in np.concatenate([10.0 ** rng.uniform(-140, 140, 8), [1.0 / 2048, (1.0 / 333) ** 2, 2.0 / 96]]):
        for x in xs:
            assert shim.quotient(x, d) == x / d


@pytest.mark.parametrize("x", [1e308, -1.7e308, float("inf"), float("-inf")])
def test_quotient_that_overflows_is_an_infinity(shim, x):
    for d in (1e-3, 1.0 / 4096, 1e-140):
        assert shim.quotient(x, d) == math.copysign(math.inf, x)
    assert math.isnan(shim.quotient(float("nan"), 0.25))


@pytest.mark.parametrize("a,da,b,db,faster", [(640.0, 6, 653.0, 4, 0), (600.0, 6, 653.0, 4, 1), (2.7, 8, 3.7, 8, 1),
                                              (39.0, 8, 38.9, 8, 0), (11.4, 8, 1e300, 1, 1), (7.1, 8, 6.9, 2, 0)])
def test_deeper_windows_must_win_back_what_they_form_past_the_end(shim, a, da, b, db, faster):
    """Measured times per iteration (register tiles first)."""
    assert shim.windows_faster(a, da, b, db) == faster


def _pair():
    return (ctypes.c_double * 2)()


def _exact(o):
    return mp.mpf(o[0]) + mp.mpf(o[1])


def test_reciprocal_factorials_are_rounded_to_double_double(shim):
    o = _pair()
    with mp.workdps(60):
        for k in range(69):
            shim.inv_fact(k, o)
            assert o[0] + o[1] == o[0]
            assert abs(_exact(o) * mp.factorial(k) - 1) <= mp.mpf(2) ** -105


def test_division_by_a_quantity_whose_reciprocal_is_at_hand(shim):
    """Two corrections of a quotient that is right to 2^-51 leave an error of the
    rounding of the last sums, a few 2^-106; the reciprocal may be off by ulps."""
    rng = np.random.default_rng(7)
    o = _pair()
    with mp.workdps(60):
        for _ in range(2000):
            x, y = rng.standard_normal(2) * 10.0 ** rng.uniform(-30, 30, 2)
            xl, yl = x * 2.0**-54 * rng.uniform(-1, 1), y * 2.0**-54 * rng.uniform(-1, 1)
            shim.div_rcp(x, xl, y, yl, float(rng.integers(-2, 3)), o)
            q = (mp.mpf(x) + mp.mpf(xl)) / (mp.mpf(y) + mp.mpf(yl))
            assert abs(_exact(o) / q - 1) <= 16 * mp.mpf(2) ** -106


@pytest.mark.parametrize("l", range(9))
def test_device_phi_has_the_accuracy_of_the_host_phi(shim, l):
    """phi_l over the arguments of a planner, the edges of the series among
    them, against 60 digits: at most 1e-29 (a hundred operations of 2^-104), and
    no worse than the host's form by more than that many roundings of its own."""
    rng = np.random.default_rng(l)
    lim = max(1.5, float(l))
    zs = np.concatenate([-(10.0 ** rng.uniform(-12, 2.9, 120)), rng.uniform(-lim, lim, 60), 10.0 ** rng.uniform(-3, 2, 30),
                         [0.0, -1000.0, np.nextafter(-lim, 0), -lim, lim, np.nextafter(lim, 0), -0.34, -0.35, 0.35]])
    o, old = _pair(), _pair()
    with mp.workdps(60):
        for z in zs:
            zl = z * 2.0**-54 * rng.uniform(-1, 1)
            shim.phi(1, l, z, zl, o)
            shim.phi(0, l, z, zl, old)
            ref = phi_mp(l, mp.mpf(z) + mp.mpf(zl))
            err, err_old = abs(_exact(o) / ref - 1), abs(_exact(old) / ref - 1)
            # (phi_0 below exp(-600) has no low part, below exp(-708) it is subnormal, in both forms)
            assert err <= max(mp.mpf("1e-29"), 4 * err_old), (z, err, err_old)


@pytest.mark.parametrize("t4,t6,depth", [(3.0, 3.8, 4), (4.0, 3.99, 6), (4.0, 4.03, 6), (4.0, 4.05, 4), (7.2, 6.4, 6),
                                         (10.9, 12.0, 4)])
def test_tuned_fp32_marching_depth_turns_on_more_than_noise(shim, t4, t6, depth):
    """Windows of six up to 1 % slower than windows of four are taken; of one
    depth the faster."""
    assert (6 if shim.fp32_taken(t6, 6, t4, 4) else 4) == depth
    assert shim.fp32_taken(t4, 4, t4 * 1.001, 4) and not shim.fp32_taken(t4, 4, t4 * 0.999, 4)
