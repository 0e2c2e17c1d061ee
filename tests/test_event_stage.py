"""The interval integrals (Eq. (10), (14)) as the recurrence's event-grid
kernel takes them, on the CPU (ev_host.cpp compiles the same source): the
expansion staged per slot and, past its bound, the evaluation that holds for
every potential.  Against mpmath over the ordinary range, and against the
closed forms over huge, infinite and undefined potentials, where no loop may
depend on the potential's size: the calls run in a process with a time limit.

Bound against mpmath: the series' 26 terms at D = -2 are up to 50 times its
sum, at a few units of 1.1e-16 each, so 2e-14, times the condition of e^u at
the end of the interval that carries the integral.
"""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

from test_event_functions import _ref

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("ev") / "ev_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wno-unknown-pragmas", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "ev_host.cpp")], check=True)
    return so


def call(so, name, D, delta):
    D, delta = (np.ascontiguousarray(v, np.float64) for v in (D, delta))
    F, H, staged = np.empty_like(D), np.empty_like(D), np.zeros(D.size, np.int32)
    p = lambda v: v.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    more = (p(staged),) if name == "ev_slot" else ()
    getattr(ctypes.CDLL(so), name)(D.size, p(D), p(delta), p(F), p(H), *more)
    return F, H, staged


@pytest.mark.parametrize("name", ["ev_any", "ev_slot"])
def test_against_mpmath(lib, name):
    rng = np.random.default_rng(1)
    D = np.concatenate([rng.uniform(-3, 3, 200), rng.uniform(-40, 60, 300), rng.uniform(-700, 700, 300),
                        -10.0 ** rng.uniform(0, 12, 100), [2.0, -2.0, 2.0 + 1e-9, -2.0 - 1e-9, 1e-12, 0.0, 709.0, -745.0]])
    delta = 10 ** rng.uniform(-6, 2.6, D.size)
    delta[400:600] = rng.uniform(0, 1.2, 200)
    F, H, staged = call(lib, name, D, delta)
    if name == "ev_slot":
        assert 100 < staged.sum() < D.size - 100
    for k in range(D.size):
        # e^u is taken at the end with the larger u, whose relative rounding is a few units more for long intervals
        u = D[k] if D[k] > 0 else D[k] * np.exp(-delta[k]) * (1.0 + delta[k])
        bound = 2e-14 * max(1.0, abs(u))
        for got, ref in zip((F[k], H[k]), _ref(D[k], delta[k])):
            if ref > 1e-290:  # else at the edge of underflow
                assert abs(float((got - ref) / ref)) <= bound, (D[k], delta[k], got, ref)


EXTREMES = r"""
import sys, numpy as np
sys.path[:0] = [%r, %r]
import test_event_stage as T
big = np.concatenate([10.0 ** np.arange(-300, 301, 10), [2.0, 7.0, 30.0, 700.0, 709.9, 711.0, 745.0, 760.0, 1e3, 1e5, 1e6, 1e15, 1e16,
                      1e18, 1.7e308, np.inf]])
D, delta = (v.ravel() for v in np.meshgrid(np.concatenate([big, -big, [0.0, np.nan]]),
                                           [0.0, 1e-18, 1e-9, 1e-3, 0.1, 0.25, 1.0, 3.0, 40.0, 600.0, 800.0]))
np.savez(%r, D=D, delta=delta, any=T.call(%r, "ev_any", D, delta)[:2], slot=T.call(%r, "ev_slot", D, delta)[:2])
"""


def test_huge_infinite_and_undefined_potentials(lib, tmp_path):
    import paper_1502_04993_amd as G
    out = str(tmp_path / "out.npz")
    subprocess.run([sys.executable, "-c", EXTREMES % (HERE, os.path.dirname(HERE), out, lib, lib)], check=True, timeout=100)
    r = np.load(out)
    D, delta = r["D"], r["delta"]
    for F, H in (r["any"], r["slot"]):
        for k in range(D.size):
            at = (D[k], delta[k], F[k], H[k])
            if delta[k] == 0.0:
                assert np.isnan(D[k]) or np.isinf(D[k]) or F[k] == H[k] == 0.0, at
            elif np.isnan(D[k]):
                assert np.isnan(F[k]) and np.isnan(H[k]), at
            elif D[k] > 720.0 + 20.0 * delta[k]:  # e^D over the interval's first 20th overflows
                assert F[k] == H[k] == np.inf, at
            elif D[k] == -np.inf:
                assert F[k] == H[k] == 0.0, at
            else:
                for got, ref in zip((F[k], H[k]), G.glmr_ei_interval(D[k], delta[k])):
                    if np.isfinite(ref):  # 1e-16 of |u| <= 750 in the exponent, and of delta <= 800 in u
                        assert abs(got - ref) <= 1e-11 * abs(ref) + 1e-290, (at, ref)


def test_exponential(lib):
    x = np.concatenate([np.linspace(-745.0, 709.7, 20001), np.random.default_rng(2).normal(0, 3, 20000)])
    y = np.empty_like(x)
    ctypes.CDLL(lib).ev_exp(x.size, x.ctypes.data_as(ctypes.c_void_p), y.ctypes.data_as(ctypes.c_void_p))
    assert np.max(np.abs(y - np.exp(x)) / np.spacing(np.exp(x))) <= 2.0  # about 1 ulp each


def test_exponential_of_infinities(lib):
    x = np.array([-np.inf, -1.7e308, -1e5, -746.0, 0.0, 710.0, 1e5, 1.7e308, np.inf, np.nan, -np.nan])
    y = np.empty_like(x)
    ctypes.CDLL(lib).ev_exp(x.size, x.ctypes.data_as(ctypes.c_void_p), y.ctypes.data_as(ctypes.c_void_p))
    with np.errstate(over="ignore"):
        assert np.array_equal(y, np.exp(x), equal_nan=True)
