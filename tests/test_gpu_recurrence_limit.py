"""Which rasters the FP64 and FP32 modes take by the recurrence (needs an
MI355X): 0.12 N + 40 spikes a bin at the most, the FP64 likelihood alone 0.03
N + 220, on both sides of each limit.  The dense contractions' reduction of
the partial gradients shows in the profile, the recurrence has none of its own
for one chunk; without a gradient the path shows in the staging of the
weights, which an evaluation repeats where it takes the other one than the
evaluation before.  All against the oracle (test_gpu_recurrence's bounds).
"""
import numpy as np
import pytest

from oracle import glm_oracle as O
from parity_check import check
from test_gpu_recurrence import TOL, params, tol32
from test_gpu_spikes import DT

pytestmark = pytest.mark.gpu


def raster(N, B, rate):
    """rate neurons in every bin, and those that then have no spike in the first."""
    rng = np.random.default_rng(rate)
    neu = np.concatenate([rng.choice(N, rate, replace=False) for _ in range(B)])
    missing = np.setdiff1d(np.arange(N), neu)
    return (np.append(np.repeat(np.arange(B), rate), np.zeros(missing.size)).astype(np.int64),
            np.append(neu, missing).astype(np.int32))


@pytest.mark.parametrize("N,rate,dense,alone64", [
    (300, 70, False, False), (300, 80, True, True), (2200, 280, False, False), (2200, 296, False, True), (2200, 310, True, True)])
def test_limits(N, rate, dense, alone64):
    import paper_1502_04993_amd as G
    B = 128
    bins, neu = raster(N, B, rate)
    assert abs(bins.size - rate * B) <= 0.01 * rate * B and np.unique(neu).size == N
    J, mu = params(N, N)
    J = (0.1 * J).astype(np.float32).astype(np.float64)
    ref = O.loglik(bins, neu, N, B, DT, 0.01, J, mu)
    for precision, alone, tol in (("fp64", alone64, TOL["fp64"]), ("fp32", dense, tol32(N, B))):
        c = G.Context(N, B, DT, precision=precision)
        c.set_spikes(bins, neu)
        c.set_kernel(0.01)
        c.set_params(J, mu)
        c.prof(True)
        got = c.eval(grad=True)
        assert ("reduce_G" in c.prof_get()) == dense, precision
        for k in range(2):
            c.prof_reset()
            ll = c.eval(grad=False)["ll"]
            assert ("prepare" in c.prof_get()) == (k == 0 and alone != dense), (precision, k)
            assert abs(ll - got["ll"]) <= 1e-12 * abs(got["ll"])
        again = c.eval(grad=True)
        assert again["ll"] == got["ll"] and np.array_equal(again["gJ"], got["gJ"])
        c.close()
        check(f"limit {precision} N={N} rate={rate}", got, ref, tol)
