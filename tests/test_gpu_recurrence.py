"""The FP64 and FP32 modes by the recurrence on the spike lists (needs an MI355X).

Against the FP64 oracle and against the dense contractions (GLMR_RECUR=0, the
path of dense rasters and self-delays) at the edges of its segments (16 to
1024 bins), windows (1024 bins), row blocks (64 and 16) and neuron groups, with
several chunks, delays, several spikes per bin, dL/dtau and the likelihood alone.

Bounds: FP64 sums of at most 1e5 terms of a few ulp each, L and L_i 1e-12 and
1e-11, gradients 1e-10 (as the other FP64 tests); FP32 as test_gpu_parity's.
Two FP64 paths differ by their rounding order only: 1e-11 of the largest value.
"""
import numpy as np
import pytest

from oracle import glm_oracle as O
import synth
from parity_check import check
from test_gpu_spikes import DT, raster

pytestmark = pytest.mark.gpu

TOL = {"fp64": dict(ll=1e-12, row=1e-11, grad=1e-10, gmax=1e-10)}


def tol32(N, B):
    ll = 1e-10 * max(1.0, (2e6 / (B * N)) ** 0.5)
    return dict(ll=ll, row=4 * N ** 0.5 * ll, grad=1e-6, gmax=1e-6)


def params(N, seed):
    rng = np.random.default_rng(seed)
    J = rng.normal(0, 0.6 / max(1.0, N ** 0.5), (N, N))
    np.fill_diagonal(J, -2.0)
    return J, rng.normal(1.5, 0.3, N)


def evaluate(N, B, bins, neu, J, mu, precision, tau=0.01, delays=None, want_tau=False, **kw):
    import paper_1502_04993_amd as G
    c = G.Context(N, B, DT, precision=precision, **kw)
    if delays:
        c.set_delays(*delays)
    c.set_spikes(bins, neu)
    c.set_kernel(tau)
    c.set_params(J, mu)
    out = c.eval(grad=True, want_tau=want_tau)
    alone = c.eval(grad=False)
    assert alone["ll"] == pytest.approx(out["ll"], rel=1e-13)
    c.close()
    return out


SIZES = [(1, 1, 0.0, 1), (2, 17, 0.1, 1), (17, 63, 0.05, 1), (64, 65, 0.02, 1), (65, 1024, 0.01, 3), (129, 1025, 0.01, 1),
         (300, 5000, 0.007, 1), (1100, 2100, 0.007, 1)]


@pytest.mark.parametrize("N,B,density,most", SIZES)
def test_against_the_oracle(N, B, density, most):
    bins, neu = raster(N, B, density, 7 * N + B, most)
    J, mu = params(N, N)
    ref = O.loglik(bins, neu, N, B, DT, 0.01, J, mu)
    check(f"rec fp64 {N} {B}", evaluate(N, B, bins, neu, J, mu, "fp64"), ref, TOL["fp64"])
    J32 = J.astype(np.float32).astype(np.float64)
    ref = O.loglik(bins, neu, N, B, DT, 0.01, J32, mu)
    check(f"rec fp32 {N} {B}", evaluate(N, B, bins, neu, J32, mu, "fp32"), ref, tol32(N, B))


@pytest.mark.parametrize("N,B,density,kw", [
    (50, 40_000, 0.007, {}), (70, 20_000, 0.01, dict(chunk_bins=4096)), (200, 70_100, 0.007, dict(chunk_bins=36864)),
    (500, 100_000, 0.007, {}), (130, 9000, 0.5, {}), (40, 6000, 0.02, dict(delays=(70, 70))),
    (90, 30_000, 0.01, dict(delays=(1500, 1500), chunk_bins=8192)), (33, 3000, 0.02, dict(tau=0.0012)),
    (33, 3000, 0.02, dict(tau=0.3))])
def test_against_the_dense_contractions(N, B, density, kw, monkeypatch):
    bins, neu = raster(N, B, density, N)
    J, mu = params(N, N)
    monkeypatch.setenv("GLMR_RECUR", "0")
    ref = evaluate(N, B, bins, neu, J, mu, "fp64", want_tau=True, **kw)
    monkeypatch.setenv("GLMR_RECUR", "1")
    got = evaluate(N, B, bins, neu, J, mu, "fp64", want_tau=True, **kw)
    for k in ("ll", "ll_rows", "gJ", "gmu", "gtau"):
        a, b = np.asarray(got[k]), np.asarray(ref[k])
        assert np.max(np.abs(a - b)) <= 1e-11 * max(1.0, np.max(np.abs(b))), k


@pytest.mark.parametrize("N,B,kw", [
    (445, 38_000, {}), (1030, 16_500, dict(chunk_bins=8192)), (130, 100_001, {}), (257, 55_000, dict(chunk_bins=20480))])
def test_two_rows_a_lane_against_the_dense_contractions(N, B, kw, monkeypatch):
    """Segments of 64 bins and more: blocks of 128 rows at 7, 17, 3 and 5 blocks of 64 (the last two one row a lane)."""
    test_against_the_dense_contractions(N, B, 0.007, kw, monkeypatch)


@pytest.mark.parametrize("N,T,precision,kw", [
    (1, 1.0, "fp64", {}), (5, 3.0, "fp64", {}), (90, 6.0, "fp64", dict(chunk_bins=4096)), (150, 4.0, "fp32", {}),
    (70, 2.0, "fp64", dict(max_gap=0.0001)), (12, 5.0, "fp64", dict(tau=0.002))])
def test_event_grid_against_the_dense_contractions(N, T, precision, kw, monkeypatch):
    import paper_1502_04993_amd as G
    kw = dict(kw)
    tau = kw.pop("tau", 0.01)
    rng = np.random.default_rng(N)
    n = max(2, int(7 * N * T))
    times = np.sort(rng.random(n) * T)
    neu = np.concatenate([np.arange(N), rng.integers(0, N, n)])[:n].astype(np.int32)
    J, mu = params(N, N)
    if N == 12:
        J *= 6.0  # intervals past the short-interval branch
    out = []
    for mode in ("0", "1"):
        monkeypatch.setenv("GLMR_RECUR", mode)
        c = G.Context.from_events(N, times, neu, 0.0, T, precision=precision, **kw)
        c.set_kernel(tau)
        c.set_params(J, mu)
        out.append(c.eval(grad=True))
        c.close()
    tol = 1e-11 if precision == "fp64" else 1e-7
    for k in ("ll", "ll_rows", "gJ", "gmu"):
        a, b = np.asarray(out[1][k]), np.asarray(out[0][k])
        assert np.max(np.abs(a - b)) <= tol * max(1.0, np.max(np.abs(b))), k


def test_repeatable_and_switched_precision():
    import paper_1502_04993_amd as G
    N, B = 100, 20_000
    rec = synth.balanced(N=N, B=B, in_frac=0.2, seed=9)
    J, mu = params(N, 1)
    c = G.Context(N, B, rec.dt, precision="bf16")
    c.set_params(J, mu)  # before the spikes: staged for the dense path first
    c.set_precision("fp64")
    c.set_spikes(rec.bins, rec.neurons)
    c.set_kernel(rec.tau)
    a, b = c.eval(), c.eval()
    assert a["ll"] == b["ll"] and np.array_equal(a["gJ"], b["gJ"])
    check("switched", a, O.loglik(rec.bins, rec.neurons, N, B, rec.dt, rec.tau, J, mu), TOL["fp64"])
    dense = raster(N, B, 0.3, 3)  # now past the recurrence's density
    c.set_spikes(*dense)
    check("dense", c.eval(), O.loglik(*dense, N, B, rec.dt, rec.tau, J, mu), TOL["fp64"])
    c.close()
