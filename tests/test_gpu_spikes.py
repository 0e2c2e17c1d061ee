"""The spike term dSigma_ij = sum_t s_i[t] x_j[t] (Eq. (12)) at the edges of
the window-major spike lists (needs an MI355X).

At mu = -700 the intensities vanish (e^-700), so dL/dJ is dSigma itself in
every mode.  Sizes: windows of 1024 bins that are one bin short, exact and one
bin over, one to 1100 neurons (rows in groups of 1, 2, ... 16, and a second
block past 1024), several spikes per bin, and a raster so dense that a
window's entries pass through LDS in pieces.  Each sum is of at most 6000
positive FP64 terms of a few ulp each, so 1e-12 relative holds with a wide margin.
"""
import numpy as np
import pytest

from oracle import glm_oracle as O
import synth

pytestmark = pytest.mark.gpu

DT = 0.001


def raster(N, B, density, seed, most=1):
    rng = np.random.default_rng(seed)
    S = (rng.random((B, N)) < density).astype(np.int64)
    if most > 1:
        S *= rng.integers(1, most + 1, (B, N))
    S[rng.integers(0, B, N), np.arange(N)] = 1  # every neuron spikes
    S[B - 1, 0] = 1                             # and the last bin is not empty
    t, i = np.nonzero(S)
    return np.repeat(t, S[t, i]).astype(np.int64), np.repeat(i, S[t, i]).astype(np.int32)


def spike_term(N, B, bins, neu, tau, precision, delays=None):
    import paper_1502_04993_amd as G
    c = G.Context(N, B, DT, precision=precision)
    if delays:
        c.set_delays(*delays)
    c.set_spikes(bins, neu)
    c.set_kernel(tau)
    c.set_params(np.zeros((N, N)), np.full(N, -700.0))
    g = c.eval(grad=True)["gJ"]
    c.close()
    return g


@pytest.mark.parametrize("N,B,density,most", [
    (1, 1, 0.0, 1), (3, 1023, 0.02, 1), (64, 1024, 0.01, 1), (65, 1025, 0.01, 1), (130, 2100, 0.01, 3),
    (257, 4097, 0.007, 1), (600, 3000, 0.007, 1), (1100, 2049, 0.007, 1), (200, 3000, 0.6, 1), (300, 2048, 0.3, 2)])
def test_spike_term_of_windows_and_groups(N, B, density, most):
    bins, neu = raster(N, B, density, N + B, most)
    ref = O.spike_term_matrix(bins, neu, N, B, DT, 0.01)
    for precision in ("bf16", "fp64"):
        got = spike_term(N, B, bins, neu, 0.01, precision)
        assert np.max(np.abs(got - ref)) <= 1e-12 * max(np.max(ref), 1.0), precision


def test_spike_term_with_delays_and_repeated_tau():
    N, B, d = 70, 3000, 1030  # the contractions' raster is shifted by more than a window
    bins, neu = raster(N, B, 0.01, 5)
    keep = bins + d < B
    S = O.spike_matrix(bins, neu, N, B).toarray()
    Sd = O.spike_matrix(bins[keep] + d, neu[keep], N, B).toarray()
    for tau in (0.01, 0.004):
        ref = S.T @ O.trace_lfilter(Sd, O.decay(DT, tau), np.zeros(N))
        got = spike_term(N, B, bins, neu, tau, "bf16", (d, d))
        assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(ref)


@pytest.mark.parametrize("N,T", [(5, 2.0), (130, 3.0)])
def test_spike_term_of_the_event_grid(N, T):
    import paper_1502_04993_amd as G
    rec = synth.balanced(N=N, B=int(T / DT), in_frac=0.3, seed=N)
    times, neu = synth.event_times(rec, seed=1)
    ref = O.continuous_eval([times[neu == j] for j in range(N)], 0.0, T, rec.tau, np.zeros((N, N)), np.full(N, -700.0))
    c = G.Context.from_events(N, times, neu, 0.0, T, precision="bf16")
    c.set_kernel(rec.tau)
    c.set_params(np.zeros((N, N)), np.full(N, -700.0))
    got = c.eval(grad=True)["gJ"]
    c.close()
    assert np.max(np.abs(got - ref["gJ"])) <= 1e-12 * np.max(ref["gJ"])
