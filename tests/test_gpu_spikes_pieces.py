"""Spike lists that pass through LDS in many pieces (needs an MI355X): eight
neurons of one group with twelve spikes in every bin of a window (24576 groups
of four entries among one group's neurons, past the 16944 from which the end
of a list that is done lies below address zero), the others with one spike.

The spike term is compared as in test_gpu_spikes, kernel G of the recurrence
with the oracle's gradient: sums of 1e5 positive FP64 terms of a few ulp each.
"""
import numpy as np
import pytest

from oracle import glm_oracle as O
from test_gpu_spikes import DT, spike_term

pytestmark = pytest.mark.gpu


def heavy(N, B, first):
    rng = np.random.default_rng(N)
    bins = [np.repeat(np.arange(B), 12 * 8), rng.integers(0, B, N), [B - 1]]
    neu = [np.tile(np.repeat(np.arange(first, first + 8), 12), B), np.arange(N), [0]]
    return np.concatenate(bins).astype(np.int64), np.concatenate(neu).astype(np.int32)


@pytest.mark.parametrize("N,first", [(513, 0), (600, 256)])
def test_finished_lists_take_nothing_more(N, first, monkeypatch):
    import paper_1502_04993_amd as G
    B = 1024
    bins, neu = heavy(N, B, first)
    ref = O.spike_term_matrix(bins, neu, N, B, DT, 0.01)
    for precision in ("bf16", "fp64"):
        got = spike_term(N, B, bins, neu, 0.01, precision)
        assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(ref), precision
    monkeypatch.setenv("GLMR_RECUR", "1")
    rng = np.random.default_rng(1)
    J, mu = rng.normal(0, 1e-3, (N, N)), rng.normal(1.5, 0.3, N)
    c = G.Context(N, B, DT, precision="fp64")
    c.set_spikes(bins, neu)
    c.set_kernel(0.01)
    c.set_params(J, mu)
    r = c.eval(grad=True)
    c.close()
    want = O.loglik(bins, neu, N, B, DT, 0.01, J, mu)
    assert abs(r["ll"] - want["ll"]) <= 1e-11 * abs(want["ll"])
    assert np.max(np.abs(r["gJ"] - want["gJ"])) <= 1e-10 * np.max(np.abs(want["gJ"]))
