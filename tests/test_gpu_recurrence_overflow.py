"""Potentials that overflow to -infinity on the regular grid (needs an MI355X):
their intensity is zero, the likelihood and its gradient stay finite.  Against
the dense contractions (GLMR_RECUR=0): FP64 sums that differ by their rounding
order, 1e-11 of the largest value as in the other comparisons of the two paths.
"""
import numpy as np
import pytest

from test_gpu_recurrence import params
from test_gpu_spikes import DT, raster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B", [(5, 300), (130, 70_000)])
def test_overflow_to_minus_infinity_is_a_zero_intensity(N, B, monkeypatch):
    import paper_1502_04993_amd as G
    bins, neu = raster(N, B, 0.01, N)
    late = B - 20
    keep = (bins < late - 1) | (neu != 0)          # neuron 0 is silent at the end,
    keep &= (neu != 1) | (bins >= late)
    bins = np.append(bins[keep], [late, late])     # where neuron 1 spikes twice in a bin for the first time
    neu = np.append(neu[keep], [1, 1]).astype(np.int32)
    J, mu = params(N, N)
    J[0, 1] = -1.7e308
    out = []
    for mode in "01":
        monkeypatch.setenv("GLMR_RECUR", mode)
        c = G.Context(N, B, DT, precision="fp64")
        c.set_spikes(bins, neu)
        c.set_kernel(0.01)
        c.set_params(J, mu)
        out.append(c.eval(grad=True))
        c.close()
    for k in ("ll", "ll_rows", "gJ", "gmu"):
        a, b = np.asarray(out[1][k]), np.asarray(out[0][k])
        assert np.all(np.isfinite(b)) and np.max(np.abs(a - b)) <= 1e-11 * max(1.0, np.max(np.abs(b))), k
