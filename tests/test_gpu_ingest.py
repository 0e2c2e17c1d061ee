"""Spike ingest: planes, counts and digest from (bin, neuron) pairs in any
order (needs an MI355X).

One context takes rasters with and without several spikes in a cell in turn,
and one that is refused, at sizes around a subtile (64 bins), a run of
subtiles (64) and a block of columns (256 neurons).  At mu = -700 the
intensities vanish, so dL/dmu is q itself and dL/dJ the spike term of the
planes (a sum of at most 9000 positive FP64 terms: 1e-12 relative holds with a
wide margin).
"""
import numpy as np
import pytest

from oracle import glm_oracle as O
from test_gpu_spikes import DT, raster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B", [(1, 1), (3, 64), (130, 65), (257, 4097), (40, 9000)])
def test_planes_counts_and_digest(N, B):
    import paper_1502_04993_amd as G
    c = G.Context(N, B, DT, precision="fp64")
    c.set_kernel(0.01)
    c.set_params(np.zeros((N, N)), np.full(N, -700.0))
    for seed, most in ((1, 1), (2, 3), (3, 2), (4, 1), (5, 1)):
        bins, neu = raster(N, B, 0.02, seed, most)
        if seed == 4:
            with pytest.raises(G.GlmrError):
                c.set_spikes(np.append(bins, B), np.append(neu, 0).astype(np.int32))
        perm = np.random.default_rng(seed).permutation(bins.size)
        ref = O.spike_term_matrix(bins, neu, N, B, DT, 0.01)
        c.set_spikes(bins, neu)
        state = c.get_state()
        got = c.eval(grad=True)
        c.set_spikes(bins[perm], neu[perm])
        again = c.eval(grad=True)
        assert c.get_state() == state
        for e in (got, again):
            assert np.array_equal(e["gmu"], np.bincount(neu, minlength=N).astype(float))
            assert np.max(np.abs(e["gJ"] - ref)) <= 1e-12 * max(np.max(ref), 1.0)
        assert c.query()["planes"] == np.unique(bins * N + neu, return_counts=True)[1].max()
    c.close()
