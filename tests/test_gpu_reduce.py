"""The reduction of kernel G's FP32 partials (needs an MI355X): one thread an
entry up to eight splits, four beyond, and added to an earlier chunk's sum.

The gradient's integral term in BF16 against the oracle's.  Trace, weights and
W are rounded to 2^-9 each, so it is within 2 % of its largest entry; a split
or a quarter of them left out would be 8 % and more.
"""
import numpy as np
import pytest
import torch

from oracle import glm_oracle as O
from test_gpu_recurrence import params
from test_gpu_spikes import DT, raster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [40, 300])
@pytest.mark.parametrize("B,kw", [(64, {}), (256, {}), (500, {}), (513, {}), (800, {}), (5000, {}), (4200, dict(chunk_bins=4096)),
                                  (9000, dict(chunk_bins=4096))])
def test_partials_of_few_and_many_splits(N, B, kw):
    import paper_1502_04993_amd as G
    bins, neu = raster(N, B, 0.03, N + B)
    J, mu = params(N, N)
    J = torch.tensor(J).to(torch.bfloat16).to(torch.float64).numpy()
    dsig = O.spike_term_matrix(bins, neu, N, B, DT, 0.01)
    ref = dsig - O.loglik(bins, neu, N, B, DT, 0.01, J, mu)["gJ"]
    c = G.Context(N, B, DT, precision="bf16", **kw)
    c.set_spikes(bins, neu)
    c.set_kernel(0.01)
    c.set_params(J, mu)
    got = dsig - c.eval(grad=True)["gJ"]
    batch = G.Batch([c])
    batch.eval()
    assert np.array_equal(dsig - batch.grad(0)[0], got)
    batch.close()
    c.close()
    assert np.max(np.abs(got - ref)) <= 0.02 * np.max(np.abs(ref))
