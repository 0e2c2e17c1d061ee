"""The set-up without allocation after a change of precision that found no
kernel set, because the last one was refused (needs an MI355X): the recurrence's
spike lists have to be there already.  Against a fresh context (bitwise)."""
import numpy as np
import pytest

from test_gpu_recurrence import params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_noalloc_after_a_refused_kernel(precision):
    import paper_1502_04993_amd as G
    N, T = 4, 60.0
    rng = np.random.default_rng(2)
    times = np.sort(rng.random(200) * T)
    neu = np.concatenate([np.arange(N), rng.integers(0, N, 196)]).astype(np.int32)
    J, mu = params(N, 1)
    out = []
    for refused in (True, False):
        c = G.Context.from_events(N, times, neu, 0.0, T, precision="bf16" if refused else precision, max_gap=1e6)
        c.set_kernel(0.5)
        if refused:
            with pytest.raises(G.GlmrError):
                c.set_kernel(0.005)  # 64 slots span more than 600 tau
            c.set_precision(precision)
        c.set_kernel_noalloc(0.4)
        c.set_params(J, mu)
        out.append(c.eval(grad=True))
        c.close()
    assert out[0]["ll"] == out[1]["ll"] and np.array_equal(out[0]["gJ"], out[1]["gJ"])
