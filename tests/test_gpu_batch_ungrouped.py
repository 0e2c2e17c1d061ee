"""Batches whose recordings are evaluated one after the other (needs an MI355X).

FP64 and FP32, the event grid, a self-delay of its own and a trace that is not
resident take no grouped launches.  The batch's log-likelihoods have to be
those of the parameters that the recordings hold, whatever was evaluated
before: the batch goes first, at two sets of parameters and at one whose
likelihood is not finite, and is compared with fresh contexts (the same
kernels: bitwise).
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

KINDS = {"fp64": ("fp64", "auto", None), "fp32": ("fp32", "auto", None), "events-fp64": ("fp64", "auto", None),
         "events-bf16": ("bf16", "auto", None), "self-delay": ("bf16", "auto", (2, 5)),
         "recompute": ("bf16", "recompute", None)}


def context(kind, k):
    import paper_1502_04993_amd as G
    precision, trace, delays = KINDS[kind]
    rec = synth.balanced(N=(40, 130)[k], B=(6_000, 5_000)[k], in_frac=0.2, seed=30 + k)
    if kind.startswith("events"):
        times, neu = synth.event_times(rec, seed=3)
        c = G.Context.from_events(rec.n_neurons, times, neu, 0.0, rec.T, precision=precision, trace=trace)
    else:
        c = G.Context(rec.n_neurons, rec.n_bins, rec.dt, precision=precision, trace=trace)
        if delays:
            c.set_delays(*delays)
        c.set_spikes(rec.bins, rec.neurons)
    c.set_kernel(rec.tau)
    return c, rec


@pytest.mark.parametrize("kind", list(KINDS))
def test_totals_are_of_the_parameters_held(kind):
    import paper_1502_04993_amd as G
    made = [context(kind, k) for k in range(2)]
    params = [[(s * rec.J, rec.mu + d) for _, rec in made] for s, d in ((1.0, 0.0), (0.5, -0.3))]
    b = G.Batch([c for c, _ in made])
    for p in params:
        for (c, _), (J, mu) in zip(made, p):
            c.set_params(J, mu)
        lls = b.eval()
        for k, (J, mu) in enumerate(p):
            c, _ = context(kind, k)
            c.set_params(J, mu)
            one = c.eval(grad=True)
            c.close()
            gJ, gmu = b.grad(k)
            assert lls[k] == one["ll"], (kind, k)
            assert np.array_equal(gJ, one["gJ"]) and np.array_equal(gmu, one["gmu"])
    # e^800 is not finite
    made[1][0].set_params(params[0][1][0], np.full(made[1][1].n_neurons, 800.0))
    with pytest.raises(G.GlmrError) as e:
        b.eval()
    assert e.value.status == G.L.GLMR_ENONFINITE
    made[1][0].set_params(*params[1][1])
    assert np.array_equal(b.eval(), lls)
    b.close()
    for c, _ in made:
        c.close()
