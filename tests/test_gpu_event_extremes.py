"""Continuous time at potentials far past the ordinary (needs an MI355X): an
absolute refractory time as a self-inhibition of -1e6, and weights whose
likelihood is not finite.

The recurrence against the dense contractions (GLMR_RECUR=0, closed forms).
Their potentials of up to 1e6 differ by a few units of 1e-16 each, the
likelihood's spike term is of that size too: 1e-11 of the largest value, as in
the other comparisons of the two paths.
"""
import numpy as np
import pytest

from test_gpu_recurrence import params

pytestmark = pytest.mark.gpu


def events(N, T, seed):
    rng = np.random.default_rng(seed)
    n = int(7 * N * T)
    times = np.sort(rng.random(n) * T)
    return times, np.concatenate([np.arange(N), rng.integers(0, N, n)])[:n].astype(np.int32)


def context(N, T, times, neu, precision, mode, monkeypatch):
    import paper_1502_04993_amd as G
    monkeypatch.setenv("GLMR_RECUR", mode)
    c = G.Context.from_events(N, times, neu, 0.0, T, precision=precision)
    c.set_kernel(0.01)
    return c


@pytest.mark.parametrize("N,T,precision,J_self", [(12, 5.0, "fp64", -1e6), (150, 2.0, "fp64", -300.0), (70, 2.0, "fp32", -40.0)])
def test_absolute_refractory_time(N, T, precision, J_self, monkeypatch):
    times, neu = events(N, T, N)
    J, mu = params(N, N)
    np.fill_diagonal(J, J_self)
    J = J.astype(np.float32).astype(np.float64)
    out = []
    for mode in "01":
        c = context(N, T, times, neu, precision, mode, monkeypatch)
        c.set_params(J, mu)
        out.append(c.eval(grad=True))
        c.close()
    tol = 1e-11 if precision == "fp64" else 1e-7 * abs(J_self)  # FP32: the dense trace is rounded, times J
    for k in ("ll", "ll_rows", "gJ", "gmu"):
        a, b = np.asarray(out[1][k]), np.asarray(out[0][k])
        assert np.max(np.abs(a - b)) <= tol * max(1.0, np.max(np.abs(b))), k


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_not_finite(precision, monkeypatch):
    import paper_1502_04993_amd as G
    N, T = 20, 2.0
    times, neu = events(N, T, 5)
    J, mu = params(N, 5)
    c = context(N, T, times, neu, precision, "1", monkeypatch)
    c.set_params(J, mu)
    ok = c.eval(grad=True)
    for bad in (1e6, 1e18, 1e300, np.inf, -np.inf, np.nan):
        K = J.copy()
        K[3, 4] = bad
        c.set_params(K, mu)
        with pytest.raises(G.GlmrError) as e:
            c.eval(grad=True)
        assert e.value.status == G.L.GLMR_ENONFINITE, bad
    c.set_params(J, mu)
    again = c.eval(grad=True)
    assert again["ll"] == ok["ll"] and np.array_equal(again["gJ"], ok["gJ"])
    c.close()


def test_empty_slot_between_tied_events(monkeypatch):
    """Between two events at one time the potential may be past e^709, over no time at all."""
    N, T = 6, 1.0
    times, neu = events(N, T, 6)
    J, mu = params(N, 6)
    at = np.searchsorted(times, 0.5)
    times = np.insert(times, at, [0.5, 0.5])
    neu = np.insert(neu, at, [1, 2]).astype(np.int32)
    J[0, 1], J[0, 2] = 1024.0, -1024.0
    mask = (neu != 1) & (neu != 2)
    mask[at:at + 2] = True
    extra = np.array([0.9, 0.9])  # 1 and 2 spike in pairs only
    times, neu = np.append(times[mask], extra), np.append(neu[mask], [1, 2]).astype(np.int32)
    order = np.lexsort((neu, times))
    times, neu = times[order], neu[order]
    out = []
    for mode in "01":
        c = context(N, T, times, neu, "fp64", mode, monkeypatch)
        c.set_params(J, mu)
        out.append(c.eval(grad=True))
        c.close()
    for k in ("ll", "gJ", "gmu"):
        a, b = np.asarray(out[1][k]), np.asarray(out[0][k])
        assert np.all(np.isfinite(b)) and np.max(np.abs(a - b)) <= 1e-11 * max(1.0, np.max(np.abs(b))), k
