"""General design matrices whose columns differ in length, from empty to every
observation, next to each other: the columns' sums against the oracle's dense A."""
import numpy as np
import pytest

from oracle import inla_oracle as O
from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu

RTOL = 1e-9   # the library's bar for FP64 evaluations


def model(n, m_obs, lik, k, seed):
    rng = np.random.default_rng(seed)
    A = np.where(rng.random((m_obs, n)) < min(1.0, 3.0 / n), rng.normal(0.0, 0.5, size=(m_obs, n)), 0.0)
    A[:, 0] = 0.3                       # an intercept
    if n > 2:
        A[:, 1] = np.linspace(-0.5, 0.5, m_obs)
        A[:, 2] = 0.0                   # an effect without observations
    A[:, n - 1] = rng.normal(0.0, 0.2, size=m_obs)
    x = rng.normal(0.0, 0.3, size=n)
    E = rng.uniform(5.0, 50.0, size=m_obs) if lik == "poisson" else None
    y = rng.poisson(E * np.exp(A @ x)).astype(np.float64) if lik == "poisson" else A @ x + rng.normal(size=m_obs)
    C = rng.normal(size=(k, n)) if k else None
    return {"n": n, "lik": lik, "prior": "dense", "y": y, "E": E, "A": A, "C": C,
            "e": rng.normal(0.0, 0.1, size=k) if k else None, "coords": None, "n_s": n, "n_t": 1,
            "Qprior": synth.random_spd(n, seed + 7, shift=1.0)}


@pytest.mark.parametrize("lik", ["gaussian", "poisson"])
@pytest.mark.parametrize("n,m_obs,k", [(1, 3, 0), (3, 700, 1), (5, 1, 0), (66, 257, 2), (131, 900, 0), (259, 40, 130)])
def test_columns(n, m_obs, k, lik):
    lib = binding.Library()
    models = [model(n, m_obs, lik, k, seed=n + m_obs), model(n, m_obs, lik, k, seed=n)]
    plain = synth.dense_poisson(n, 0, seed=1)          # A = I in the same batch
    models.insert(1, plain)
    th = np.array([[0.1], [0.0], [-0.2]])
    dms = [binding.DeviceModel(m) for m in models]
    res, xs = lib.laplace_eval(dms, th)
    var, info = lib.marginal_var(dms, th, xs)
    for b, m in enumerate(models):
        ref = O.laplace_eval(m, th[b])
        assert res[b]["info"] == 0 and info[b] == 0
        for f in ("objective", "xqx", "loglik", "logdet_qstar", "logdet_s"):
            assert abs(res[b][f] - ref[f]) <= RTOL * max(1.0, abs(ref[f])), (b, f, res[b][f], ref[f])
        x = xs[b].cpu().numpy()
        assert np.max(np.abs(x - ref["x"])) <= RTOL * max(1.0, np.max(np.abs(ref["x"])))
        want = O.marginal_var(m, th[b], ref["x"])
        assert np.max(np.abs(var[b].cpu().numpy() - want)) <= RTOL * max(1.0, np.max(want))
