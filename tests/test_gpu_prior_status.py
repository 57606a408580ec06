"""Built priors that are singular to rounding are reported as the factorisation of
Q_prior reports them, whichever way their prior terms are computed."""
import numpy as np
import pytest

from oracle import inla_oracle as O
from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("constrained", [False, True])
@pytest.mark.parametrize("n_s,n_t,log_delta", [(30, 6, -60.0), (64, 5, -80.0), (20, 33, -50.0), (130, 4, -120.0)])
def test_delta_below_rounding(n_s, n_t, log_delta, constrained):
    lib = binding.Library()
    m = synth.kron_poisson(n_s, n_t, seed=n_s, constrained=constrained)
    th = synth.kron_theta0(n_t)
    low = th.copy()
    low[2] = log_delta
    dense = binding.DeviceModel(dict(m, Qprior=O.prior_precision(m, low), prior="dense"))
    ref, _ = lib.laplace_eval([dense], low[None, -1:])
    dm = binding.DeviceModel(m)
    res, _ = lib.laplace_eval([dm, dm], np.stack([th, low]))
    # the general pass stops at a pivot of the last n_s (the others carry R_t's part)
    assert ref[0]["info"] > n_s * (n_t - 1)
    assert res[0]["info"] == 0
    assert res[1]["info"] > n_s * (n_t - 1)


@pytest.mark.parametrize("n,pairs", [(60, 3), (130, 1), (130, 3)])
def test_points_a_rounding_apart(n, pairs):
    """Pairs of points 2 to 16 half-ulps of their correlation apart: Sigma has a factor,
    but Q_prior = tau Sigma^{-1}, with elements of 1e15 and an eigenvalue below 1, mostly
    has none in 64 bits (the same for every call: several distances, one of which at least
    is refused).  At 1e-9 every one is accepted."""
    lib = binding.Library()
    info = []
    for d in [j * 2.0**-54 for j in range(2, 17)] + [1e-9]:
        m = synth.expcov_gaussian(n, seed=n)
        c = np.array(m["coords"], dtype=np.float64)
        for q in range(pairs):
            c[2 * q] = [0.25 * (q + 1), 0.25]
            c[2 * q + 1] = [0.25 * (q + 1), 0.25 + d]
        res, _ = lib.laplace_eval([binding.DeviceModel(dict(m, coords=c))], np.array([[0.2, 0.0, -1.4]]))
        info.append(res[0]["info"])
    assert all(0 <= i <= n for i in info) and info[-1] == 0
    assert any(i > 0 for i in info[:-1]), info


@pytest.mark.parametrize("n_s,n_t,log_delta", [(30, 6, -20.0), (64, 5, -22.0)])
def test_small_delta_is_accepted(n_s, n_t, log_delta):
    """Well above rounding: both ways accept, and each of the n_s pivots of size tau delta
    agrees to n roundings of Q_prior's largest element (below 100 tau)."""
    lib = binding.Library()
    m = synth.kron_poisson(n_s, n_t, seed=n_s)
    th = synth.kron_theta0(n_t)
    th[2] = log_delta
    dense = binding.DeviceModel(dict(m, Qprior=O.prior_precision(m, th), prior="dense"))
    (r,), _ = lib.laplace_eval([binding.DeviceModel(m)], th[None])
    (s,), _ = lib.laplace_eval([dense], th[None, -1:])
    assert r["info"] == s["info"] == 0
    assert abs(r["logdet_qprior"] - s["logdet_qprior"]) <= n_s * n_s * n_t * 2.3e-16 * 100.0 / np.exp(log_delta)
