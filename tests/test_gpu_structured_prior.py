"""The prior pass of the built priors (space x time: block diagonal in the temporal
eigenbasis; exponential covariance: from the factor of Sigma) against the
general pass, which the same prior takes when it is supplied as a dense matrix."""
import numpy as np
import pytest

from oracle import inla_oracle as O
from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    return binding.Library()


def _as_dense(model, th):
    """The same model with its prior precision supplied by the caller."""
    m = dict(model)
    m["Qprior"] = O.prior_precision(model, th)
    m["prior"] = "dense"
    return m, np.asarray(th)[-1:]


def _compare(lib, models, thetas):
    dms = [binding.DeviceModel(m) for m in models]
    res, x = lib.laplace_eval(dms, thetas)
    pairs = [_as_dense(m, t) for m, t in zip(models, thetas)]
    ref, xr = lib.laplace_eval([binding.DeviceModel(m) for m, _ in pairs], np.stack([t for _, t in pairs]))
    for a, b, u, v, m, t in zip(res, ref, x, xr, models, thetas):
        assert a["info"] == b["info"] == 0
        # both log-determinants carry a few ulp per pivot times the condition of
        # Q_prior (at most 1e5 here): 1e-9 is the library's bar for them
        for f in ("objective", "logdet_qprior", "logdet_sprior", "ese", "xqx", "loglik", "logdet_qstar", "logdet_s"):
            assert abs(a[f] - b[f]) <= 1e-9 * max(1.0, abs(b[f])), (f, a[f], b[f])
        assert float((u - v).abs().max()) <= 1e-9 * max(1.0, float(v.abs().max()))


@pytest.mark.parametrize("n_s,n_t,k", [(2, 2, None), (5, 1, 2), (1, 7, 3), (63, 3, 0), (64, 5, 1), (65, 4, None),
                                       (20, 33, None), (130, 4, 129), (9, 40, 16), (127, 2, 130)])
def test_space_time(lib, n_s, n_t, k):
    m = synth.kron_poisson(n_s, n_t, seed=n_s + n_t, constrained=k is None)
    rng = np.random.default_rng(n_s)
    if k:   # general constraint rows with a right-hand side
        m["C"] = rng.normal(size=(k, m["n"]))
        m["e"] = rng.normal(0.0, 0.2, size=k)
    th = np.stack([[0.3, -1.2, -4.0, 0.1], [-0.5, -2.0, -2.5, -0.2], [1.0, -1.6, -4.6, 0.0]])
    _compare(lib, [m] * 3, th)


@pytest.mark.parametrize("n,k", [(2, 1), (63, 0), (64, 1), (130, 16), (130, 17), (257, 3)])
def test_exponential_covariance(lib, n, k):
    m = synth.expcov_gaussian(n, seed=n)
    rng = np.random.default_rng(n)
    if k:
        m["C"] = rng.normal(size=(k, n))
        m["e"] = rng.normal(0.0, 0.2, size=k)
    _compare(lib, [m, m], np.array([[0.2, -1.6, -1.4], [-0.4, -1.0, -0.7]]))


@pytest.mark.parametrize("overlap", [False, True])
def test_mixed_batch_and_failures(lib, overlap):
    """Structured and factored priors in one call; dependent constraints and a
    singular prior are reported as the general pass reports them."""
    good = synth.kron_poisson(30, 6, seed=1)
    dep = dict(good, C=np.concatenate([good["C"], good["C"][:1] + good["C"][1:2]]), e=np.zeros(good["C"].shape[0] + 1))
    exp = synth.expcov_gaussian(100, seed=2, constrained=True)
    th_k = [0.3, -1.2, -4.0, 0.1]
    dense, th_d = _as_dense(good, th_k)
    models = [good, dep, exp, dense, good]
    th = np.zeros((5, 4))
    th[0] = th[1] = th_k
    th[2, :3] = [0.2, -1.6, -1.4]
    th[3, :1] = th_d
    th[4] = [0.3, -1.2, -800.0, 0.1]   # delta underflows to zero: Q_prior is singular
    try:
        lib.set_overlap(overlap)
        res, _ = lib.laplace_eval([binding.DeviceModel(m) for m in models], th)
    finally:
        lib.set_overlap(False)
    assert [r["info"] for r in res[:4]] == [0, binding.INFO_CONSTRAINT_RANK, 0, 0]
    assert res[4]["info"] != 0
    assert abs(res[0]["objective"] - res[3]["objective"]) <= 1e-9 * abs(res[3]["objective"])
