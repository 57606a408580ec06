"""The diagonal-block factorisation of the blocked Cholesky at the edges of its
16-wide sub-panels, at scales where 1 / pivot leaves the FP64 range, and at a
failing pivot in every sub-panel (``inla_logdet`` against numpy)."""
import numpy as np
import pytest

from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def lib():
    return binding.Library()


def _factor(lib, Q):
    import torch
    m = torch.as_tensor(Q).cuda()
    ld, info = lib.logdet([m])
    return float(ld[0]), int(info[0]), np.triu(m.cpu().numpy()).T   # column-major lower triangle


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 48, 63, 64, 65, 127, 130])
@pytest.mark.parametrize("exponent", [-960, 0, 960])
def test_factor_and_logdet(lib, n, exponent):
    Q0 = synth.random_spd(n, seed=n)
    ld, info, L = _factor(lib, np.ldexp(Q0, exponent))
    assert info == 0
    # backward error of Cholesky: |L L^T - Q| <= gamma_{n+1} |L| |L^T| elementwise,
    # at most (n + 1) eps times the largest diagonal entry; doubled for the
    # multiplications by reciprocals
    L0 = np.ldexp(L, -exponent // 2)
    assert np.max(np.abs(L0 @ L0.T - Q0)) <= 2 * (n + 1) * EPS * np.max(np.diag(Q0))
    ref = np.linalg.slogdet(Q0)[1] + n * exponent * np.log(2.0)
    assert abs(ld - ref) <= 1e-12 * max(1.0, abs(ref))


@pytest.mark.parametrize("bad", [1, 2, 16, 17, 32, 33, 48, 49, 64, 65, 100])
@pytest.mark.parametrize("value", [-1.0, 0.0, float("nan")])
def test_first_failing_pivot(lib, bad, value):
    Q = synth.random_spd(100, seed=7)
    Q[bad - 1, bad - 1] = value
    ld, info, _ = _factor(lib, Q)
    assert info == bad and np.isnan(ld)


@pytest.mark.parametrize("prec,unit", [("fp64", EPS), ("fp32", 2.0 ** -23)])
@pytest.mark.parametrize("nb", [128, 256, 512])
def test_panels_of_an_uneven_batch(lib, prec, unit, nb):
    """Every panel step's tile 0 (updated one step ahead inside a panel, not at
    its first two columns nor at its end), with panels that end early in some
    matrices of the batch."""
    import torch
    ns = [65, 128, 129, 192, 257, 320, 385, 513, 577, 640, 769, 1025]
    Qs = [synth.random_spd(n, seed=n) for n in ns]
    mats = [torch.as_tensor(Q).cuda() for Q in Qs]
    try:
        lib.tune_set(prec, max(ns), len(ns), nb, 64, 0)
        ld, info = lib.logdet(mats, prec=prec)
    finally:
        lib.tune_set(prec, max(ns), len(ns))
    assert not info.any()
    for Q, m, v in zip(Qs, mats, ld):
        L = np.triu(m.cpu().numpy()).T
        n = len(Q)
        # as above, the bound of a blocked Cholesky with explicit block inverses
        # (condition at most 10 here)
        assert np.max(np.abs(L @ L.T - Q)) <= 2 * (n + 1) * unit * np.max(np.diag(Q))
        ref = np.linalg.slogdet(Q)[1]
        assert abs(v - ref) <= 4 * n * unit * max(1.0, abs(ref))
