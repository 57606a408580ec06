"""Orders and border heights whose last block column of 64 is padding alone (it takes
no panel step) and those around them: log-determinants with the returned factor, and
evaluations with the padding in the posterior, the kriging system and the prior, alone
and in an uneven batch, for every panel width.  Bars: 1e-12 relative for a
log-determinant in FP64 (n pivots of a few u each), 1e-9 for an evaluation."""
import numpy as np
import pytest
import torch

from oracle import inla_oracle as O
from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu
ORDERS = (1, 63, 64, 65, 128, 129, 192, 193, 320, 448, 449, 576, 640)


@pytest.fixture(scope="module")
def lib():
    return binding.Library()


@pytest.mark.parametrize("nb", [128, 256, 512, 1024])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_logdet(lib, prec, nb):
    mats = [synth.random_spd(n, seed=n) for n in ORDERS]
    lib.tune_set(prec, max(ORDERS), len(ORDERS), nb, 128 if prec == "bf16" else 64, 0)
    try:
        dev = [torch.tensor(q).cuda() for q in mats]
        ld, info = lib.logdet(dev, prec=prec)
    finally:
        lib.tune_set(prec, max(ORDERS), len(ORDERS))
    tol = {"fp64": 1e-12, "fp32": 1e-5, "bf16": 2e-2}[prec]
    for n, q, f, v, i in zip(ORDERS, mats, dev, ld, info):
        ref = np.linalg.cholesky(q)
        want = 2.0 * np.sum(np.log(np.diag(ref)))
        assert i == 0 and abs(v - want) <= tol * max(1.0, abs(want)), (n, v, want)
        low = np.tril(f.cpu().numpy().T)   # column-major factor
        assert np.max(np.abs(low - ref)) <= 10 * tol * np.max(np.abs(ref)), n


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shapes", [[(8, 8)], [(20, 16)], [(30, 15)], [(9, 7), (20, 16), (30, 15), (8, 8)]], ids=str)
def test_evaluation(lib, shapes, prec):
    ms = [synth.kron_poisson(a, b, seed=a * b) for a, b in shapes]
    ths = [synth.kron_theta0(b) for _, b in shapes]
    res, xs = lib.laplace_eval([binding.DeviceModel(m) for m in ms], np.stack(ths), prec=prec)
    for m, th, r, x in zip(ms, ths, res, xs):
        ref = O.laplace_eval(m, th)
        assert r["info"] == 0 and r["fallback"] == 0
        assert np.max(np.abs(x.cpu().numpy() - ref["x"])) <= 1e-9 * max(1.0, np.max(np.abs(ref["x"])))
        tol = 1e-9 if prec == "fp64" else 2e-6
        for key in ("objective", "logdet_qstar", "logdet_qprior"):
            assert abs(r[key] - ref[key]) <= (1e-9 if key == "logdet_qprior" else tol) * max(1.0, abs(ref[key])), key
