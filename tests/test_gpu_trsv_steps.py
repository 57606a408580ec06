"""Solves of a pass: triangular solves in steps of 256 rows at the edges of their blocks: orders just
below, at and above multiples of 64, 128 and 256, alone and as an uneven batch
(whose shorter matrices join the chain late or leave it early).  Against the
oracle: the mode is solved or refined to FP64 accuracy, 1e-9 relative.  The kriging
factor's solves and the border's products at border heights that take one block of
256, a partial second one and a third, with prior precisions of one and of several
workgroups per block column (Q_prior v)."""
import numpy as np
import pytest

from oracle import inla_oracle as O
from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu
ORDERS = (1, 63, 128, 129, 250, 256, 257, 384, 500, 513, 640, 769)


@pytest.fixture(scope="module")
def lib():
    return binding.Library()


def model(n, k=2):
    m = synth.dense_poisson(n, k if n > 2 else 0, seed=n)
    m["Qprior"] = m["Qprior"] + 0.5 * np.eye(n)
    return m


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("orders", [(n,) for n in ORDERS] + [ORDERS, ORDERS[::-1]], ids=str)
def test_modes(lib, orders, prec):
    ms = [model(n) for n in orders]
    th = np.linspace(-0.3, 0.2, len(orders))[:, None]
    res, xs = lib.laplace_eval([binding.DeviceModel(m) for m in ms], th, prec=prec)
    for m, t, r, x in zip(ms, th, res, xs):
        ref = O.laplace_eval(m, t)
        assert r["info"] == 0 and r["fallback"] == 0
        err = np.max(np.abs(x.cpu().numpy()[:len(ref["x"])] - ref["x"]))
        assert err <= 1e-9 * max(1.0, np.max(np.abs(ref["x"]))), (len(ref["x"]), err)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,k", [(300, 128), (321, 129), (513, 256), (700, 257), (900, 520)])
def test_borders(lib, n, k, prec):
    m, t = model(n, k), np.array([0.1])
    res, xs = lib.laplace_eval([binding.DeviceModel(m)], t[None], prec=prec)
    ref = O.laplace_eval(m, t)
    assert res[0]["info"] == 0 and res[0]["fallback"] == 0
    err = np.max(np.abs(xs[0].cpu().numpy() - ref["x"]))
    assert err <= 1e-9 * max(1.0, np.max(np.abs(ref["x"])))
    assert abs(res[0]["xqx"] - ref["xqx"]) <= 1e-9 * max(1.0, abs(ref["xqx"]))
    # the constraints' term: w = L_S^{-1} (C x_u - e) and log|S|
    assert abs(res[0]["logdet_s"] - ref["logdet_s"]) <= (1e-9 if prec == "fp64" else 1e-5) * max(1.0, abs(ref["logdet_s"]))
