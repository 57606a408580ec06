"""The FP32 trailing update on split BF16 operands at the edges of its use: panels
and border heights that leave partial tiles, one and two packed slots
(lookahead), both mixed precisions.  Against the FP64 evaluation, at the
library's mixed-precision bars."""
import numpy as np
import pytest

from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    return binding.Library()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n,k,nb,look", [(513, 0, 512, 0), (640, 1, 512, 0), (641, 127, 128, 0), (700, 128, 256, 1),
                                         (1025, 129, 512, 1), (1300, 5, 1024, 0), (1664, 300, 512, 1)])
def test_against_fp64(lib, n, k, nb, look, prec):
    m = synth.dense_poisson(n, k, seed=n)
    m["Qprior"] = m["Qprior"] + 0.5 * np.eye(n)
    dms = [binding.DeviceModel(m)] * 3
    th = np.array([[0.0], [0.2], [-0.3]])
    ref, xr = lib.laplace_eval(dms, th)
    try:
        lib.tune_set(prec, n, 3, nb, 128, look)
        lib.tune_set("fp32", n, 3, nb, 128, look)
        res, x = lib.laplace_eval(dms, th, prec=prec)
    finally:
        lib.tune_set(prec, n, 3)
        lib.tune_set("fp32", n, 3)
    for a, b, u, v in zip(res, ref, x, xr):
        assert a["info"] == b["info"] == 0 and a["fallback"] == 0
        assert abs(a["logdet_qstar"] - b["logdet_qstar"]) <= 2e-6 * max(1.0, abs(b["logdet_qstar"]))
        assert abs(a["logdet_s"] - b["logdet_s"]) <= 1e-5 * max(1.0, abs(b["logdet_s"]))
        assert float((u - v).abs().max()) <= 1e-9 * max(1.0, float(v.abs().max()))
