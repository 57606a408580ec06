"""The packed panel copies of the FP32 and BF16 factorisations of an evaluation:
every order and every way of running (lookahead on and off, pass graphs on and
off, profiled, alone or beside other orders) multiplies with the same kernel, so
the results agree bit for bit."""
import numpy as np
import pytest

from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu

KEYS = ("objective", "logdet_qprior", "logdet_sprior", "ese", "xqx", "loglik", "logdet_qstar", "logdet_s", "step",
        "iters", "info", "ir_steps", "fallback")


def dense(n, k, seed):
    m = synth.dense_poisson(n, k, seed=seed)
    m["Qprior"] = m["Qprior"] + 0.5 * np.eye(n)
    return binding.DeviceModel(m)


def same(a, b, what):
    import torch
    for (r, x), (s, y) in zip(zip(*a), zip(*b)):
        for f in KEYS:
            assert r[f] == s[f], (what, f, r[f], s[f])
        assert torch.equal(x, y), what


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n,k,nb", [(1025, 129, 512), (200, 3, 128), (129, 0, 128), (1200, 700, 1024)])
def test_every_way_of_running(n, k, nb, prec):
    dms = [dense(n, k, n)] * 3
    th = np.array([[0.0], [0.2], [-0.3]])

    def handle(look, graphs, passes):
        lib = binding.Library()
        lib.set_lookahead(look)
        lib.set_graphs(graphs)
        lib.set_pass_graphs(passes)
        for p in ("fp32", "bf16"):
            lib.tune_set(p, n, 3, nb, 128, 1)
        return lib

    ref = handle(False, False, False).laplace_eval(dms, th, prec=prec)
    assert [r["info"] for r in ref[0]] == [0, 0, 0]
    for look, graphs, passes in [(True, False, False), (False, True, False), (True, True, False), (False, True, True),
                                 (True, True, True)]:
        lib = handle(look, graphs, passes)
        for rep in range(3):
            same(lib.laplace_eval(dms, th, prec=prec), ref, (look, graphs, passes, rep))
    lib = handle(True, True, True)
    lib.profile(True)
    same(lib.laplace_eval(dms, th, prec=prec), ref, "profiled")


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_alone_and_beside_small_orders(prec):
    small, large = [dense(100, 0, 1), dense(400, 5, 2), dense(500, 140, 3)], [dense(1300, 7, 4), dense(1900, 129, 5)]
    for d in small + large:
        alone = binding.Library().laplace_eval([d], np.array([[0.1]]), prec=prec)
        assert alone[0][0]["info"] == 0 and alone[0][0]["fallback"] == 0
        batch = [large[0], *small, large[1]]
        res, x = binding.Library().laplace_eval(batch, np.full((5, 1), 0.1), prec=prec)
        i = [id(m) for m in batch].index(id(d))
        same(([res[i]], [x[i]]), alone, d.n)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n,k", [(1, 0), (2, 1), (128, 40), (129, 0), (400, 5), (500, 140), (512, 0), (639, 130)])
def test_small_orders_against_fp64(n, k, prec):
    """Orders of few panels, at the library's mixed-precision bars."""
    lib = binding.Library()
    dms = [dense(n, k, n)] * 2
    th = np.array([[0.0], [0.2]])
    ref, xr = lib.laplace_eval(dms, th)
    res, x = lib.laplace_eval(dms, th, prec=prec)
    for a, b, u, v in zip(res, ref, x, xr):
        assert a["info"] == b["info"] == 0 and a["fallback"] == 0
        assert abs(a["logdet_qstar"] - b["logdet_qstar"]) <= 2e-6 * max(1.0, abs(b["logdet_qstar"]))
        assert abs(a["logdet_s"] - b["logdet_s"]) <= 1e-5 * max(1.0, abs(b["logdet_s"]))
        assert float((u - v).abs().max()) <= 1e-9 * max(1.0, float(v.abs().max()))
