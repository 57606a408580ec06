"""The concurrent prior pass where it runs: priors that are factored (dense ones)
beside priors of the structured pass, one that cannot be factored among them.  The
aux stream's pass has a workspace of its own, by which the tests see that it ran."""
import numpy as np
import pytest

from oracle import inla_oracle as O
from paper_2311_08050_amd import binding, synth

pytestmark = pytest.mark.gpu

KEYS = ("objective", "logdet_qprior", "logdet_sprior", "ese", "xqx", "loglik", "logdet_qstar", "logdet_s", "iters",
        "info", "ir_steps", "fallback")


def case():
    """Orders on both sides of a 512-wide panel; theta rows (the dense priors' are
    their likelihood parameter)."""
    models, thetas = [], []
    for n_s, n_t, dense in ((30, 6, False), (45, 20, True), (20, 8, True), (60, 12, True), (70, 10, False)):
        m = synth.kron_poisson(n_s, n_t, seed=n_s)
        th = synth.kron_theta0(n_t)
        if dense:
            m = dict(m, Qprior=O.prior_precision(m, th), prior="dense")
            th = np.array([th[-1], 0.0, 0.0, 0.0])
        models.append(m)
        thetas.append(th)
    bad = dict(models[2], Qprior=models[2]["Qprior"].copy())
    bad["Qprior"][100, 100] = -1.0   # leading minor 101
    models.append(bad)
    thetas.append(thetas[2])
    return [binding.DeviceModel(m) for m in models], np.stack(thetas)


def aux_bytes(dms):
    """Bytes of the bordered FP64 matrices that the concurrent pass keeps."""
    up = lambda v: -(-v // 128) * 128
    return sum(8 * (up(d.n) + up(d.k + 1)) ** 2 for d in dms if d.model["prior"] == "dense")


def run(overlap, graphs, dms, th, prec, reps):
    import torch
    torch.cuda.synchronize()
    lib = binding.Library()
    lib.set_overlap(overlap)
    lib.set_graphs(graphs)
    out, used = [], []
    for _ in range(reps):
        free = torch.cuda.mem_get_info()[0]
        out.append(lib.laplace_eval(dms, th, prec=prec))
        torch.cuda.synchronize()
        used.append(free - torch.cuda.mem_get_info()[0])
    return lib, out, used[0]   # (the workspace is taken by the first call)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_dense_priors_beside_structured(prec):
    import torch
    dms, th = case()
    torch.cuda.empty_cache()
    _, ref, plain = run(False, False, dms, th, prec, 1)
    assert [r["info"] for r in ref[0][0]] == [0, 0, 0, 0, 0, 101]
    for graphs in (False, True):
        lib, out, used = run(True, graphs, dms, th, prec, 4)
        assert used - plain >= 0.9 * aux_bytes(dms), (used, plain)   # the aux pass's workspace
        for rep, (res, x) in enumerate(out):
            for b, (r, s) in enumerate(zip(res, ref[0][0])):
                for f in KEYS:
                    assert r[f] == s[f], (graphs, rep, b, f, r[f], s[f])
                if s["info"] == 0:
                    assert torch.equal(x[b], ref[0][1][b]), (graphs, rep, b)
        if graphs and prec != "bf16":
            st = lib.pass_graph_stats()
            assert st["captured"] > 0 and st["replays"] > st["captured"], st
    m1, _ = lib.constrained_mode(dms, th, prec=prec)
    assert [(r["info"], r["iters"]) for r in m1] == [(r["info"], r["iters"]) for r in ref[0][0]]
