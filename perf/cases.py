"""The library's work by size: cases that a timing program can prepare and run.

Each case is a call, or the short chain of calls, that a program doing dense
INLA makes: a batch of Laplace evaluations (Stage 1, exploration, mixed
precision), the posterior of a batch of modes, the Moore-Penrose route, plain
log-determinants and the warm-start network's gradient.  ``listed`` names twelve
of them over the sizes of this repository's workloads, ``draw`` gives others of
the same ranges, ``prepare`` makes inputs, ``run`` is one pass, ``work`` what it
cannot do without, ``exact`` the same outputs from plain torch in 64 bits.

A mixed-precision evaluation's objective, log|Q*| and log|S| come from an FP32
factor, so ``run`` keeps those as float32; its modes and prior terms are
computed to 64 bits and stay float64.
"""
import math

import numpy as np
import torch

from paper_2311_08050_amd import binding, synth

# Flops of a pass beyond which the 64-bit comparison would take too long.
EXACT_FLOPS = 2.5e13
# Newton iterations from each kind of start (Poisson; a Gaussian likelihood takes one).
NEWTON = {"zero": 6, "stage1": 2, "learned": 2}
# The largest evaluation that is drawn, in flops of its Newton factorisations.
DRAW_FLOPS = {"fp64": 8.0e12, "fp32": 8.0e12, "bf16": 8.0e12}


def listed():
    return [
        # the smallest evaluation: exponential-covariance Gaussian model, theta0 and its six
        # finite-difference neighbours; a call of about a millisecond, all launches and latency
        {"name": "expcov400", "kind": "laplace", "model": "expcov", "n": 400, "batch": 7, "prec": "fp64",
         "start": "zero", "constrained": False, "overlap": False},
        # plain log-determinants (Gaussian normalisers) of a small batch of dense matrices
        {"name": "logdet1000", "kind": "logdet", "n": 1000, "batch": 8},
        # the 100 regions x 30 times Poisson model with 129 constraints, 9 theta from zero
        {"name": "kron3000", "kind": "laplace", "model": "kron", "n_s": 100, "n_t": 30, "batch": 9, "prec": "fp64",
         "start": "zero", "constrained": True, "overlap": False},
        # a CCD batch (t = 4: 25 points) of a small space-time model in mixed precision
        {"name": "ccd1024_fp32", "kind": "laplace", "model": "kron", "n_s": 32, "n_t": 32, "batch": 25,
         "prec": "fp32", "start": "zero", "constrained": True, "overlap": False},
        # theta of several data sets of different orders in one call (the batching workload's shapes)
        {"name": "uneven", "kind": "uneven", "batch": 20, "prec": "fp64"},
        # Stage 1 at the headline's order: a central-difference gradient, every point started
        # from the mode at the current theta
        {"name": "stage1_8192", "kind": "laplace", "model": "kron", "n_s": 128, "n_t": 64, "batch": 8,
         "prec": "fp64", "start": "stage1", "constrained": True, "overlap": False},
        # the headline's variant: mixed precision from the learned warm start, the prior pass
        # beside the Newton iteration, on a CCD batch
        {"name": "ccd8192_learned", "kind": "laplace", "model": "kron", "n_s": 128, "n_t": 64, "batch": 25,
         "prec": "fp32", "start": "learned", "constrained": True, "overlap": True},
        # the largest order: 128 regions x 128 times with BF16 trailing updates
        {"name": "kron16384_bf16", "kind": "laplace", "model": "kron", "n_s": 128, "n_t": 128, "batch": 2,
         "prec": "bf16", "start": "zero", "constrained": True, "overlap": False},
        # Stage 2 at the explored points: marginal variances, then the variational-Bayes mean
        {"name": "posterior3000", "kind": "posterior", "n_s": 100, "n_t": 30, "batch": 9},
        # an intrinsic prior on the Moore-Penrose route: evaluation and variances
        {"name": "intrinsic3000", "kind": "woodbury", "n_s": 100, "n_t": 30, "batch": 9},
        # the pseudo-inverses of the Type IV prior's structure blocks (orders 5, 200 and 1000)
        {"name": "pinv1000", "kind": "pinv", "n_s": 200, "n_t": 5, "graph": "random"},
        # one gradient of the warm-start network (4 -> 256 -> 256 -> n) on a training batch
        {"name": "mlp8192", "kind": "mlp", "n": 8192, "hidden": 256, "batch": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["expcov", "kron", "kron", "kron", "logdet", "uneven", "posterior", "woodbury", "pinv", "mlp"])
    if kind == "expcov":
        return {"kind": "laplace", "model": "expcov", "n": _log_int(rng, 64, 2048), "batch": rng.randint(1, 15),
                "prec": rng.choice(["fp64", "fp64", "fp32"]), "start": "zero",
                "constrained": rng.random() < 0.5, "overlap": False}
    if kind == "kron":
        n_s = _log_int(rng, 12, 128)
        n_t = _log_int(rng, 6, 128)
        prec = rng.choice(["fp64", "fp64", "fp32", "fp32", "bf16"])
        c = {"kind": "laplace", "model": "kron", "n_s": n_s, "n_t": n_t, "batch": 1, "prec": prec,
             "start": rng.choice(["zero", "stage1", "learned"]), "constrained": rng.random() < 0.8,
             "overlap": rng.random() < 0.3}
        most = int(DRAW_FLOPS[prec] / work(c)["flops"])
        c["batch"] = max(1, min(most, 8 if c["start"] == "stage1" else rng.randint(1, 32)))
        return c
    if kind == "logdet":
        return {"kind": "logdet", "n": _log_int(rng, 32, 4096), "batch": rng.randint(1, 12)}
    if kind == "uneven":
        return {"kind": "uneven", "batch": rng.randint(5, 20), "prec": rng.choice(["fp64", "fp32"])}
    if kind == "posterior":
        return {"kind": "posterior", "n_s": _log_int(rng, 12, 100), "n_t": _log_int(rng, 5, 40),
                "batch": rng.randint(1, 9)}
    if kind == "woodbury":
        return {"kind": "woodbury", "n_s": _log_int(rng, 12, 100), "n_t": _log_int(rng, 4, 30),
                "batch": rng.randint(1, 9)}
    if kind == "pinv":
        n_t = rng.randint(3, 6)
        return {"kind": "pinv", "n_s": _log_int(rng, 10, 1000 // n_t), "n_t": n_t,
                "graph": rng.choice(["random", "delaunay"])}
    return {"kind": "mlp", "n": _log_int(rng, 100, 8192), "hidden": rng.choice([32, 64, 100, 128, 256]),
            "batch": rng.randint(16, 256)}


# ------------------------------------------------------------------- inputs
_handles = {}


def _library(overlap=False):
    """The program's handle (one with the concurrent prior pass, one without)."""
    if overlap not in _handles:
        _handles[overlap] = binding.Library()
        _handles[overlap].set_overlap(overlap)
    return _handles[overlap]


def _order(case):
    return case["n"] if "n" in case else case["n_s"] * case["n_t"]


def _models(case, seed):
    """(host models, theta rows): one model per theta (the same one repeated but for the uneven batch)."""
    B = case["batch"]
    if case["kind"] == "uneven":
        models = [synth.kron_poisson(ns, nt, seed=1000 * seed + i) for i, (ns, nt) in enumerate(synth.UNEVEN_SHAPES)]
        which = _uneven_shapes(B)
        rng = np.random.default_rng(seed)
        th = np.stack([synth.kron_theta0(synth.UNEVEN_SHAPES[w][1]) + 0.5 * rng.normal(size=4) for w in which])
        return [models[w] for w in which], th
    if case.get("model") == "expcov":
        m = synth.expcov_gaussian(case["n"], seed=seed, constrained=case["constrained"])
        th0 = np.array([0.0, math.log(0.2), math.log(0.25)])
        th = synth.fd_batch(th0, 0.01, [0, 1, 2])
        if B > len(th):
            th = np.concatenate([th, synth.normal_batch(th0, B - len(th), 0.3, seed + 1)])
        return [m] * B, np.ascontiguousarray(th[:B])
    if case["kind"] == "woodbury":
        m = synth.rw1_besag(case["n_s"], case["n_t"], seed=seed)
        return [m] * B, synth.normal_batch(synth.rw1_besag_theta0(case["n_t"]), B, 0.3, seed + 1)
    m = synth.kron_poisson(case["n_s"], case["n_t"], seed=seed, constrained=case.get("constrained", True))
    th0 = synth.kron_theta0(case["n_t"])
    if case.get("start") == "stage1":
        th0 = th0 + np.random.default_rng(seed).normal(0.0, 0.2, size=4)
        th = np.concatenate([synth.fd_batch(th0, 1e-3, [0, 1, 2, 3])[1:]] * (B // 8 + 1))[:B]
    elif B == 9 and case.get("start") == "zero":
        th = synth.fd_batch(th0 + np.random.default_rng(seed).normal(0.0, 0.2, size=4), 0.01, [0, 1, 2, 3])
    else:
        th = synth.normal_batch(th0, B, 0.5 if case["kind"] == "laplace" else 0.3, seed + 1)
    return [m] * B, np.ascontiguousarray(th)


def _uneven_shapes(B):
    """Shape indices of an uneven batch: every shape in turn, in a mixed order."""
    return [(3 * i + i // 5) % len(synth.UNEVEN_SHAPES) for i in range(B)]


def _device_models(models):
    made = {}
    for m in models:
        if id(m) not in made:
            made[id(m)] = binding.DeviceModel(m)
    return [made[id(m)] for m in models]


def _besag(n_s, edges):
    R = np.zeros((n_s, n_s))
    R[edges[:, 0], edges[:, 1]] = R[edges[:, 1], edges[:, 0]] = -1.0
    return R - np.diag(R.sum(axis=1))


def _rw(n_t, order):
    D = np.diff(np.eye(n_t), n=order, axis=0)
    return D.T @ D


def _pinv_blocks(case, seed):
    rng = np.random.default_rng(seed)
    n_s, n_t = case["n_s"], case["n_t"]
    edges = (synth.random_besag_graph(n_s, rng) if case["graph"] == "random"
             else synth.region_graph(synth.points(rng, n_s)))
    Rt, Rs = _rw(n_t, 2), _besag(n_s, edges)
    tau = np.exp(synth.type4_theta0()[:3] + rng.normal(0.0, 0.3, size=3))
    return [tau[0] * Rt, tau[1] * Rs, tau[2] * np.kron(Rt, Rs)]


def _spd(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    G = torch.randn((n, n + 8), dtype=torch.float64, device="cuda", generator=g)
    return G @ G.T / (n + 8) + 0.5 * torch.eye(n, dtype=torch.float64, device="cuda")


def _mlp_params(case, seed):
    H, O = case["hidden"], case["n"]
    g = torch.Generator().manual_seed(seed)
    parts = []
    for rows, cols, a in ((H, 4, math.sqrt(6 / 4)), (H, H, math.sqrt(6 / H)), (O, H, math.sqrt(3 / H))):
        parts.append((a * (2 * torch.rand(rows, cols, generator=g) - 1)).reshape(-1))
        parts.append(0.01 * torch.randn(rows, generator=g))
    x = torch.randn(case["batch"], 4, generator=g)
    target = torch.randn(case["batch"], O, generator=g, dtype=torch.float64)
    return torch.cat(parts), x, target


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "lib": _library(case.get("overlap", False))}
    lib = s["lib"]
    if kind == "logdet":
        s["mats"] = [_spd(case["n"], 100 * seed + i) for i in range(case["batch"])]
        return s
    if kind == "pinv":
        s["mats"] = [torch.as_tensor(b).cuda() for b in _pinv_blocks(case, seed)]
        return s
    if kind == "mlp":
        w, x, target = _mlp_params(case, seed)
        s["net"] = binding.Mlp(lib, 4, case["hidden"], case["n"], seed=seed)
        s["net"].set_params(w.cuda())
        s["x"], s["target"] = x.cuda(), target.cuda()
        return s
    models, th = _models(case, seed)
    s["models"], s["theta"] = _device_models(models), th
    if kind == "woodbury":
        m = models[0]
        P = np.kron(np.linalg.pinv(_rw(m["n_t"], 1), hermitian=True),
                    np.linalg.pinv(_besag(m["n_s"], m["edges"]), hermitian=True))
        s["prior"] = binding.PinvPrior([{"offset": 0, "P": torch.as_tensor(P).cuda(), "tau_index": 0}], lik_index=1)
    if kind == "posterior":
        _, s["modes"] = lib.constrained_mode(s["models"], th)
    s["x0"] = None
    if case.get("start") == "stage1":
        centre = (th[0] + th[1]) / 2
        _, x = lib.constrained_mode(s["models"][:1], centre[None])
        s["x0"] = [x[0].clone() for _ in models]
    elif case.get("start") == "learned":
        # a start as near as the trained network's: the mode, off by about 3e-4
        _, x = lib.constrained_mode(s["models"], th, prec=case["prec"])
        g = torch.Generator(device="cuda").manual_seed(seed)
        s["x0"] = [v + 1e-4 * torch.randn(v.shape, dtype=v.dtype, device="cuda", generator=g) for v in x]
    return s


# --------------------------------------------------------------------- pass
def _evaluated(res, x, mixed):
    low = np.float32 if mixed else np.float64
    of = lambda f, t=np.float64: np.array([r[f] for r in res], dtype=t)  # noqa: E731
    return {"objective": of("objective", low), "logdet_qstar": of("logdet_qstar", low),
            "logdet_s": of("logdet_s", low), "logdet_qprior": of("logdet_qprior"),
            "logdet_sprior": of("logdet_sprior"), "xqx": of("xqx"), "loglik": of("loglik"),
            "info": of("info", np.int32), "mode": x}


def run(s):
    case, lib = s["case"], s["lib"]
    kind = case["kind"]
    if kind in ("laplace", "uneven"):
        if s["x0"] is None:
            res, x = lib.laplace_eval(s["models"], s["theta"], prec=case["prec"])
        else:
            res, x = lib.laplace_eval(s["models"], s["theta"], x=[v.clone() for v in s["x0"]], start=1,
                                      prec=case["prec"])
        return _evaluated(res, x, case["prec"] != "fp64")
    if kind == "logdet":
        mats = [m.clone() for m in s["mats"]]   # the call overwrites its matrices with the factor
        ld, info = lib.logdet(mats)
        return {"logdet": ld, "info": info, "factor": mats}
    if kind == "posterior":
        var, info = lib.marginal_var(s["models"], s["theta"], s["modes"])
        mean, _, vinfo = lib.vb_mean(s["models"], s["theta"], var, s["modes"])
        return {"var": var, "mean": mean, "info": info, "vb_info": vinfo}
    if kind == "woodbury":
        P = lib.pinv_prior_assemble(s["prior"], s["models"][0].n, s["theta"])
        res, x = lib.woodbury_eval(s["models"], s["theta"][:, 1], P)
        var, info = lib.woodbury_var(s["models"], s["theta"][:, 1], P, x)
        return {"objective": np.array([r["objective"] for r in res]),
                "logdet_qstar": np.array([r["logdet_qstar"] for r in res]), "mode": x, "var": var, "info": info}
    if kind == "pinv":
        P, rank, _, info = lib.pinv(s["mats"])
        return {"pinv": P, "rank": rank, "info": info}
    loss, g = s["net"].grad(s["x"], s["target"])
    return {"loss": np.float32(loss), "grad": g}


# --------------------------------------------------------------------- work
def _constraints(case):
    if case.get("model") == "expcov":
        return 1 if case["constrained"] else 0
    if case["kind"] == "woodbury" or not case.get("constrained", True):
        return 0
    return case["n_s"] + case["n_t"] - 1


def _factor_flops(n, k):
    """Cholesky of order n with k + 1 border rows (constraints and right-hand side)."""
    return n ** 3 / 3 + n * n * (k + 1) + n * (k + 1) ** 2


def work(case):
    """The factorisations of the Newton iteration (and of what each call returns), inputs and outputs."""
    kind, B = case["kind"], case.get("batch", 1)
    if kind == "uneven":
        flops = bytes_ = 0.0
        for w in _uneven_shapes(B):
            ns, nt = synth.UNEVEN_SHAPES[w]
            flops += NEWTON["zero"] * _factor_flops(ns * nt, ns + nt - 1)
            bytes_ += 8.0 * ns * nt * (ns + nt + 2)
        return {"bytes": bytes_, "flops": flops}
    if kind == "pinv":
        orders = [case["n_t"], case["n_s"], case["n_s"] * case["n_t"]]
        # tridiagonal reduction, its back-transformation and the product of the eigenvectors
        return {"bytes": sum(16.0 * n * n for n in orders), "flops": sum((4 / 3 + 2 + 1) * n ** 3 for n in orders)}
    n = _order(case)
    if kind == "logdet":
        return {"bytes": B * 16.0 * n * n, "flops": B * n ** 3 / 3}
    if kind == "mlp":
        H = case["hidden"]
        params = H * 5 + H * H + H + n * H + n
        # forward, and in the backward pass the gradient of every weight and of the two hidden layers
        return {"bytes": 8.0 * params + 8.0 * B * n + 16.0 * B,
                "flops": 2.0 * B * (2 * 4 * H + 3 * H * H + 3 * n * H)}
    k = _constraints(case)
    io = 8.0 * n * (4 * B + 2 + k)
    if kind == "posterior":
        # variances: factor and its inverse; the mean correction: about three constrained solves
        return {"bytes": io, "flops": B * (2 * n ** 3 / 3 + n * n * (k + 1) + 3 * _factor_flops(n, k))}
    if kind == "woodbury":
        return {"bytes": io + 8.0 * n * n, "flops": B * ((NEWTON["zero"] + 1) * n ** 3 / 3 + n ** 3)}
    passes = 1 if case["model"] == "expcov" else NEWTON[case["start"]]
    return {"bytes": io, "flops": B * passes * _factor_flops(n, k)}


# ------------------------------------------------------------ 64-bit values
def _cuda(a):
    return torch.as_tensor(np.asarray(a, dtype=np.float64)).cuda()


def _logdet(L):
    return 2.0 * torch.log(torch.diagonal(L)).sum()


def _prior64(m, th):
    p = _cuda(m["coords"])
    # distances from coordinate differences: the Gram form would cancel
    d = torch.sqrt(((p[:, None, :] - p[None, :, :]) ** 2).sum(-1))
    inv = torch.cholesky_inverse(torch.linalg.cholesky(torch.exp(-d / math.exp(th[1]))))
    if m["prior"] == "expcov":
        return math.exp(th[0]) * inv.contiguous()
    Q = torch.kron(_cuda(_rw(m["n_t"], 1)), inv.contiguous())
    Q.diagonal().add_(math.exp(th[2]))
    return math.exp(th[0]) * Q


class _Laplace64:
    """Newton, kriging and the terms of the Laplace objective of one theta."""

    def __init__(self, m, th):
        self.m, self.lik = m, float(th[-1])
        self.y = _cuda(m["y"])
        self.E = None if m["E"] is None else _cuda(m["E"])
        self.C = None if m["C"] is None else _cuda(m["C"])
        self.e = None if m["C"] is None else _cuda(m["e"])
        self.Q = _prior64(m, th)

    def terms(self, x, var=None):
        """g, W and log-likelihood at x (expectations over N(x, var) of g and W with var)."""
        if self.m["lik"] == "gaussian":
            s2 = math.exp(self.lik)
            r = self.y - x
            ll = -0.5 * (r * r).sum() / s2 - 0.5 * len(r) * math.log(2 * math.pi * s2)
            return r / s2, torch.full_like(x, 1 / s2), ll
        eta = self.lik + x
        W = self.E * torch.exp(eta if var is None else eta + 0.5 * var)
        ll = (self.y * (torch.log(self.E) + eta) - W - torch.lgamma(self.y + 1)).sum()
        return self.y - W, W, ll

    def step(self, x, var=None):
        """The constrained Newton iterate from x, and the factors of Q* and S."""
        g, W, _ = self.terms(x, var)
        L = torch.linalg.cholesky(self.Q + torch.diag(W))
        new = torch.cholesky_solve((g + W * x)[:, None], L)[:, 0]
        LS = V = None
        if self.C is not None:
            V = torch.cholesky_solve(self.C.T.contiguous(), L)
            LS = torch.linalg.cholesky(self.C @ V)
            new = new - V @ torch.cholesky_solve((self.C @ new - self.e)[:, None], LS)[:, 0]
        return new, L, LS, V

    def mode(self, x, var=None):
        for _ in range(50):
            new = self.step(x, var)[0]
            moved = float((new - x).abs().max())
            x = new
            if self.m["lik"] == "gaussian" or moved <= 1e-11 * max(1.0, float(x.abs().max())):
                break
        return x

    def evaluate(self, x0):
        x = self.mode(x0)
        Lp = torch.linalg.cholesky(self.Q)
        ld_sp = ese = ld_s = torch.zeros((), dtype=torch.float64, device="cuda")
        if self.C is not None:
            LSp = torch.linalg.cholesky(self.C @ torch.cholesky_solve(self.C.T.contiguous(), Lp))
            ld_sp = _logdet(LSp)
            ese = self.e @ torch.cholesky_solve(self.e[:, None], LSp)[:, 0]
        _, L, LS, _ = self.step(x)
        if LS is not None:
            ld_s = _logdet(LS)
        ll = self.terms(x)[2]
        xqx = x @ (self.Q @ x)
        obj = 0.5 * (_logdet(Lp) + ld_sp + ese - xqx - _logdet(L) - ld_s) + ll
        return {"objective": obj, "logdet_qstar": _logdet(L), "logdet_s": ld_s, "logdet_qprior": _logdet(Lp),
                "logdet_sprior": ld_sp, "xqx": xqx, "loglik": ll, "mode": x}

    def variances(self, x):
        _, L, LS, V = self.step(x)
        Z = torch.linalg.solve_triangular(L, torch.eye(len(x), dtype=x.dtype, device="cuda"), upper=False)
        var = (Z * Z).sum(0)
        if LS is not None:
            U = torch.linalg.solve_triangular(LS, V.T, upper=False)
            var = var - (U * U).sum(0)
        return var


def _woodbury64(m, th):
    Rt, Rs = _rw(m["n_t"], 1), _besag(m["n_s"], m["edges"])
    tau = math.exp(th[0])
    P = _cuda(np.kron(np.linalg.pinv(Rt, hermitian=True), np.linalg.pinv(Rs, hermitian=True)) / tau)
    y, E = _cuda(m["y"]), _cuda(m["E"])
    x = torch.zeros(len(y), dtype=torch.float64, device="cuda")

    def factor(x):
        W = E * torch.exp(th[1] + x)
        s = torch.sqrt(W)
        M = s[:, None] * P * s[None, :]
        M.diagonal().add_(1.0)
        return W, s, torch.linalg.cholesky(M)

    for _ in range(50):
        W, s, L = factor(x)
        b = y - W + W * x
        u = P @ b
        z = b - s * torch.cholesky_solve((s * u)[:, None], L)[:, 0]
        new = P @ z
        moved = float((new - x).abs().max())
        x = new
        if moved <= 1e-12 * max(1.0, float(x.abs().max())):
            break
    W, s, L = factor(x)
    eta = th[1] + x
    ll = (y * (torch.log(E) + eta) - W - torch.lgamma(y + 1)).sum()
    G = torch.linalg.solve_triangular(L, s[:, None] * P, upper=False)
    # at the mode the gradient y - W equals Q_prior x on the prior's range
    return {"objective": ll - 0.5 * (x @ (y - W)) - 0.5 * _logdet(L), "logdet_qstar": _logdet(L), "mode": x,
            "var": torch.diagonal(P) - (G * G).sum(0)}


def _column(rows, field):
    return np.array([float(r[field]) for r in rows])


def exact(case, seed):
    kind = case["kind"]
    if work(case)["flops"] > EXACT_FLOPS or (kind == "laplace" and _order(case) > 10000):
        return None
    if kind == "logdet":
        mats = [_spd(case["n"], 100 * seed + i) for i in range(case["batch"])]
        L = [torch.linalg.cholesky(m) for m in mats]
        return {"logdet": np.array([float(_logdet(f)) for f in L]), "info": None,
                "factor": [torch.triu(f.T) + torch.tril(m, -1) for f, m in zip(L, mats)]}
    if kind == "pinv":
        out = [torch.as_tensor(np.linalg.pinv(b, rcond=1e-9, hermitian=True)).cuda() for b in _pinv_blocks(case, seed)]
        return {"pinv": out, "rank": None, "info": None}
    if kind == "mlp":
        H, O = case["hidden"], case["n"]
        w, x, target = _mlp_params(case, seed)
        w = w.double().cuda().requires_grad_(True)
        W1, b1, W2, b2, W3, b3 = torch.split(w, [H * 4, H, H * H, H, O * H, O])
        gelu = torch.nn.functional.gelu
        h = gelu(x.double().cuda() @ W1.view(H, 4).T + b1)
        h = gelu(h @ W2.view(H, H).T + b2)
        loss = ((h @ W3.view(O, H).T + b3 - target.cuda()) ** 2).mean()
        loss.backward()
        return {"loss": float(loss.detach()), "grad": w.grad}
    models, th = _models(case, seed)
    if kind == "woodbury":
        rows = [_woodbury64(m, t) for m, t in zip(models, th)]
        return {"objective": _column(rows, "objective"), "logdet_qstar": _column(rows, "logdet_qstar"),
                "mode": [r["mode"] for r in rows], "var": [r["var"] for r in rows], "info": None}
    zero = lambda m: torch.zeros(m["n"], dtype=torch.float64, device="cuda")  # noqa: E731
    if kind == "posterior":
        out = {"var": [], "mean": [], "info": None, "vb_info": None}
        for m, t in zip(models, th):
            p = _Laplace64(m, t)
            x = p.mode(zero(m))
            out["var"].append(p.variances(x))
            out["mean"].append(p.mode(x, out["var"][-1]))
        return out
    rows, x = [], None
    for m, t in zip(models, th):
        near = x is not None and kind == "laplace"
        rows.append(_Laplace64(m, t).evaluate(x if near else zero(m)))
        x = rows[-1]["mode"]
    fields = ["objective", "logdet_qstar", "logdet_s", "logdet_qprior", "logdet_sprior", "xqx", "loglik"]
    return {**{f: _column(rows, f) for f in fields}, "info": None, "mode": [r["mode"] for r in rows]}
