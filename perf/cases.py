"""The work that programs built on this package do on the GPU, as cases whose time can be measured.

A case names a kind of call and its sizes:

    step      one optimisation step on a diagonal Hamiltonian: the refresh of the working weights that
              follows every update, then sampling, energies, statistics and gradient (binding.step);
    grad      log pi of given strings and its gradient through autograd (vqmc.log_prob);
    logprob   log pi of given strings alone (binding.logprob);
    evaluate  a fresh batch from the current model with its energies and their moments, as
              Trainer.evaluate takes them;
    sr        one stochastic-reconfiguration step without its update, as SRTrainer.step takes it:
              sampling with byproducts, energies, coefficients, the SR direction;
    tim       one optimisation step on a transverse-field Ising model (binding.step with a Tim).

Weights are drawn at the scale every training run starts from, U(+-1/sqrt(fan_in)); graphs and
couplings follow the recipes of paper_2106_13308_amd.inputs.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2106_13308_amd import binding as B
from paper_2106_13308_amd import inputs, vqmc

LAMBDA = 1e-3  # ridge of the SR direction (the package's default)


# ---------------------------------------------------------------- cases
def listed():
    return [
        # the smallest training run: a 20-site Max-Cut instance, latency and launches only
        dict(name="step_paper20", kind="step", n=20, h=45, B=1024, wdtype="f32", graph="paper"),
        # the largest of the small Max-Cut protocol: an ordinary training step in FP32
        dict(name="step_paper500", kind="step", n=500, h=193, B=1024, wdtype="f32", graph="paper"),
        # the benchmark workload: sparse Max-Cut on 10^4 sites
        dict(name="step_maxcut10k", kind="step", n=10000, h=1000, B=2048, wdtype="bf16", graph="regular10"),
        # a spin glass with dense couplings, wide model, large batch
        dict(name="step_sk2000", kind="step", n=2000, h=2000, B=8192, wdtype="bf16", graph="sk"),
        # scoring and differentiating given strings in a user's own loss, FP32
        dict(name="grad_f32", kind="grad", n=500, h=500, B=4096, wdtype="f32"),
        # the same in BF16 at sizes that fill no tile
        dict(name="grad_bf16_ragged", kind="grad", n=3001, h=611, B=1500, wdtype="bf16"),
        # scoring a large batch without a gradient
        dict(name="logprob_bf16", kind="logprob", n=10000, h=1000, B=2048, wdtype="bf16"),
        # scoring a few strings: the smallest call
        dict(name="logprob_small", kind="logprob", n=100, h=106, B=64, wdtype="f32"),
        # evaluation batch on a graph with real weights, odd site count
        dict(name="evaluate_f32", kind="evaluate", n=1001, h=239, B=1024, wdtype="f32", graph="er0.02"),
        # natural-gradient training at the protocol's size
        dict(name="sr_paper500", kind="sr", n=500, h=193, B=1024, wdtype="f32", graph="paper"),
        # natural-gradient training at the benchmark size
        dict(name="sr_maxcut10k", kind="sr", n=10000, h=1000, B=2048, wdtype="bf16", graph="regular10"),
        # transverse-field Ising training, off-diagonal local energy included
        dict(name="tim_1k", kind="tim", n=1000, h=239, B=512, wdtype="bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "sk", "grad", "grad", "logprob", "evaluate", "sr", "sr", "tim"])
    wdtype = rng.choice(["f32", "bf16"])
    if kind == "step":
        n, h, b = _log_uniform(rng, 20, 10000), _log_uniform(rng, 16, 2000), _log_uniform(rng, 64, 8192)
        b = max(64, min(b, int(2e10 / (n * h))))
        return dict(kind="step", n=n, h=h, B=b, wdtype=wdtype, graph="paper" if n <= 600 else "regular10")
    if kind == "sk":
        n, h, b = _log_uniform(rng, 64, 2000), _log_uniform(rng, 32, 2000), _log_uniform(rng, 64, 8192)
        return dict(kind="step", n=n, h=h, B=b, wdtype=wdtype if n * h * b < 1e10 else "bf16", graph="sk")
    if kind == "grad":
        n, h, b = _log_uniform(rng, 20, 5000), _log_uniform(rng, 16, 2000), _log_uniform(rng, 64, 8192)
        b = max(64, min(b, int((1e10 if wdtype == "bf16" else 4e9) / (n * h))))
        return dict(kind="grad", n=n, h=h, B=b, wdtype=wdtype)
    if kind == "logprob":
        n, h, b = _log_uniform(rng, 20, 10000), _log_uniform(rng, 16, 2000), _log_uniform(rng, 16, 8192)
        b = max(16, min(b, int((2e10 if wdtype == "bf16" else 8e9) / (n * h))))
        return dict(kind="logprob", n=n, h=h, B=b, wdtype=wdtype)
    if kind == "evaluate":
        n, h, b = _log_uniform(rng, 50, 2000), _log_uniform(rng, 32, 600), _log_uniform(rng, 256, 4096)
        return dict(kind="evaluate", n=n, h=h, B=b, wdtype=wdtype, graph=rng.choice(["er0.02", "er0.25"]))
    if kind == "sr":
        n, h, b = _log_uniform(rng, 20, 10000), _log_uniform(rng, 32, 1000), _log_uniform(rng, 100, 2048)
        if wdtype == "f32":
            n = min(n, 3000)
        return dict(kind="sr", n=n, h=h, B=b, wdtype=wdtype, graph="paper" if n <= 600 else "regular10")
    n, h, b = _log_uniform(rng, 20, 1000), _log_uniform(rng, 32, 239), _log_uniform(rng, 64, 512)
    return dict(kind="tim", n=n, h=h, B=b, wdtype=wdtype)


# ---------------------------------------------------------------- inputs
def _counts(n, h):
    """c[d] = number of hidden units with degree <= d (0-based site d), as an int32 array."""
    return np.searchsorted(inputs.made_degrees(n, h), np.arange(n), side="right").astype(np.int32)


def _weights(case, seed):
    """Packed FP32 parameters on the GPU: P (n x h), b1, b2, c."""
    n, h = case["n"], case["h"]
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)
    r1, r2 = 1.0 / math.sqrt(n), 1.0 / math.sqrt(h)
    c = torch.from_numpy(_counts(n, h)).cuda()
    lower = torch.arange(h, device="cuda")[None, :] < c[:, None]
    P = (2 * torch.rand(n, h, generator=g, device="cuda") - 1) * torch.where(lower, r2, r1)
    b1 = (2 * torch.rand(h, generator=g, device="cuda") - 1) * r1
    b2 = (2 * torch.rand(n, generator=g, device="cuda") - 1) * r2
    return P.contiguous(), b1, b2, c


def _edges(case, seed):
    n, graph = case["n"], case["graph"]
    if graph == "paper":
        e = inputs.paper_maxcut_graph(n, seed)
    elif graph == "regular10":
        e = inputs.random_regular_graph(n, 10, seed)
    else:
        e = inputs.erdos_renyi_graph(n, float(graph[2:]), seed)
    if case["kind"] == "evaluate":  # real weights
        w = np.random.default_rng(seed + 1).uniform(0.1, 1.0, len(e)).astype(np.float32)
    elif graph == "regular10":
        w = inputs.integer_weights(len(e), 1, 5, seed + 1)
    else:
        w = inputs.unit_weights(len(e))
    return e, w


def _symmetric(n, seed, normal):
    """Dense couplings, symmetric with a zero diagonal: N(0, 1/n) or U(-1, 1), FP32 on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 29)
    if normal:
        J = torch.randn(n, n, generator=g, device="cuda") / math.sqrt(n)
    else:
        J = 2 * torch.rand(n, n, generator=g, device="cuda") - 1
    J = torch.triu(J, 1)
    return J + J.T


def _tim_fields(n, seed):
    rng = np.random.default_rng(seed + 3)
    return rng.uniform(0, 1, n).astype(np.float32), rng.uniform(-1, 1, n).astype(np.float32)


def _strings(case, seed):
    """Given strings (B x ld(n) int8, zero padding) and a coefficient for each."""
    n, b = case["n"], case["B"]
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 41)
    S = torch.zeros(b, (n + 63) // 64 * 64, dtype=torch.int8, device="cuda")
    S[:, :n] = 2 * torch.randint(0, 2, (b, n), generator=g, device="cuda", dtype=torch.int8) - 1
    return S, torch.randn(b, generator=g, device="cuda") / b


def prepare(case, seed):
    P, b1, b2, c = _weights(case, seed)
    made = B.Made(case["n"], case["h"], P, b1, b2, c, B.BF16 if case["wdtype"] == "bf16" else B.F32)
    st = dict(kind=case["kind"], made=made, B=case["B"], seed=seed % (1 << 31), t=seed % 1000)
    if case["kind"] in ("grad", "logprob"):
        st["S"], st["coef"] = _strings(case, seed)
        if case["kind"] == "grad":
            st["params"] = [p.requires_grad_(True) for p in (made.P32, made.b1, made.b2)]
        else:
            st["ws"] = B.workspace(B.WS_LOGPROB, made, case["B"])
        return st
    if case["kind"] == "tim":
        alpha, beta = _tim_fields(case["n"], seed)
        st["H"] = B.Tim(alpha, beta, _symmetric(case["n"], seed, False).cpu().numpy())
    elif case["graph"] == "sk":
        st["H"] = B.Hamiltonian(case["n"], B.H_DENSE_F32, J=_symmetric(case["n"], seed, True).contiguous())
    else:
        st["H"] = B.Hamiltonian.from_edges(case["n"], *_edges(case, seed))
    if case["kind"] in ("step", "tim"):
        st["bufs"] = B.StepBuffers.allocate(made, st["H"], case["B"])
    elif case["kind"] == "sr":
        st["ws"] = B.workspace(B.WS_SR_DIRECTION, made, case["B"])
    return st


# ---------------------------------------------------------------- one pass
def _moments(stats):
    """The vqmc_stats record as plain numbers: mean, variance, minimum; the minimum's index; the sum."""
    f, i = stats.view(torch.float64), stats.view(torch.int64)
    return {"mean_var_min": f[:3], "argmin": i[3:4], "sum": f[4:5]}


def run(st):
    made, kind, b = st["made"], st["kind"], st["B"]
    if kind in ("step", "tim"):
        made.refresh()
        f = B.step(made, st["H"], b, st["seed"], st["t"], st["bufs"])
        return {"S": f.S, "logp": f.logp, "E": f.E, "stats": _moments(f.stats), "coef": f.coef, "dP": f.dP,
                "db1": f.db1, "db2": f.db2}
    if kind == "grad":
        lp = vqmc.log_prob(made, st["S"])
        dP, db1, db2 = torch.autograd.grad(lp, st["params"], grad_outputs=st["coef"])
        return {"logp": lp, "dP": dP, "db1": db1, "db2": db2}
    if kind == "logprob":
        return {"logp": B.logprob(made, st["S"], ws=st["ws"])}
    if kind == "evaluate":
        S, _ = B.sample(made, b, st["seed"], st["t"], tag=B.TAG_EVAL, want_logp=False)
        E = B.energy(st["H"], S, b)
        stats, _ = B.batch_stats(E, want_coef=False)
        return {"S": S, "E": E, "stats": _moments(stats)}
    made.refresh()
    S, logp, Zs, Rt = B.sample_fwd(made, b, st["seed"], st["t"])
    E = B.energy(st["H"], S, b)
    stats, coef = B.batch_stats(E)
    xP, xb1, xb2 = vqmc.sr_direction(made, S, coef, LAMBDA, b, Zs=Zs, Rt=Rt, ws=st["ws"])
    return {"S": S, "logp": logp, "E": E, "stats": _moments(stats), "coef": coef, "xP": xP, "xb1": xb1, "xb2": xb2}


def work(case):
    n, h, b, kind = case["n"], case["h"], case["B"], case["kind"]
    nhb = float(n) * h * b
    params, spins = 4.0 * n * h + 4.0 * (n + h), float(b) * n
    # each unmasked weight meets each sample once in a forward pass (half of them in either layer)
    if kind == "logprob":
        return {"bytes": (2.0 if case["wdtype"] == "bf16" else 4.0) * n * h + spins + 4 * b, "flops": 2 * nhb}
    if kind == "grad":
        return {"bytes": (2.0 if case["wdtype"] == "bf16" else 4.0) * n * h + params + spins + 8 * b, "flops": 5 * nhb}
    if kind == "tim":
        # single-flip differences: sum over i < d of the units between, n^2 h / 6 of them
        return {"bytes": 2 * params + 2.0 * n * n + spins, "flops": 5 * nhb + b * (float(n) * n * h / 3 + float(n) * n)}
    graph = case["graph"]
    pairs = n * (n - 1) / 2 * {"sk": 1.0, "paper": 0.25, "er0.02": 0.02, "er0.25": 0.25}.get(graph, 0.0) + (5.0 * n if graph == "regular10" else 0.0)
    coupling = (4.0 if graph == "sk" else 8.0) * pairs
    if kind == "evaluate":
        return {"bytes": params + coupling + spins + 8 * b, "flops": 2 * nhb + 2 * pairs * b}
    flops = 5 * nhb + 2 * pairs * b
    if kind == "sr":
        flops += 5.0 * (n + h) * b * (b + 1) / 2 + b ** 3 / 3.0
    return {"bytes": 2 * params + coupling + spins + 16 * b, "flops": flops}


# ---------------------------------------------------------------- the same in 64 bits
def _mulhilo(a, x):
    t = a * (x & 0xFFFF)
    hi = a * (x >> 16) + (t >> 16)
    return hi >> 16, ((hi & 0xFFFF) << 16) | (t & 0xFFFF)


def _uniforms(seed, step, tag, samples, blk):
    """Philox4x32-10 (Salmon et al., SC'11) uniforms of sites 4 blk .. 4 blk + 3, one row per sample."""
    x = [torch.full_like(samples, blk), samples & 0xFFFFFFFF, torch.full_like(samples, step), torch.full_like(samples, tag)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, x[0])
        h1, l1 = _mulhilo(0xCD9E8D57, x[2])
        x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return torch.stack([(v >> 8).double() * 2.0 ** -24 for v in x], 1)


class _Model:
    """The MADE in float64, on the working weights as the package rounds them."""

    def __init__(self, case, seed):
        P, b1, b2, c = _weights(case, seed)
        self.P = (P.to(torch.bfloat16) if case["wdtype"] == "bf16" else P).double()
        self.b1, self.b2, self.c = b1.double(), b2.double(), c.cpu().numpy()
        self.low = torch.arange(case["h"], device="cuda")[None, :] < c[:, None]  # W2 side of P
        self.n, self.h = case["n"], case["h"]

    def sample(self, b, seed, step, tag):
        A = self.b1.repeat(b, 1)
        R = torch.zeros_like(A)
        s = torch.zeros(b, self.n, dtype=torch.float64, device="cuda")
        ids, done = torch.arange(b, device="cuda"), 0
        for d in range(self.n):
            k = int(self.c[d])
            if k > done:
                R[:, done:k] = A[:, done:k].clamp_min(0)
                done = k
            if d % 4 == 0:
                u = _uniforms(seed, step, tag, ids, d // 4)
            z = torch.mv(R[:, :k], self.P[d, :k]) + self.b2[d]
            s[:, d] = torch.where(u[:, d % 4] < torch.sigmoid(z), 1.0, -1.0)
            A[:, k:].addr_(s[:, d], self.P[d, k:])
        return s

    def forward(self, s):
        A = s @ torch.where(self.low, 0.0, self.P) + self.b1
        R = A.clamp_min(0)
        return A, R, R @ torch.where(self.low, self.P, 0.0).T + self.b2

    def logp(self, s):
        return torch.nn.functional.logsigmoid(s * self.forward(s)[2]).sum(1)

    def scores(self, s, coef):
        """relu(A), and the adjoints of the logits and of the pre-activations, each row times coef."""
        A, R, z = self.forward(s)
        G = coef[:, None] * s * torch.sigmoid(-s * z)
        D = (G @ torch.where(self.low, self.P, 0.0)) * (A > 0)
        return R, G, D

    def gradient(self, s, coef):
        R, G, D = self.scores(s, coef)
        return torch.where(self.low, G.T @ R, s.T @ D), D.sum(0), G.sum(0)

    def gram(self, s):
        """O O^T by runs of sites that share c: the two staircases advance together."""
        R, G, D = self.scores(s, torch.ones_like(s[:, 0]))
        F, Q = torch.ones(len(s), len(s), dtype=torch.float64, device="cuda"), None
        Q = F.clone()
        K = torch.zeros_like(F)
        starts = [0] + [d for d in range(1, self.n) if self.c[d] != self.c[d - 1]] + [self.n]
        unit = 0
        for i, e in zip(starts[:-1], starts[1:]):
            while unit < self.c[i]:  # sites with c <= unit have entered Q; units below c[i] enter F
                K.addcmul_(torch.outer(D[:, unit], D[:, unit]), Q)
                F.addr_(R[:, unit], R[:, unit])
                unit += 1
            K.addcmul_(G[:, i:e] @ G[:, i:e].T, F)
            Q += s[:, i:e] @ s[:, i:e].T
        while unit < self.h:
            K.addcmul_(torch.outer(D[:, unit], D[:, unit]), Q)
            unit += 1
        return K


def _energies(case, seed, s, model):
    n = case["n"]
    if case["kind"] == "tim":
        alpha, beta = (torch.from_numpy(x).cuda().double() for x in _tim_fields(n, seed))
        J = torch.triu(_symmetric(n, seed, False).double(), 1)
        A, _, z = model.forward(s)
        base = torch.nn.functional.logsigmoid(s * z).sum(1)
        W1, W2 = torch.where(model.low, 0.0, model.P), torch.where(model.low, model.P, 0.0)
        E = -(s @ beta) - ((s @ J) * s).sum(1)
        for i in range(n):
            f = s.clone()
            f[:, i] = -f[:, i]
            z = (A - 2 * s[:, i:i + 1] * W1[i]).clamp_min(0) @ W2.T + model.b2
            E -= alpha[i] * torch.exp((torch.nn.functional.logsigmoid(f * z).sum(1) - base) / 2)
        return E
    if case["graph"] == "sk":
        return ((s @ torch.triu(_symmetric(n, seed, True).double(), 1)) * s).sum(1)
    e, w = _edges(case, seed)
    e, w = torch.from_numpy(e.astype(np.int64)).cuda(), torch.from_numpy(np.asarray(w, np.float64)).cuda()
    E = torch.zeros(len(s), dtype=torch.float64, device="cuda")
    for p in range(0, len(w), 16384):
        q = slice(p, p + 16384)
        E += (s[:, e[q, 0]] * s[:, e[q, 1]]) @ w[q]
    return E


def exact(case, seed):
    model, kind = _Model(case, seed), case["kind"]
    if kind in ("grad", "logprob"):
        S, coef = _strings(case, seed)
        s = S[:, :case["n"]].double()
        if kind == "logprob":
            return {"logp": model.logp(s)}
        dP, db1, db2 = model.gradient(s, coef.double())
        return {"logp": model.logp(s), "dP": dP, "db1": db1, "db2": db2}
    s = model.sample(case["B"], seed % (1 << 31), seed % 1000, 1 if kind == "evaluate" else 0)
    E = _energies(case, seed, s, model)
    stats = {"mean_var_min": torch.stack([E.mean(), E.var(unbiased=False), E.min()]), "argmin": None, "sum": E.sum()[None]}
    e = E if kind in ("evaluate", "tim") or case["graph"] == "sk" else E.round().long()
    out = {"S": None, "E": e, "stats": stats}
    if kind == "evaluate":
        return out
    coef = (E - E.mean()) / case["B"]
    out |= {"logp": model.logp(s), "coef": coef}
    if kind == "sr":
        K = model.gram(s)
        K.diagonal().add_(LAMBDA * case["B"])
        y = torch.cholesky_solve((case["B"] * coef)[:, None], torch.linalg.cholesky(K))[:, 0]
        out["xP"], out["xb1"], out["xb2"] = model.gradient(s, y)
    else:
        out["dP"], out["db1"], out["db2"] = model.gradient(s, coef)
    return out
