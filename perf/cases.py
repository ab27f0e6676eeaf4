"""Workloads of the SMC sweep for timing: whole short runs of the tracking
filter and of the tempered mixture sampler, the one-shot resampling, the
mixture likelihood with its gradient and a mixed batch, through the package's
public entry points.

Sizes follow the framework's own workloads (the 1000-particle filter over 100
observations, the 2^22-particle filter, the four-component mixture with 1000
data points and 2^14 particles, the six-component one with 10^4 points, 2^16
particles and MALA moves, the mixed batch of filters and samplers) and the
ranges between them.  A run here has fewer steps than a full analysis; every
pass starts from the prior draws, so a pass on the same state repeats the same
numbers.

listed() / draw(rng): the cases; prepare(case, seed): inputs and the handle a
program keeps; run(state): one pass; work(case): the bytes and operations the
pass cannot do without; exact(case, seed): the outputs in 64-bit torch,
independent of the package's kernels.
"""
import math

import numpy as np
import torch

from paper_1306_5583_amd import (BatchRunner, GmmSampler, GmmSpec, ParticleFilter, PfSpec,
                                 gmm_loglik)
from paper_1306_5583_amd import _lib as L

DEV = "cuda"
SCHEMES = ("systematic", "stratified", "multinomial")


# ------------------------------------------------------------------ cases ---

def _filter(name, n, steps, scheme="systematic", fp32=False):
    return {"name": name, "kind": "filter", "n": n, "steps": steps, "scheme": scheme,
            "fp32": fp32}


def _sampler(name, n, K, nd, steps, move, scheme="systematic"):
    return {"name": name, "kind": "sampler", "n": n, "K": K, "n_data": nd, "steps": steps,
            "move": move, "scheme": scheme}


def _loglik(name, n, K, nd, grad=True):
    return {"name": name, "kind": "loglik", "n": n, "K": K, "n_data": nd, "grad": grad}


def _resample(name, n, scheme, zeros=0.0):
    return {"name": name, "kind": "resample", "n": n, "scheme": scheme, "zeros": zeros}


def _batch(name, filters, samplers, steps, shape_seed):
    return {"name": name, "kind": "batch", "filters": filters, "samplers": samplers,
            "steps": steps, "shape_seed": shape_seed}


def listed():
    return [
        # one object tracked online over a hundred observations by a small filter
        _filter("filter-1k", 1000, 100),
        # an ordinary filter, ragged population
        _filter("filter-70k", 70001, 20),
        # the largest filter: the data-parallel sweep proper, its FP32-state
        # option, and the other resampling scheme it is run with
        _filter("filter-4m", 1 << 22, 8),
        _filter("filter-4m-fp32", 1 << 22, 8, fp32=True),
        _filter("filter-1m-multinomial", 1 << 20, 8, scheme="multinomial"),
        # a caller's own small population resampled in one call
        _resample("resample-1k", 1000, "systematic"),
        # value and gradient of the mixture log-likelihood through autograd:
        # a handful of parameter vectors, and a whole population
        _loglik("loglik-200", 200, 4, 1000),
        _loglik("loglik-16k", 1 << 14, 6, 10000),
        # the tempered sampler: a small population, the four-component
        # example, and the large six-component one with MALA moves
        _sampler("sampler-rw-1k", 1000, 4, 1000, 20, "rw"),
        _sampler("sampler-rw-16k", 1 << 14, 4, 1000, 10, "rw"),
        _sampler("sampler-mala-64k", 1 << 16, 6, 10000, 4, "mala"),
        # many filters and samplers of uneven sizes advanced together
        _batch("batch-16", 12, 4, 5, 5583),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["filter", "filter", "resample", "loglik", "sampler", "sampler", "batch"])
    if kind == "filter":
        n = _log_int(rng, 128, 1 << 22)
        c = _filter("", n, rng.randint(3, 8) if n > 1 << 18 else rng.randint(8, 40),
                    scheme=rng.choice(SCHEMES), fp32=rng.random() < 0.25)
    elif kind == "resample":
        c = _resample("", _log_int(rng, 64, 1 << 22), rng.choice(SCHEMES),
                      zeros=rng.choice([0.0, 0.0, 0.3]))
    elif kind == "loglik":
        K, nd = rng.randint(1, 8), _log_int(rng, 100, 20000)
        n = _log_int(rng, 32, min(1 << 16, int(2e9 / (K * nd))))
        c = _loglik("", n, K, nd, grad=rng.random() < 0.7)
    elif kind == "sampler":
        K, nd = rng.randint(2, 8), _log_int(rng, 500, 20000)
        steps = rng.randint(4, 12)
        n = _log_int(rng, 64, min(1 << 16, int(4e10 / (3 * steps * K * nd))))
        c = _sampler("", n, K, nd, steps, rng.choice(["rw", "mala"]),
                     scheme=rng.choice(SCHEMES))
    else:
        c = _batch("", rng.randint(2, 14), rng.randint(1, 5), rng.randint(3, 8),
                   rng.randrange(1 << 30))
    del c["name"]
    return c


# ----------------------------------------------------------------- inputs ---

def _track(T, seed):
    """Observations of a constant-velocity trajectory with Student-t noise."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(4)
    y = np.empty((T, 2))
    for t in range(T):
        if t:
            e = rng.standard_normal(4)
            x = np.array([x[0] + 0.1 * x[2] + 0.02 * e[0], x[1] + 0.1 * x[3] + 0.02 * e[1],
                          x[2] + 0.5 * e[2], x[3] + 0.5 * e[3]])
        y[t] = x[:2] + 0.1 * rng.standard_t(10.0, 2)
    return y


def _mixture(nd, K, seed):
    """nd points of a K-component mixture (the paper's four components, else
    means evenly spaced in [-5, 5] with Dirichlet(2) weights)."""
    rng = np.random.default_rng(seed)
    if K == 4:
        means, prec, w = np.array([-3.0, 0.0, 3.0, 6.0]), 2.0, np.full(4, 0.25)
    else:
        means = np.linspace(-5.0, 5.0, K) if K > 1 else np.zeros(1)
        prec, w = 1.5, rng.dirichlet(np.full(K, 2.0))
    return means[rng.choice(K, size=nd, p=w)] + rng.standard_normal(nd) / math.sqrt(prec)


def _alphas(steps):
    return (np.arange(steps + 1) / steps) ** 4


def _weights(case, seed):
    """Unnormalised log-weights far from zero, some particles dead."""
    rng = np.random.default_rng(seed)
    lw = rng.normal(0.0, 2.0, case["n"]) - 700.0
    if case["zeros"]:
        lw[rng.random(case["n"]) < case["zeros"]] = -np.inf
        lw[0] = -700.0
    return lw


def _params(case, seed):
    """Parameter vectors around the data's own mixture."""
    rng = np.random.default_rng(seed + 1)
    K, n = case["K"], case["n"]
    means = np.array([-3.0, 0.0, 3.0, 6.0]) if K == 4 else np.linspace(-5.0, 5.0, K)
    mu = means[:, None] + rng.normal(0.0, 0.7, (K, n))
    return (mu, rng.normal(0.4, 0.5, (K, n)), rng.normal(0.0, 0.5, (K - 1, n)),
            rng.normal(1.0, 0.3, n))


def _batch_shapes(case):
    """Uneven sizes: filters of 2^10..2^18 particles, samplers of 2^10..2^14
    with 2..8 components and 500..5000 data points (log-uniform)."""
    rng = np.random.default_rng(case["shape_seed"])
    out = []
    for p in range(case["filters"]):
        out.append(("filter", int(2.0 ** rng.uniform(10, 18)),
                    "stratified" if p % 4 == 3 else "systematic"))
    for q in range(case["samplers"]):
        out.append(("sampler", int(2.0 ** rng.uniform(10, 14)), int(rng.integers(2, 9)),
                    int(math.exp(rng.uniform(math.log(500), math.log(5000)))),
                    "rw" if q % 4 == 3 else "mala"))
    return out


def _batch_specs(case, seed):
    specs = []
    for p, sh in enumerate(_batch_shapes(case)):
        if sh[0] == "filter":
            specs.append(PfSpec(n=sh[1], y=_track(case["steps"] + 1, seed + p), seed=seed + p,
                                problem_id=p, scheme=sh[2]))
        else:
            specs.append(GmmSpec(n=sh[1], y=_mixture(sh[3], sh[2], seed + p), K=sh[2],
                                 alphas=_alphas(case["steps"]), move=sh[4], seed=seed + p,
                                 problem_id=p))
    return specs


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "filter":
        s["pf"] = ParticleFilter(case["n"], _track(case["steps"] + 1, seed), seed=seed,
                                 scheme=case["scheme"], fp32_state=case["fp32"], device=DEV)
    elif kind == "sampler":
        s["gm"] = GmmSampler(case["n"], _mixture(case["n_data"], case["K"], seed), case["K"],
                             case["steps"], seed=seed, move=case["move"],
                             scheme=case["scheme"], device=DEV)
        s["alphas"] = _alphas(case["steps"])
    elif kind == "resample":
        n, code = case["n"], L.SCHEMES[case["scheme"]]
        s["lw"] = torch.as_tensor(_weights(case, seed), device=DEV)
        s["anc"] = torch.zeros(n, dtype=torch.int32, device=DEV)
        s["summary"] = torch.zeros(5, dtype=torch.float64, device=DEV)
        s["bytes"] = L.smc_resample_weights_workspace(n, code)
        s["ws"] = torch.empty(s["bytes"], dtype=torch.uint8, device=DEV)
        s["seed"] = seed
    elif kind == "loglik":
        mu, eta, z, w = _params(case, seed)
        s["y"] = torch.as_tensor(_mixture(case["n_data"], case["K"], seed), device=DEV)
        s["par"] = [torch.as_tensor(v, device=DEV) for v in (mu, eta, z)]
        if case["grad"]:
            for v in s["par"][:3 if case["K"] > 1 else 2]:
                v.requires_grad_(True)
        s["w"] = torch.as_tensor(w, device=DEV)
    else:
        s["runner"] = BatchRunner(_batch_specs(case, seed), device=DEV)
    return s


# ------------------------------------------------------------------- pass ---

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "filter":
        pf = s["pf"]
        log_z = pf.run()
        return {"log_z": log_z, "state": pf.state(), "history": pf.history,
                "ancestors": pf.ancestors}
    if kind == "sampler":
        gm = s["gm"]
        log_z = gm.run(s["alphas"])
        return {"log_z": log_z, "state": gm.state(), "history": gm.history,
                "ancestors": gm.ancestors}
    if kind == "resample":
        L.smc_resample_weights(s["lw"].data_ptr(), case["n"], L.SCHEMES[case["scheme"]], 0.5, 1,
                               s["seed"], 3, 0, s["anc"].data_ptr(), s["summary"].data_ptr(),
                               s["ws"].data_ptr(), s["bytes"],
                               torch.cuda.current_stream().cuda_stream)
        return {"ancestors": s["anc"], "summary": s["summary"]}
    if kind == "loglik":
        ll = gmm_loglik(*s["par"], s["y"])
        if not case["grad"]:
            return {"loglik": ll}
        grads = torch.autograd.grad(ll, s["par"][:3 if case["K"] > 1 else 2], s["w"])
        return {"loglik": ll, "grads": list(grads)}
    r = s["runner"]
    r.run(case["steps"])
    return [{"history": r.bufs[i].history, "state": r.state(i), "ancestors": r.bufs[i].ancestors}
            for i in range(len(r.specs))]


# ------------------------------------------------------------------- work ---

def _filter_work(n, steps, elem):
    # prior draws written with their weights; per step the state in and out,
    # the log-weight in and out and the ancestors out.  About 200 FP64
    # operations a particle: four normals, transition, density, weight
    return {"bytes": n * ((4 * elem + 8 + 4) + steps * (8 * elem + 16 + 4)),
            "flops": 200.0 * n * (steps + 1)}


def _sampler_work(n, K, nd, steps, mala):
    rows = 6 * K if mala else 3 * K + 1
    # a mixture term: distance, square, exponential (about 20 operations),
    # sum; with the gradient about 6 more
    terms = float(n) * nd * K * (1 + (3 if K > 1 else 2) * steps)
    return {"bytes": n * (8 * rows + steps * (16 * rows + 24 + 4)),
            "flops": terms * (32 if mala else 26)}


def work(case):
    kind = case["kind"]
    if kind == "filter":
        return _filter_work(case["n"], case["steps"], 4 if case["fp32"] else 8)
    if kind == "sampler":
        return _sampler_work(case["n"], case["K"], case["n_data"], case["steps"],
                             case["move"] == "mala")
    if kind == "resample":
        return {"bytes": 12 * case["n"] + 40, "flops": 30.0 * case["n"]}
    if kind == "loglik":
        D = 3 * case["K"] - 1
        g = case["grad"]
        return {"bytes": 8 * case["n"] * (D * (2 if g else 1) + 1 + (1 if g else 0)) +
                8 * case["n_data"],
                "flops": float(case["n"]) * case["n_data"] * case["K"] * (32 if g else 26)}
    b = f = 0.0
    for sh in _batch_shapes(case):
        w = _filter_work(sh[1], case["steps"], 8) if sh[0] == "filter" else \
            _sampler_work(sh[1], sh[2], sh[3], case["steps"], sh[4] == "mala")
        b, f = b + w["bytes"], f + w["flops"]
    return {"bytes": b, "flops": f}


# ------------------------------------------------------- 64-bit reference ---

def _words(seed, i, t, tag, call, p=0):
    """Philox4x32-10 (Salmon et al. 2011) at counters (i, t, tag<<16|call, p)."""
    m = 0xFFFFFFFF
    c = [i & m, torch.full_like(i, t), torch.full_like(i, tag << 16 | call),
         torch.full_like(i, p)]
    k0, k1 = seed & m, (seed >> 32) & m
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & m) ^ c[1] ^ k0, p1 & m, ((p0 >> 32) & m) ^ c[3] ^ k1, p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c


def _u53(a, b):
    return a.double() * 2.0 ** -32 + ((b >> 11) + 1).double() * 2.0 ** -53


def _unif(seed, i, t, tag, call, p=0):
    w = _words(seed, i, t, tag, call, p)
    return _u53(w[0], w[1])


def _normal2(seed, i, t, tag, call, p=0):
    w = _words(seed, i, t, tag, call, p)
    r = torch.sqrt(-2.0 * torch.log(_u53(w[0], w[1])))
    a = 2.0 * math.pi * _u53(w[2], w[3])
    return r * torch.cos(a), r * torch.sin(a)


class _Weights:
    """Normalisation, decision and resampling shared by both references."""

    def __init__(self, n, seed, p, scheme, steps):
        self.n, self.seed, self.p, self.scheme = n, seed, p, scheme
        self.i = torch.arange(n, dtype=torch.int64, device=DEV)
        self.hist = torch.zeros((steps, L.SMC_HIST_COLS), dtype=torch.float64, device=DEV)
        self.lw = torch.zeros(n, dtype=torch.float64, device=DEV)
        self.Lprev, self.logz, self.resampled = math.log(n), 0.0, False

    def normalise(self, t):
        L1 = float(torch.logsumexp(self.lw, 0))
        ess = math.exp(2.0 * L1 - float(torch.logsumexp(2.0 * self.lw, 0)))
        d = L1 - self.Lprev
        self.logz += d
        self.Lprev = L1
        self.flag = ess < 0.5 * self.n
        self.hist[t, :5] = torch.tensor([ess, float(self.flag), d, self.logz, L1],
                                        dtype=torch.float64)

    def resample(self, t):
        """Ancestors, or None when the decision is not to resample."""
        self.resampled = self.flag
        if not self.flag:
            return None
        n = self.n
        S = torch.cumsum(torch.exp(self.lw - self.lw.max()), 0)
        if self.scheme == "systematic":
            u = (self.i.double() + _unif(self.seed, self.i[:1], t, 7, 0, self.p)) / n
        elif self.scheme == "stratified":
            u = (self.i + _unif(self.seed, self.i, t, 7, 0, self.p)) / n
        else:
            k = torch.arange(n + 1, dtype=torch.int64, device=DEV)
            G = torch.cumsum(-torch.log(_unif(self.seed, k, t, 7, 1, self.p)), 0)
            u = G[:-1] / G[-1]
        self.Lprev = math.log(n)
        last = int(torch.nonzero(self.lw > -math.inf)[-1])
        return torch.searchsorted(S, u * S[-1], right=True).clamp(max=last)

    def weights(self):
        return torch.ones_like(self.lw) if self.resampled else torch.exp(self.lw - self.lw.max())


def _exact_filter(n, y, seed, scheme, p=0, last_monitor=True):
    W = _Weights(n, seed, p, scheme, len(y))
    nu, sc = 10.0, 0.1
    const = 2.0 * (math.lgamma(0.5 * (nu + 1)) - math.lgamma(0.5 * nu) -
                   0.5 * math.log(nu * math.pi) - math.log(sc))

    def density(x, t):
        r0, r1 = (y[t, 0] - x[0]) / sc, (y[t, 1] - x[1]) / sc
        return const - 0.5 * (nu + 1) * (torch.log1p(r0 * r0 / nu) + torch.log1p(r1 * r1 / nu))

    x = torch.stack(_normal2(seed, W.i, 0, 1, 0, p) + _normal2(seed, W.i, 0, 1, 1, p))
    W.lw = density(x, 0)
    for t in range(len(y)):
        if t:
            a = _normal2(seed, W.i, t, 2, 0, p)
            b = _normal2(seed, W.i, t, 2, 1, p)
            x = torch.stack([x[0] + 0.1 * x[2] + 0.02 * a[0], x[1] + 0.1 * x[3] + 0.02 * a[1],
                             x[2] + 0.5 * b[0], x[3] + 0.5 * b[1]])
            W.lw = (torch.zeros_like(W.lw) if W.resampled else W.lw) + density(x, t)
        W.normalise(t)
        raw = x
        anc = W.resample(t)
        if anc is not None:
            x = x[:, anc]
        if last_monitor or t + 1 < len(y):
            w = W.weights()
            W.hist[t, 9:13] = (x * w).sum(1) / w.sum()
    return {"log_z": W.logz, "state": raw, "history": W.hist, "ancestors": None}


def _mix_loglik(phi, K, y, grad):
    """Log-likelihood of parameter columns phi[3K-1][n], and its gradient."""
    n = phi.shape[1]
    mu, eta = phi[:K], phi[K:2 * K]
    zz = torch.cat([phi[2 * K:], torch.zeros((1, n), dtype=phi.dtype, device=phi.device)])
    logw = torch.log_softmax(zz, 0)
    c, lam = logw + 0.5 * eta - 0.5 * math.log(2.0 * math.pi), torch.exp(eta)
    ll = torch.zeros(n, dtype=phi.dtype, device=phi.device)
    g = torch.zeros_like(phi) if grad else None
    step = max(1, int(2e8 // (8 * K * n)))
    for k in range(0, len(y), step):
        d = y[None, None, k:k + step] - mu[:, :, None]
        e = c[:, :, None] - 0.5 * lam[:, :, None] * d * d
        lse = torch.logsumexp(e, 0)
        ll += lse.sum(1)
        if grad:
            r = torch.exp(e - lse)
            g[:K] += (r * lam[:, :, None] * d).sum(2)
            g[K:2 * K] += (r * (0.5 - 0.5 * lam[:, :, None] * d * d)).sum(2)
            if K > 1:
                g[2 * K:] += r.sum(2)[:K - 1]
    if grad and K > 1:
        g[2 * K:] -= len(y) * torch.exp(logw[:K - 1])
    return ll, g, logw


def _log_prior(phi, K, logw):
    a = (-phi[:K] ** 2 / 200.0).sum(0) + (phi[K:2 * K] - torch.exp(phi[K:2 * K])).sum(0)
    return a + logw.sum(0) if K > 1 else a


def _prior_grad(phi, K, logw):
    return torch.cat([-phi[:K] / 100.0, 1.0 - torch.exp(phi[K:2 * K]),
                      1.0 - K * torch.exp(logw[:K - 1])])


def _exact_sampler(n, y, K, seed, move, alphas, scheme, p=0):
    mala = move == "mala"
    y = torch.as_tensor(y, device=DEV)
    W = _Weights(n, seed, p, scheme, len(alphas))
    mu = []
    for j in range(0, K, 2):
        mu += list(_normal2(seed, W.i, 0, 1, j // 2, p))
    mu = [10.0 * m for m in mu[:K]]
    eta = [torch.log(-torch.log(_unif(seed, W.i, 0, 1, 64 + 64 * j, p))) for j in range(K)]
    h = [torch.log(-torch.log(_unif(seed, W.i, 0, 1, 64 + 1024 + 64 * j, p))) for j in range(K)]
    phi = torch.stack(mu + eta + [v - h[-1] for v in h[:-1]])
    ll, g, logw = _mix_loglik(phi, K, y, mala)
    lp = _log_prior(phi, K, logw)
    W.normalise(0)
    W.hist[0, 8] = U = float(ll.mean())
    ps, a0 = 0.0, 0.0
    for t in range(1, len(alphas)):
        a = float(alphas[t])
        W.lw = (torch.zeros_like(W.lw) if W.resampled else W.lw) + (a - a0) * ll
        W.normalise(t)
        anc = W.resample(t)
        if anc is not None:
            phi, ll, lp = phi[:, anc], ll[anc], lp[anc]
            g = g[:, anc] if mala else None
        b = max(a, 0.02)
        scales = (0.15 / b, 0.15 * (1 + math.sqrt(1 / b)), 0.2 * (1 + math.sqrt(1 / b)))
        for blk in range(3 if K > 1 else 2):
            s = 0.05 * scales[blk] / 0.15 if mala else scales[blk]
            rows = range(blk * K, blk * K + (K if blk < 2 else K - 1))
            xi = []
            for m in range(0, len(rows), 2):
                xi += list(_normal2(seed, W.i, t, 3 + blk, m // 2, p))
            new = phi.clone()
            sl = slice(rows[0], rows[-1] + 1)
            step = s * torch.stack(xi[:len(rows)])
            drift = 0.0
            if mala:
                logw0 = _mix_weights(phi, K)
                drift = 0.5 * s * s * (_prior_grad(phi, K, logw0)[sl] + a * g[sl])
            new[sl] = phi[sl] + drift + step
            ll1, g1, logw1 = _mix_loglik(new, K, y, mala)
            lp1 = _log_prior(new, K, logw1)
            logr = lp1 + a * ll1 - (lp + a * ll)
            if mala:
                back = 0.5 * s * s * (_prior_grad(new, K, logw1)[sl] + a * g1[sl])
                fwd = ((new[sl] - phi[sl] - drift) ** 2).sum(0)
                bwd = ((phi[sl] - new[sl] - back) ** 2).sum(0)
                logr = logr + (fwd - bwd) / (2.0 * s * s)
            ok = torch.log(_unif(seed, W.i, t, 6, blk, p)) <= logr
            W.hist[t, 5 + blk] = float(ok.sum())
            phi, ll, lp = torch.where(ok, new, phi), torch.where(ok, ll1, ll), \
                torch.where(ok, lp1, lp)
            g = torch.where(ok, g1, g) if mala else None
        w = W.weights()
        U1 = float((w * ll).sum() / w.sum())
        ps += 0.5 * (a - a0) * (U1 + U)
        W.hist[t, 8], W.hist[t, 13] = U1, ps
        U, a0 = U1, a
    rows = [phi, ll[None], lp[None]] + ([g] if mala else [])
    return {"log_z": W.logz, "state": torch.cat(rows), "history": W.hist, "ancestors": None}


def _mix_weights(phi, K):
    zz = torch.cat([phi[2 * K:], torch.zeros((1, phi.shape[1]), dtype=phi.dtype,
                                             device=phi.device)])
    return torch.log_softmax(zz, 0)


def exact(case, seed):
    kind = case["kind"]
    if kind == "filter":
        if case["fp32"]:
            return None  # single-precision draws are part of what this option computes
        return _exact_filter(case["n"], _track(case["steps"] + 1, seed), seed, case["scheme"])
    if kind == "sampler":
        if _sampler_work(case["n"], case["K"], case["n_data"], case["steps"],
                         False)["flops"] > 3e11:
            return None
        return _exact_sampler(case["n"], _mixture(case["n_data"], case["K"], seed), case["K"],
                              seed, case["move"], _alphas(case["steps"]), case["scheme"])
    if kind == "resample":
        lw = torch.as_tensor(_weights(case, seed), device=DEV)
        L1, L2 = torch.logsumexp(lw, 0), torch.logsumexp(2.0 * lw, 0)
        return {"ancestors": None,
                "summary": torch.stack([L1, L2, torch.exp(2.0 * L1 - L2), torch.ones_like(L1),
                                        torch.zeros_like(L1)])}
    if kind == "loglik":
        mu, eta, z, w = (torch.as_tensor(v, device=DEV) for v in _params(case, seed))
        K = case["K"]
        y = torch.as_tensor(_mixture(case["n_data"], K, seed), device=DEV)
        ll, g, _ = _mix_loglik(torch.cat([mu, eta, z]), K, y, case["grad"])
        if not case["grad"]:
            return {"loglik": ll}
        g = g * w
        return {"loglik": ll, "grads": [g[:K], g[K:2 * K]] + ([g[2 * K:]] if K > 1 else [])}
    out = []
    for p, sh in enumerate(_batch_shapes(case)):
        if sh[0] == "filter":
            r = _exact_filter(sh[1], _track(case["steps"] + 1, seed + p), seed + p, sh[2], p,
                              last_monitor=False)
        else:
            r = _exact_sampler(sh[1], _mixture(sh[3], sh[2], seed + p), sh[2], seed + p, sh[4],
                               _alphas(case["steps"]), "systematic", p)
        out.append({k: r[k] for k in ("history", "state", "ancestors")})
    return out
