"""The work that programs have this library do, as cases that can be timed.

Kinds of cases:
  sweep   a chain in mid-run advances some sweeps and its new draws are fetched
  batch   many chains on uneven designs advance together, draws fetched per chain
  shared  several chains on one bfloat16 design (the multi-chain pass)
  gram    X^T X of a design on the device through hsp_gram
  fit     a new design: sampler created, some sweeps, draws fetched, released

Sizes are those of this repository's workloads (synth/, bench.py, tests/) or
generic ones.  Chains start from a state such as a chain reaches after burn-in
(set_state, as a program that resumes a checkpoint does), drawn from the seed.
"""
import math

import numpy as np
import torch

from paper_1608_04329_amd import hsp

ROWS = 1 << 16  # rows per chunk of the float64 references


def listed():
    return [
        # the paper's smallest synthetic design: a few sweeps at a time for a
        # program that looks at every draw; bound by launches and latencies
        dict(name="sweep_f32_n1e3_p10", kind="sweep", xt="f32", N=1000, p=10, sweeps=8),
        # the paper's middle design
        dict(name="sweep_f32_n1e5_p100", kind="sweep", xt="f32", N=100_000, p=100, sweeps=8),
        # the headline design, 4 GB of X, in both storage types
        dict(name="sweep_f32_n1e6_p1000", kind="sweep", xt="f32", N=1_000_000, p=1000, sweeps=4),
        dict(name="sweep_bf16_n1e6_p1000", kind="sweep", xt="bf16", N=1_000_000, p=1000, sweeps=4),
        # rare events (mean of y 0.0048): many rows of few covariates
        dict(name="sweep_f32_rare_p141", kind="sweep", xt="f32", N=1_295_848, p=141, sweeps=4, ybar=0.0048),
        # many covariates: the factorisation outweighs the pass over X
        dict(name="sweep_f32_n2e5_p4096", kind="sweep", xt="f32", N=200_000, p=4096, sweeps=1),
        # ragged and wide in bfloat16, the larger end of p
        dict(name="sweep_bf16_n6e4_p7003", kind="sweep", xt="bf16", N=60_013, p=7003, sweeps=1),
        # uneven datasets advanced together (a study of many outcomes)
        dict(name="batch_f32_24uneven", kind="batch", xt="f32", datasets=24, n_min=10_000, n_max=200_000,
             p_min=50, p_max=500, sweeps=4),
        # chains on one design, for convergence diagnostics
        dict(name="shared_bf16_16chains", kind="shared", xt="bf16", N=250_000, p=1000, chains=16, sweeps=2),
        # the one-time product of the headline design, and a ragged strided one
        dict(name="gram_f32_n1e6_p1000", kind="gram", xt="f32", N=1_000_000, p=1000, ld=1000),
        dict(name="gram_bf16_n3e5_p777", kind="gram", xt="bf16", N=300_007, p=777, ld=784),
        # a new ragged design from start to end, lambda recorded
        dict(name="fit_f32_n5e4_p333", kind="fit", xt="f32", N=50_003, p=333, sweeps=8, lam=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "mid", "mid", "wide", "batch", "shared", "gram", "fit"])
    xt = rng.choice(["f32", "bf16"])
    if kind == "small":
        return dict(kind="sweep", xt=xt, N=_log(rng, 500, 100_000), p=_log(rng, 2, 128), sweeps=rng.randint(2, 8))
    if kind == "mid":
        p = _log(rng, 100, 1536)
        return dict(kind="sweep", xt=xt, N=_log(rng, 20_000, min(1_300_000, 1_000_000_000 // p)), p=p,
                    sweeps=rng.randint(1, 4), lam=rng.random() < 0.3)
    if kind == "wide":
        p = _log(rng, 1537, 7000)
        return dict(kind="sweep", xt=xt, N=_log(rng, 5_000, min(200_000, 400_000_000 // p)), p=p, sweeps=1)
    if kind == "batch":
        return dict(kind="batch", xt=xt, datasets=rng.randint(4, 20), n_min=10_000, n_max=_log(rng, 20_000, 200_000),
                    p_min=rng.randint(10, 60), p_max=rng.randint(100, 500), sweeps=rng.randint(1, 4))
    if kind == "shared":
        return dict(kind="shared", xt="bf16", N=_log(rng, 30_000, 250_000), p=_log(rng, 64, 1000),
                    chains=rng.randint(2, 16), sweeps=rng.randint(1, 2))
    if kind == "gram":
        p = _log(rng, 10, 1000)
        return dict(kind="gram", xt=xt, N=_log(rng, 10_000, 1_000_000), p=p, ld=p + rng.randint(0, 9))
    return dict(kind="fit", xt=xt, N=_log(rng, 5_000, 50_000), p=_log(rng, 20, 333), sweeps=rng.randint(2, 8),
                lam=rng.random() < 0.5)


# ---- inputs ------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _design(N, p, seed, ybar=None):
    """X ~ N(0, 1) with an intercept column, sparse effects, probit outcomes."""
    r = np.random.default_rng([seed, N, p])
    k = min(10, p - 1)
    at = 1 + r.choice(p - 1, size=k, replace=False)
    beta = np.zeros(p)
    if ybar is None:
        beta[0] = r.uniform(-0.5, 0.5)
        beta[at] = r.uniform(-1.0, 1.0, k)
    else:
        beta[at] = r.uniform(-0.5, 0.5, k)
        from statistics import NormalDist
        beta[0] = NormalDist().inv_cdf(ybar) * math.sqrt(1.0 + float(np.sum(beta[1:] ** 2)))
    g = _generator(seed)
    X = torch.randn(N, p, generator=g, device="cuda")
    X[:, 0] = 1.0
    eps = torch.randn(N, generator=g, device="cuda", dtype=torch.float64)
    b = torch.from_numpy(beta).cuda()
    eta = torch.cat([X[i:i + ROWS].double() @ b for i in range(0, N, ROWS)])
    return X, (eta + eps > 0).to(torch.uint8), beta


def _state(beta, N, seed):
    """A chain's state after burn-in: beta near its truth, its horseshoe scales."""
    r = np.random.default_rng([seed, beta.size, 5])
    p = beta.size
    tau = max(1e-3, np.count_nonzero(beta) / p / math.sqrt(N) * 10.0)
    lam = np.abs(r.standard_cauchy(p)).clip(1e-2, 1e3)
    live = beta != 0.0
    lam[live] = np.abs(beta[live]) / tau
    sd = 1.5 / math.sqrt(N)
    b = beta + r.normal(0.0, 1.0, p) * np.where(live, sd, sd * (tau * lam) / np.hypot(tau * lam, sd))
    lam_m2, tau_m2 = lam ** -2.0, tau ** -2.0
    return dict(beta=b, lam_m2=lam_m2, nu_m1=r.exponential(1.0, p) / (1.0 + lam_m2), tau_m2=tau_m2,
                xi_m1=float(r.exponential(1.0)) / (1.0 + tau_m2), sweep=1000)


def _resume(chain, beta, N, seed):
    chain.set_state(**_state(beta, N, seed))


def _shapes(c, seed=77):
    """Uneven shapes of a batch: the case's, whatever the inputs' seed."""
    r = np.random.default_rng([seed, c["datasets"], c["n_max"], c["p_max"]])
    Ns = np.exp(r.uniform(math.log(c["n_min"]), math.log(c["n_max"]), c["datasets"]))
    return [(int(n), int(p)) for n, p in zip(Ns, r.integers(c["p_min"], c["p_max"] + 1, c["datasets"]))]


def prepare(case, seed):
    kind, xt = case["kind"], case["xt"]
    if kind == "gram":
        X = torch.randn(case["N"], case["ld"], generator=_generator(seed), device="cuda")
        if xt == "bf16":
            X = X.to(torch.bfloat16)
        return dict(case=case, X=X, G=torch.empty(case["p"], case["p"], dtype=torch.float64, device="cuda"))
    if kind == "batch":
        ds = [_design(n, p, seed + 1000 * i) for i, (n, p) in enumerate(_shapes(case))]
        b = hsp.Batch([(X, y, xt) for X, y, _ in ds], chains=1, seed=seed + 1)
        for i, (X, _, beta) in enumerate(ds):
            _resume(b.chain(i), beta, X.shape[0], seed + i)
        return dict(case=case, b=b, done=0)
    X, y, beta = _design(case["N"], case["p"], seed, case.get("ybar"))
    if kind == "fit":
        torch.cuda.synchronize()
        return dict(case=case, X=X, y=y, seed=seed + 1)
    if kind == "shared":
        b = hsp.Batch([(X, y, xt)], chains=case["chains"], seed=seed + 1)
        for i in range(case["chains"]):
            _resume(b.chain(i), beta, case["N"], seed + i)
        return dict(case=case, b=b, done=0)
    s = hsp.Sampler(X, y, seed=seed + 1, x_type=xt, record_lambda=case.get("lam", False))
    _resume(s, beta, case["N"], seed)
    return dict(case=case, s=s, done=0)


def _named(d):
    out = {"beta": d[0], "tau_m2": d[1]}
    if len(d) == 4:
        out["lam_m2"] = d[2]
    return out


def run(state):
    case = state["case"]
    kind, xt = case["kind"], case["xt"]
    if kind == "gram":
        hsp.hsp_gram(state["X"].data_ptr(), hsp.HSP_X_F32 if xt == "f32" else hsp.HSP_X_BF16, case["N"], case["p"],
                     case["ld"], state["G"].data_ptr())
        return state["G"]
    n = case["sweeps"]
    if kind == "fit":
        s = hsp.Sampler(state["X"], state["y"], seed=state["seed"], x_type=xt, record_lambda=case.get("lam", False))
        s.sweep(n)
        d = s.draws(0, n)
        s.close()
        return _named(d)
    first = state["done"]
    state["done"] = first + n
    if kind == "sweep":
        state["s"].sweep(n)
        return _named(state["s"].draws(first, n))
    state["b"].sweep(n)
    got = [state["b"].chain(i).draws(first, n) for i in range(len(state["b"]))]
    return {"beta": np.concatenate([g[0].ravel() for g in got]), "tau_m2": np.concatenate([g[1] for g in got])}


def work(case):
    es = 4 if case["xt"] == "f32" else 2
    kind = case["kind"]
    if kind == "gram":
        N, p = case["N"], case["p"]
        return {"bytes": N * p * es + 8 * p * p, "flops": N * p * (p + 1)}
    shapes = _shapes(case) if kind == "batch" else [(case["N"], case["p"])]
    chains, n = case.get("chains", 1), case["sweeps"]
    nbytes = sum(N * p * es + N for N, p in shapes) * n  # one read of every distinct design per sweep
    flops = sum(4 * N * p + p ** 3 / 3 + 2 * p * p for N, p in shapes) * n * chains
    if kind == "fit":  # X and y as given, the Gram, then the sweeps
        N, p = shapes[0]
        nbytes += N * p * 4 + N + 8 * p * p
        flops += N * p * (p + 1)
    out = sum(8 * (p * (2 if case.get("lam") else 1) + 1) for _, p in shapes) * n * chains
    return {"bytes": nbytes + out, "flops": flops}


# ---- the same in float64, in plain torch -----------------------------------------------
M32 = 0xFFFFFFFF
TAG_Z, TAG_LAM, TAG_TAU, TAG_S, TAG_NU, TAG_XI = 1, 2, 3, 4, 5, 6


def _uniforms(seed, idx, sweep, tag, rnd, chain):
    """The four uniforms of Philox4x32-10 at counter (idx, sweep, tag << 24 | rnd, chain)."""
    c0, c2 = idx.to(torch.int64), torch.zeros_like(idx, dtype=torch.int64) + ((tag << 24) | rnd)
    c1, c3 = torch.full_like(c0, sweep), torch.full_like(c0, chain)
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((b >> 32) & M32) ^ c1 ^ k0, b & M32, ((a >> 32) & M32) ^ c3 ^ k1, a & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return [((w >> 8) | 1).double() * 2.0 ** -24 for w in (c0, c1, c2, c3)]


def _z(eta, y, seed, sweep, chain):
    """Truncated normals by the paper's two rejection samplers (branch at 0.47)."""
    ys = 2.0 * y.double() - 1.0
    mu_all = ys * eta
    t_all = torch.zeros_like(mu_all)
    left = torch.arange(eta.numel(), device=eta.device)
    for rnd in range(2048):
        if not left.numel():
            break
        mu = mu_all[left]
        u = _uniforms(seed, left, sweep, TAG_Z, rnd, chain)
        gauss = mu.float() > 0.47
        theta = ((mu * mu + 4.0).sqrt() - mu) / 2.0
        t = torch.zeros_like(mu)
        ok = torch.zeros_like(gauss)
        for u1, u2 in ((u[0], u[1]), (u[2], u[3])):
            tg = mu + (-2.0 * u1.log()).sqrt() * torch.cos(2.0 * math.pi * u2)
            tr = -u1.log() / theta
            acc = torch.where(gauss, tg > 0.0, u2 < torch.exp(-0.5 * (tr - 1.0 / theta) ** 2)) & ~ok
            t = torch.where(acc, torch.where(gauss, tg, tr), t)
            ok = ok | acc
        t_all[left[ok]] = t[ok]
        left = left[~ok]
    return ys * t_all


def _tau(p, rate, seed, sweep, chain):
    """Gamma((p + 1) / 2, rate): the first acceptance of Cheng's GB."""
    sh = (p + 1) / 2.0
    A, B = 1.0 / math.sqrt(2.0 * sh - 1.0), sh - math.log(4.0)
    C, D = sh + 1.0 / A, 1.0 + math.log(4.5)
    for m in range(1 << 16):
        u = _uniforms(seed, torch.zeros(1, dtype=torch.int64), sweep, TAG_TAU, m >> 1, chain)
        u1, u2 = (float(u[2 * (m & 1)]), float(u[2 * (m & 1) + 1]))
        V = A * math.log(u1 / (1.0 - u1))
        X, Z = sh * math.exp(V), u1 * u1 * u2
        R = B + C * V - X
        if R + D - 4.5 * Z >= 0.0 or R >= math.log(Z):
            return X / rate


def _gram64(X, p):
    G = torch.zeros(p, p, dtype=torch.float64, device="cuda")
    for i in range(0, X.shape[0], ROWS):
        x = X[i:i + ROWS, :p].double()
        G += x.T.contiguous() @ x
    return G


def _chain64(X, y, G, st, seed, chain, sweeps, lam_too):
    """`sweeps` whole sweeps in float64 from the state st."""
    N, p = X.shape
    G = G.cpu()
    beta, lam, nu = (torch.from_numpy(np.array(st[k])) for k in ("beta", "lam_m2", "nu_m1"))
    tau, xi = st["tau_m2"], st["xi_m1"]
    j = torch.arange(p)
    betas, taus, lams = [], [], []
    for k in range(st["sweep"] + 1, st["sweep"] + 1 + sweeps):
        bg = beta.cuda()
        eta = torch.cat([X[i:i + ROWS].double() @ bg for i in range(0, N, ROWS)])
        z = _z(eta, y, seed, k, chain)
        b = sum(X[i:i + ROWS].double().T @ z[i:i + ROWS] for i in range(0, N, ROWS)).cpu()
        lam = -_uniforms(seed, j, k, TAG_LAM, 0, chain)[0].log() / (nu + tau * beta * beta / 2.0)
        tau = _tau(p, xi + float((lam * beta * beta).sum()) / 2.0, seed, k, chain)
        us = _uniforms(seed, j, k, TAG_S, 0, chain)
        s = (-2.0 * us[0].log()).sqrt() * torch.cos(2.0 * math.pi * us[1])
        L = torch.linalg.cholesky(G + torch.diag(tau * lam))  # Q = L L^T, U = L^T
        y1 = torch.linalg.solve_triangular(L, b[:, None], upper=False) + s[:, None]
        beta = torch.linalg.solve_triangular(L.T, y1, upper=True)[:, 0]
        nu = -_uniforms(seed, j, k, TAG_NU, 0, chain)[0].log() / (1.0 + lam)
        xi = -math.log(float(_uniforms(seed, torch.zeros(1, dtype=torch.int64), k, TAG_XI, 0, chain)[0])) / (1.0 + tau)
        betas.append(beta.numpy())
        taus.append(tau)
        lams.append(lam.numpy())
    out = {"beta": np.stack(betas), "tau_m2": np.array(taus)}
    if lam_too:
        out["lam_m2"] = np.stack(lams)
    return out


def _stored(X, xt):
    return X.to(torch.bfloat16).float() if xt == "bf16" else X


def exact(case, seed):
    kind, xt = case["kind"], case["xt"]
    if kind == "gram":
        return _gram64(prepare(case, seed)["X"], case["p"])
    n, lam = case["sweeps"], case.get("lam", False)
    if kind == "batch":
        got = []
        for i, (N, p) in enumerate(_shapes(case)):
            X, y, beta = _design(N, p, seed + 1000 * i)
            X = _stored(X, xt)
            got.append(_chain64(X, y, _gram64(X, p), _state(beta, N, seed + i), seed + 1, i, n, False))
    else:
        X, y, beta = _design(case["N"], case["p"], seed, case.get("ybar"))
        X = _stored(X, xt)
        G = _gram64(X, case["p"])
        if kind == "fit":
            p = case["p"]
            cold = dict(beta=np.zeros(p), lam_m2=np.ones(p), nu_m1=np.ones(p), tau_m2=1.0, xi_m1=1.0, sweep=0)
            return _chain64(X, y, G, cold, seed + 1, 0, n, lam)
        if kind == "sweep":
            return _chain64(X, y, G, _state(beta, case["N"], seed), seed + 1, 0, n, lam)
        got = [_chain64(X, y, G, _state(beta, case["N"], seed + i), seed + 1, i, n, False) for i in range(case["chains"])]
    return {"beta": np.concatenate([g["beta"].ravel() for g in got]), "tau_m2": np.concatenate([g["tau_m2"] for g in got])}
