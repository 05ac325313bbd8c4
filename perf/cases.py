"""The framework's work as its users have it do, with sizes over the real range.

``listed()`` gives the standing cases, ``draw(rng)`` one more of the same
ranges; ``prepare`` makes what a program holds before the call, ``run`` is one
pass through the public entry points, ``work`` what the pass cannot do
without and ``exact`` its outputs in 64 bits by plain torch, written from the
models' and the generator's definitions.

Kinds of case:

* ``systematic``: the stateless resampler on a caller's own log-weights;
* ``filter``: one likelihood estimate (every filter re-initialised, T
  intervals, the estimates and their traces read back), plain or batched
  layout, optionally with a history and the state sample drawn from it;
* ``pmmh``: marginal Metropolis-Hastings chains on the Lorenz '96 forcing;
* ``smc2``: SMC over the parameters with a particle filter each;
* ``kalman``: the windkessel's exact likelihood for many parameter sets;
* ``kalman_pmmh``: chains on the windkessel's circuit parameters driven by it.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1306_3277_amd as pf

WK, L96, L96_STAGE = 1, 2, 3
PRECISION = {"fp64": pf.PF_FP64, "fast": pf.PF_FP32_MIXED, "accurate": pf.PF_FP32_ACCURATE}
SCHEME = {"systematic": pf.PF_RESAMPLE_SYSTEMATIC, "stratified": pf.PF_RESAMPLE_STRATIFIED,
          "multinomial": pf.PF_RESAMPLE_MULTINOMIAL, "metropolis": pf.PF_RESAMPLE_METROPOLIS,
          "rejection": pf.PF_RESAMPLE_REJECTION}
UNEVEN = (256, 512, 1024, 2048, 4096, 8192)


def _filter(name, model, d, K, T, B, n, layout, precision, obs_every=1, obs_sd=None,
            scheme="systematic", ess=0.0, uneven=False, history=False, state=False, groups=0):
    """ess 0: resample every time; uneven: n is the most a filter holds;
    groups 0: the handle's own tuning."""
    return dict(name=name, kind="filter", model=model, d=d, K=K, T=T, B=B, n=n, layout=layout,
                precision=precision, obs_every=obs_every,
                obs_sd=obs_sd if obs_sd is not None else (1.0 if model == WK else 0.5),
                scheme=scheme, ess=ess, uneven=uneven, history=history, state=state,
                groups=groups)


def listed():
    return [
        # a program with its own model resamples a small particle set: launches and latency
        dict(name="systematic_1000", kind="systematic", n=1000, spread=1.0),
        # the same on a large, odd set with concentrated weights
        dict(name="systematic_1000003", kind="systematic", n=1000003, spread=8.0),
        # the windkessel example: 1,024 particles, one likelihood with the final particles
        _filter("windkessel_1024_fp64", WK, 1, 10, 100, 1, 1024, "plain", "fp64", state=True),
        # the Lorenz '96 example, one filter of 65,536 particles in the accurate form
        _filter("lorenz96_d8_65536_accurate", L96, 8, 8, 200, 1, 65536, "plain", "accurate"),
        # the large filter: d = 40, 2^20 particles, every second component observed
        _filter("lorenz96_d40_1048576_fast", L96, 40, 8, 60, 1, 1 << 20, "plain", "fast",
                obs_every=2),
        # multinomial resampling (as the paper writes the filter) of an odd particle count
        _filter("lorenz96_d16_100003_multinomial", L96, 16, 8, 50, 1, 100003, "plain", "fast",
                scheme="multinomial"),
        # parameter particles: 512 filters of uneven size, the headline workload
        _filter("batched_512_uneven_accurate", L96, 8, 8, 100, 512, 8192, "batched", "accurate",
                uneven=True, groups=2),
        # a smoother: FP64, the paper's noise inside the stages, stored ancestry, state samples
        _filter("batched_64_fp64_history", L96_STAGE, 8, 8, 50, 64, 3000, "batched", "fp64",
                history=True),
        # parallel marginal Metropolis-Hastings chains on the forcing
        dict(name="pmmh_64x4096", kind="pmmh", d=8, K=8, T=100, B=64, n=4096, iters=4),
        # SMC over the parameters, a filter of its own for each
        dict(name="smc2_64", kind="smc2", d=8, K=8, T=40, B=64, n=2048),
        # exact likelihoods of a batch of windkessel parameter sets
        dict(name="kalman_512", kind="kalman", K=10, T=100, B=512),
        # long chains on the windkessel's circuit parameters
        dict(name="kalman_pmmh_512x500", kind="kalman_pmmh", K=10, T=100, B=512, iters=500),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["systematic", "wk", "plain", "batched", "pmmh", "smc2", "kalman",
                       "kalman_pmmh"])
    precision = rng.choice(["fp64", "fast", "accurate"])
    if kind == "systematic":
        return dict(kind=kind, n=_log(rng, 1, 4000000), spread=rng.choice([0.3, 1.0, 8.0, 40.0]))
    if kind == "wk":
        c = _filter("", WK, 1, rng.randint(1, 20), rng.randint(20, 200), 1, _log(rng, 64, 32768),
                    "plain", precision, scheme=rng.choice(["systematic", "stratified",
                                                           "multinomial", "metropolis"]),
                    ess=rng.choice([0.0, 0.0, 0.5]), state=rng.random() < 0.5)
    elif kind == "plain":
        c = _filter("", rng.choice([L96, L96_STAGE]), rng.choice([4, 8, 16, 32, 40]),
                    rng.randint(2, 10), rng.randint(10, 40), 1, _log(rng, 1000, 200000), "plain",
                    precision, obs_every=rng.choice([1, 2]), obs_sd=rng.choice([0.5, 2.0]),
                    scheme=rng.choice(["systematic", "stratified", "multinomial", "metropolis"]),
                    ess=rng.choice([0.0, 0.0, 0.5]))
    elif kind == "batched":
        spread = rng.random() < 0.3  # rejection's attempts follow the weights: spread ones
        c = _filter("", rng.choice([L96, L96_STAGE]), rng.choice([4, 8, 16]), rng.randint(2, 10),
                    rng.randint(10, 60), _log(rng, 2, 300), _log(rng, 100, 8192), "batched",
                    precision, obs_sd=4.0 if spread else 0.5,
                    scheme=rng.choice(["systematic", "stratified", "multinomial", "metropolis"]
                                      + (["rejection"] * 2 if spread else [])),
                    uneven=rng.random() < 0.5, groups=rng.choice([0, 1, 2]))
        if c["ess"] == 0.0 and rng.random() < 0.3:
            c["history"] = True
    elif kind == "pmmh":
        c = dict(kind=kind, d=8, K=8, T=rng.randint(10, 100), B=rng.randint(1, 64),
                 n=_log(rng, 100, 4096), iters=rng.randint(1, 4))
    elif kind == "smc2":
        c = dict(kind=kind, d=rng.choice([4, 8]), K=8, T=rng.randint(5, 40), B=rng.randint(4, 64),
                 n=_log(rng, 100, 2048))
    elif kind == "kalman":
        c = dict(kind=kind, K=rng.randint(1, 20), T=rng.randint(5, 300), B=_log(rng, 1, 20000))
    else:
        c = dict(kind=kind, K=rng.randint(1, 12), T=rng.randint(5, 100), B=_log(rng, 1, 1024),
                 iters=rng.randint(20, 300))
    c.pop("name", None)
    return c


# ---------------------------------------------------------------- inputs

def _counts(c):
    """Particles of each filter: n, or (uneven) drawn once for the case from
    the powers of two up to n and a few odd counts."""
    if not c.get("uneven"):
        return np.full(c["B"], c["n"], dtype=np.int64)
    rng = np.random.default_rng(2)
    top = [k for k in UNEVEN if k <= c["n"]] or [c["n"]]
    n = rng.choice(np.asarray(top, dtype=np.int64), size=c["B"])
    n[::7] = np.maximum(1, n[::7] - rng.integers(1, 100, size=n[::7].size))
    return np.minimum(n, c["n"])


def _flow(n, h=0.01):
    """The paper's windkessel flow: a half-period pulse of 500 per 0.8 s."""
    t = np.arange(n + 1, dtype=np.float64) * h
    return np.where(np.mod(t, 0.8) <= 0.3, 500.0 * np.sin(np.pi * t / 0.8) ** 2, 0.0)


def _wk_theta(R, C, Z, sigma2, m0=90.0, s0=15.0, h=0.01):
    a = np.exp(-h / (R * C))
    cc = R * (1.0 - a)
    one = np.ones_like(a)
    return np.stack([a, cc, Z * one, cc * np.sqrt(sigma2), m0 * one, s0 * one], axis=-1)


def _problem(c, seed):
    """The filtering problem of a case: parameters from the seed, data
    simulated from the model."""
    rng = np.random.default_rng([seed, 1])
    B, T, K = c["B"], c["T"], c["K"]
    model = c.get("model", WK if c["kind"].startswith("kalman") else L96)
    n = _counts(c) if "n" in c else np.ones(B, dtype=np.int64)
    if model == WK:
        scale = rng.uniform(0.8, 1.2, size=(B, 4))
        theta = _wk_theta(*(np.array([1.0, 1.5, 0.03, 25.0]) * scale).T)
        p = SimpleNamespace(d=1, h=0.01, obs_idx=np.zeros(1, dtype=np.int32), q=_flow(T * K),
                            data_theta=_wk_theta(np.float64(1.0), 1.5, 0.03, 25.0))
    else:
        theta = np.stack([rng.uniform(6.0, 10.0, size=B), rng.uniform(0.05, 0.3, size=B)], axis=1)
        if B == 1:  # one filter: at the data's parameters
            theta[:] = (8.0, 0.1)
        p = SimpleNamespace(d=c["d"], h=0.05, q=None, data_theta=np.array([8.0, 0.1]),
                            obs_idx=np.arange(0, c["d"], c.get("obs_every", 1), dtype=np.int32))
    p.model, p.K, p.T, p.theta, p.n_particles = model, K, T, theta, n
    p.obs_sd = c.get("obs_sd", 2.0 if model == WK else 0.5)
    p.precision = PRECISION[c.get("precision", "fast")]
    p.seed, p.data_seed, p.obs = seed * 7919 + 11, seed * 104729 + 5, None
    data = SimpleNamespace(**vars(p))
    data.obs_sd = min(p.obs_sd, 1.0)
    p.obs = pf.simulate(data)[1]
    return p


def _uniforms(rng, shape):
    return (rng.integers(0, 2 ** 32, size=shape, dtype=np.uint64).astype(np.float64) + 0.5) * 2.0 ** -32


WK_MH = SimpleNamespace(prior_shape=(2.0, 2.0, 2.0), prior_scale=(0.9, 1.5, 0.03), ig_shape=2.0,
                        ig_scale=25.0, step_sd=(0.03, 0.1, 0.002), ig_prop_shape=2.0,
                        ig_prop_factor=3.0, m0=90.0, s0=15.0)


def _chain_inputs(c, seed):
    rng = np.random.default_rng([seed, 2])
    B, n = c["B"], c["iters"]
    theta0 = np.array([1.0, 1.5, 0.03, 25.0]) * rng.uniform(0.8, 1.2, size=(B, 4))
    prop = np.concatenate([_uniforms(rng, (n, B, 3)), rng.gamma(2.0, 1.0, size=(n, B, 1))], axis=2)
    return theta0, np.ascontiguousarray(prop), _uniforms(rng, (n, B))


def _log_weights(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    lw = torch.randn(c["n"], generator=g, device="cuda", dtype=torch.float64) * c["spread"]
    u = torch.rand((), generator=torch.Generator().manual_seed(seed), dtype=torch.float64).item()
    return lw, u


def prepare(case, seed):
    c = case
    if c["kind"] == "systematic":
        lw, u = _log_weights(c, seed)
        nb = int(pf.load().pf_systematic_workspace_bytes(c["n"]))
        return SimpleNamespace(
            c=c, lw=lw, u=u, workspace=torch.empty(nb + 256, dtype=torch.uint8, device="cuda"),
            anc=torch.empty(c["n"], dtype=torch.int32, device="cuda"),
            stats=torch.empty(2, dtype=torch.float64, device="cuda"))
    p = _problem(c, seed)
    s = SimpleNamespace(c=c, problem=p)
    if c["kind"] == "filter":
        s.f = pf.Filter(p, layout=pf.PF_LAYOUT_BATCHED if c["layout"] == "batched"
                        else pf.PF_LAYOUT_PLAIN)
        if c["scheme"] != "systematic" or c["ess"]:
            s.f.set_resampler(SCHEME[c["scheme"]], 8 if c["scheme"] == "metropolis" else 0,
                              c["ess"] or float("inf"))
        if c["groups"]:
            s.f.set_tuning(512, c["groups"])
        if c["history"]:
            s.f.attach_history()
    elif c["kind"] == "pmmh":
        s.f = pf.Filter(p, layout=pf.PF_LAYOUT_BATCHED)
        s.f.set_tuning(512, 2)
        rng = np.random.default_rng([seed, 3])
        s.inputs = SimpleNamespace(
            log_f0=np.log(rng.uniform(6.0, 10.0, size=c["B"])),
            z=rng.standard_normal(size=(c["iters"], c["B"])),
            alpha=_uniforms(rng, (c["iters"], c["B"])), step_sd=0.05, f_lo=6.0, f_hi=10.0,
            sigma=0.1)
    elif c["kind"] == "smc2":
        s.f = pf.Filter(p, layout=pf.PF_LAYOUT_BATCHED)
        s.proposal = pf.Filter(p, layout=pf.PF_LAYOUT_BATCHED)
        rng = np.random.default_rng([seed, 4])
        T, B = c["T"], c["B"]
        s.inputs = SimpleNamespace(
            T=T, theta0=p.theta, z=rng.standard_normal(size=(T, B, 2)),
            log_alpha=np.log(_uniforms(rng, (T, B))), u=_uniforms(rng, T) - 2.0 ** -33,
            w_copy=rng.integers(0, 2 ** 32, size=(T, B), dtype=np.uint64).astype(np.uint32),
            step_sd=[0.1, 0.01], lo=[6.0, 0.05], hi=[10.0, 0.3])
    else:
        s.f = pf.Filter(p)
        if c["kind"] == "kalman_pmmh":
            s.inputs = [torch.from_numpy(a).cuda() for a in _chain_inputs(c, seed)]
    return s


# ---------------------------------------------------------------- a pass

def run(s):
    c = s.c
    if c["kind"] == "systematic":
        return pf.systematic(s.lw, s.u, anc=s.anc, stats=s.stats, workspace=s.workspace)
    f = s.f
    if c["kind"] == "filter":
        f.reset(0)
        f.graph_run(c["T"])
        ll, ess, _ = f.loglik(allow_numeric=True)
        ell, ess_t = f.trace()
        out = dict(loglik=ll, ess=ess, ell=ell, ess_trace=ess_t)
        if c["state"]:
            out["state"] = f.get_state()
        if c["history"]:
            out["path"], out["index"] = f.backtrace()
        return out
    if c["kind"] == "pmmh":
        return f.pmmh(s.inputs)
    if c["kind"] == "smc2":
        r = f.smc2(s.proposal, s.inputs)
        return {k: v for k, v in r.items() if k != "status"}
    if c["kind"] == "kalman":
        return f.kalman()
    return f.kalman_pmmh(WK_MH, *s.inputs)


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    c = case
    if c["kind"] == "systematic":
        return {"bytes": 12.0 * c["n"] + 16, "flops": 20.0 * c["n"]}
    B, T, K = c["B"], c["T"], c["K"]
    if c["kind"].startswith("kalman"):
        # per interval and parameter set: the predictions' two affine maps and the correction
        runs = c.get("iters", 0) + 1
        per = 56.0 * c["iters"] + 72 if "iters" in c else 56.0 + 8 * T
        return {"bytes": per * B + 8.0 * T * (K + 1), "flops": float(runs) * B * T * (6 * K + 20)}
    n, d = float(_counts(c).sum()), c["d"]
    model = c.get("model", L96)
    sx = 8.0 if c.get("precision", "fast") == "fp64" else 4.0
    # particle-intervals of the pass
    steps = n * {"filter": T, "pmmh": T * (c.get("iters", 0) + 1), "smc2": T * (T + 1) / 2}[c["kind"]]
    # a substep: the transition (fourth-order Runge-Kutta: about 30 per component) and a normal
    flops = steps * (K * (14.0 if model == WK else 30.0 * d) + 3.0 * d + 10)
    nbytes = steps * 2 * d * sx  # resampling moves every particle once an interval
    if c.get("history"):
        nbytes += steps * (d * sx + 4)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- the outputs in 64 bits

def exact(case, seed):
    c = case
    if c["kind"] == "systematic":
        lw, _ = _log_weights(c, seed)
        w = torch.exp(lw - lw.max())
        ell = lw.max() + torch.log(w.sum()) - math.log(c["n"])
        return None, torch.stack([ell, w.sum() ** 2 / (w * w).sum()])
    if c["kind"] in ("pmmh", "smc2"):
        return None  # every decision rests on FP32 filters of a chaotic model
    p = _problem(c, seed)
    if c["kind"] == "kalman":
        return _kalman(p, torch.from_numpy(p.theta))
    if c["kind"] == "kalman_pmmh":
        return _kalman_chains(p, *_chain_inputs(c, seed))
    # single filters whose particles keep to one trajectory in 64 bits; an FP32 filter of the
    # chaotic model leaves it within a few intervals
    if c["B"] > 1 or (c["precision"] != "fp64" and p.model != WK):
        return None
    if c["scheme"] == "metropolis":
        return None
    return _particle_filter(c, p)


def _kalman(p, theta):
    """Kalman filter of the windkessel: (loglik [B], increments [B, T])."""
    a, cc, Z, sp, m, s0 = (theta[..., i] for i in range(6))
    V, R = s0 * s0, p.obs_sd ** 2
    ell = []
    for t in range(p.T):
        for k in range(p.K):
            m = a * m + cc * p.q[t * p.K + k]
            V = a * a * V + sp * sp
        v = p.obs[t, 0] - (m + Z * p.q[(t + 1) * p.K])
        S = V + R
        ell.append(-0.5 * (torch.log(2 * math.pi * S) + v * v / S))
        m = m + V / S * v
        V = (1 - V / S) * V
    ell = torch.stack(ell, dim=-1)
    return ell.sum(-1), ell


def _kalman_chains(p, theta0, prop, alpha):
    h = WK_MH
    x, prop, alpha = (torch.from_numpy(v) for v in (theta0, prop, alpha))
    sd = torch.tensor(h.step_sd, dtype=torch.float64)
    shape, scale = (torch.tensor(v, dtype=torch.float64) for v in (h.prior_shape, h.prior_scale))

    def cdf(v):
        return 0.5 * torch.erfc(-v / math.sqrt(2.0))

    def params(y):
        a = torch.exp(-p.h / (y[:, 0] * y[:, 1]))
        cc = y[:, 0] * (1 - a)
        one = torch.ones_like(a)
        return torch.stack([a, cc, y[:, 2], cc * torch.sqrt(y[:, 3]), h.m0 * one, h.s0 * one], dim=1)

    def prior(y):
        return ((shape - 1) * torch.log(y[:, :3]) - y[:, :3] / scale).sum(1) \
            - (h.ig_shape + 1) * torch.log(y[:, 3]) - h.ig_scale / y[:, 3]

    ll0 = ll = _kalman(p, params(x))[0]
    lp = prior(x)
    accepts = torch.zeros(len(x), dtype=torch.int32)
    theta, lls = [], []
    for u, al in zip(prop, alpha):
        p0 = cdf(-x[:, :3] / sd)
        up = u[:, :3]
        z = torch.where(up <= 0.5, torch.special.ndtri(p0 + up * (1 - p0)),
                        -torch.special.ndtri((1 - up) * (1 - p0)))
        y = torch.cat([x[:, :3] + sd * z, (h.ig_prop_factor * x[:, 3] / u[:, 3])[:, None]], dim=1)
        inside = ((y > 0) & torch.isfinite(y)).all(1)
        ys = torch.where(inside[:, None], y, x)
        r = ys[:, 3] / x[:, 3]
        lq = (torch.log(cdf(x[:, :3] / sd)) - torch.log(cdf(ys[:, :3] / sd))).sum(1) \
            + (2 * h.ig_prop_shape + 1) * torch.log(r) - h.ig_prop_factor * (r - 1 / r)
        llp, lpp = _kalman(p, params(ys))[0], prior(ys)
        take = inside & (torch.log(al) <= (llp - ll) + ((lpp - lp) + lq))
        x = torch.where(take[:, None], ys, x)
        ll, lp = torch.where(take, llp, ll), torch.where(take, lpp, lp)
        accepts += take.to(torch.int32)
        theta.append(x)
        lls.append(ll)
    return dict(theta=torch.stack(theta), ll=torch.stack(lls), accepts=accepts, ll0=ll0)


def _philox(c0, c1, c2, c3, key):
    """Philox4x32-10 (Salmon et al., 2011) on int64 tensors of 32-bit words."""
    m = 0xFFFFFFFF
    k0, k1 = key & m, key >> 32

    def mul(k, x):  # high and low words of a 32 x 32 product, within 63 bits
        lo, hi = k * (x & 0xFFFF), k * (x >> 16)
        s = lo + ((hi & 0xFFFF) << 16)
        return ((hi >> 16) + (s >> 32)) & m, s & m

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c0)
        h1, l1 = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c0, c1, c2, c3


def _particle_filter(c, p):
    """The bootstrap filter of one set of parameters in 64 bits on the
    generator's numbers (counter: particle, substep, tag | block, filter)."""
    N, d, dev = int(p.n_particles[0]), p.d, "cuda"
    idx = torch.arange(N, dtype=torch.int64, device=dev)
    word = torch.zeros_like(idx)

    def uniforms(tag, blk, n, j):
        w = _philox(j, torch.full_like(j, n), torch.full_like(j, (tag << 28) | (blk << 20)),
                    torch.zeros_like(j), p.seed)
        return [(v.double() + 0.5) * 2.0 ** -32 for v in w]

    def normals(tag, n):
        z = []
        for blk in range(max(1, d // 4)):
            u = uniforms(tag, blk, n, idx)
            for a, b in ((u[0], u[1]), (u[2], u[3])):
                r = torch.sqrt(-2 * torch.log(a))
                z += [r * torch.cos(2 * math.pi * b), r * torch.sin(2 * math.pi * b)]
        return torch.stack(z[:d])

    th = [float(v) for v in p.theta[0]]
    x = normals(1, 0)
    if p.model == WK:
        x = th[4] + th[5] * x
    else:
        F, sq = th[0], th[1] * math.sqrt(p.h)

        def drift(y, f):
            return (y.roll(-1, 0) - y.roll(2, 0)) * y.roll(1, 0) - y + f

    yobs = torch.from_numpy(p.obs).to(dev)
    cst = -len(p.obs_idx) * (math.log(p.obs_sd) + 0.5 * math.log(2 * math.pi))
    loglik, ells, esss, carried, lprev = 0.0, [], [], None, math.log(N)
    anc = idx
    for t in range(1, p.T + 1):
        for s in range(1, p.K + 1):
            n = (t - 1) * p.K + s
            z = normals(2, n)
            if p.model == WK:
                x = th[0] * x + th[1] * p.q[n - 1] + th[3] * z
                continue
            f = F + sq * z / p.h if p.model == L96_STAGE else F
            k1 = drift(x, f)
            k2 = drift(x + 0.5 * p.h * k1, f)
            k3 = drift(x + 0.5 * p.h * k2, f)
            k4 = drift(x + p.h * k3, f)
            x = x + p.h / 6 * (k1 + k4 + 2 * (k2 + k3))
            if p.model == L96:
                x = x + sq * z
        mean = x + th[2] * p.q[t * p.K] if p.model == WK else x[torch.from_numpy(p.obs_idx).long().to(dev)]
        lw = -0.5 * (((yobs[t - 1][:, None] - mean) / p.obs_sd) ** 2).sum(0) + cst
        lw = lw if carried is None else carried + lw
        M = lw.max()
        w = torch.exp(lw - M)
        S = w.sum()
        L = (M + torch.log(S)).item()
        ells.append(L - lprev)
        loglik += ells[-1]
        esss.append((S * S / (w * w).sum()).item())
        if c["ess"] and not esss[-1] < c["ess"] * N:
            carried, lprev = lw, L
            continue
        carried, lprev = None, math.log(N)
        W = torch.cumsum(w, 0)
        if c["scheme"] == "systematic":
            thr = (uniforms(3, 0, t, word[:1])[0] + idx.double()) * (S / N)
        else:
            tag, blk = (3, 1) if c["scheme"] == "stratified" else (10, 0)
            u = torch.stack(uniforms(tag, blk, t, idx[: (N + 3) // 4]), 1).reshape(-1)[:N]
            thr = (u + idx.double()) * (S / N) if c["scheme"] == "stratified" else u * S
        anc = torch.searchsorted(W, thr, right=True).clamp(max=N - 1)
        x = x[:, anc]
    out = dict(loglik=np.array([loglik]), ess=np.array([esss[-1]]), ell=np.array([ells]),
               ess_trace=np.array([esss]))
    if c["state"]:
        out["state"] = x.cpu().numpy()
    return out
