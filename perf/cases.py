"""The workloads whose speed is followed: one call each through the public entry points.

Every case is a dict of plain values; its "kind" names the entry point:

  chisq   rv_chisq              chi-square of a batch of models on one data set
  grad    rv_chisq_grad         chi-square and gradient (optimisers, samplers with gradients)
  nll     rv_nll_grad           likelihood with a free jitter and its gradient
  gn      rv_chisq_gn           Gauss-Newton products (Levenberg-Marquardt steps)
  ragged  RaggedPlan            chi-square of uneven systems, a plan reused for many calls
  static  rv_chisq_ragged_static  the same without a plan (a new batch on every call)
  demc    DEMC.run              generations of the population sampler
  kepler  kepler_solve          Kepler's equation for pairs (M, e)
  astro   astro_chisq           astrometric chi-square

Sizes and distributions are those of the framework's own workloads (`synth/`): periods log-uniform
over 1 to 1000 days, semi-amplitudes 1 to 100 m/s, e up to 0.9 (0.8 for derivatives), sigma 1 to
5 m/s, observed velocities those of one truth system plus noise.
"""
import math

import torch

import paper_0812_2976_amd as kp

TWO_PI = 2.0 * math.pi
DEV = "cuda"
F64 = torch.float64


def _case(name, kind, **kw):
    return {"name": name, "kind": kind, **kw}


def listed():
    return [
        # the smallest calls: a handful of trial models of one star on an ordinary data set
        _case("chisq_trial", "chisq", prec="mixed", n_sys=16, n_pl=2, n_obs=60, offset=False, jitter=False),
        # the largest: a grid or population of a million four-planet models (the default benchmark's workload)
        _case("chisq_million", "chisq", prec="mixed", n_sys=1048576, n_pl=4, n_obs=256, offset=False, jitter=False),
        # an ordinary batch with nothing round about it, offset and jitter fitted
        _case("chisq_odd", "chisq", prec="mixed", n_sys=100003, n_pl=3, n_obs=157, offset=True, jitter=True),
        # plain binary64: the accuracy reference of the same batch evaluation
        _case("chisq_fp64", "chisq", prec="fp64", n_sys=65536, n_pl=4, n_obs=256, offset=False, jitter=False),
        # gradients of a large batch (gradient-based samplers and optimisers)
        _case("grad_batch", "grad", prec="mixed", n_sys=262144, n_pl=4, n_obs=256, offset=True, jitter=False),
        # likelihood and gradient in binary64: a population's final refinement, jitter free
        _case("nll_fp64", "nll", prec="fp64", n_sys=2000, n_pl=2, n_obs=75, offset=True, jitter=True),
        # one Levenberg-Marquardt step of a large batch
        _case("gn_batch", "gn", prec="mixed", n_sys=262144, n_pl=4, n_obs=256, offset=True, jitter=False),
        # a survey: every star with its own observations and planet count, evaluated again and again
        _case("ragged_survey", "ragged", prec="mixed", n_sys=262144, n_pl_max=7, obs_lo=16, obs_hi=1024),
        # a smaller survey evaluated once per call (the batch changes between calls)
        _case("ragged_once", "static", prec="mixed", n_sys=30011, n_pl_max=5, obs_lo=16, obs_hi=400),
        # population MCMC with a few thousand chains: many short dependent launches
        _case("demc_4096", "demc", prec="mixed", n_half=2048, n_pl=4, n_obs=256, n_gen=32),
        # Kepler's equation alone, in binary64
        _case("kepler_fp64", "kepler", prec="fp64", n=4194301),
        # astrometric orbits
        _case("astro_batch", "astro", prec="mixed", n_sys=200000, n_pl=2, n_obs=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Most triples (systems x planets x observations) of a drawn case, mixed and binary64.
_MOST = {"chisq": (1 << 30, 1 << 26), "grad": (1 << 28, 1 << 22), "nll": (1 << 28, 1 << 22), "gn": (1 << 28, 1 << 25),
         "ragged": (1 << 28, 1 << 25), "static": (1 << 28, 1 << 25), "astro": (1 << 28, 1 << 25)}


def draw(rng):
    kind = rng.choice(["chisq", "chisq", "chisq", "grad", "nll", "gn", "ragged", "static", "demc", "kepler", "astro"])
    prec = rng.choice(["mixed", "mixed", "fp64"])
    if kind == "kepler":
        return {"kind": kind, "prec": prec, "n": _log_int(rng, 1000, 16777216)}
    if kind == "demc":
        n_pl, n_obs = rng.randint(1, 4), _log_int(rng, 30, 400)
        n_half = min(_log_int(rng, 32, 32768), (1 << 29) // (2 * 32 * n_pl * n_obs))
        return {"kind": kind, "prec": "mixed", "n_half": n_half, "n_pl": n_pl, "n_obs": n_obs, "n_gen": 32}
    most = _MOST[kind][prec == "fp64"]
    if kind in ("ragged", "static"):
        n_pl_max, obs_hi = rng.randint(1, 7), _log_int(rng, 64, 1024)
        mean = (1 + n_pl_max) / 2 * (obs_hi - 16) / math.log(obs_hi / 16)
        return {"kind": kind, "prec": prec, "n_sys": min(_log_int(rng, 500, 262144), int(most / mean)),
                "n_pl_max": n_pl_max, "obs_lo": 16, "obs_hi": obs_hi}
    hi = {"chisq": 1048576, "grad": 262144, "nll": 262144, "gn": 262144, "astro": 1048576}[kind]
    lo = 200 if prec == "fp64" and kind in ("grad", "nll") else 16
    n_pl, n_obs = rng.randint(1, 6 if kind != "astro" else 3), _log_int(rng, 16, 1024)
    if lo == 200:
        n_pl, n_obs = rng.randint(1, 3), _log_int(rng, 16, 160)
    n_sys = max(lo, min(_log_int(rng, lo, hi), most // (n_pl * n_obs)))
    case = {"kind": kind, "prec": prec, "n_sys": n_sys, "n_pl": n_pl, "n_obs": n_obs}
    if kind != "astro":
        case["offset"] = kind != "chisq" or rng.random() < 0.5
        case["jitter"] = kind == "nll" or rng.random() < 0.5
    return case


# ------------------------------------------------------------------ inputs
def _uniform(g, lo, hi, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=F64) * (hi - lo) + lo


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=F64)


def _planets(g, n_pl, n_sys, e_max):
    P = _uniform(g, 0.0, math.log(1000.0), n_pl, n_sys).exp().sort(dim=0).values.contiguous()
    return dict(P=P, K=_uniform(g, 1.0, 100.0, n_pl, n_sys), e=_uniform(g, 0.0, e_max, n_pl, n_sys),
                omega=_uniform(g, 0.0, TWO_PI, n_pl, n_sys), M0=_uniform(g, 0.0, TWO_PI, n_pl, n_sys))


def _dense(case, g, e_max):
    """Observations (t, v, sigma) and parameter planes; system 0 is the truth behind v."""
    n_sys, n_pl, n_obs = case["n_sys"], case["n_pl"], case["n_obs"]
    t = _uniform(g, 2454000.0, 2457000.0, n_obs).sort().values
    sigma = _uniform(g, 1.0, 5.0, n_obs)
    par = _planets(g, n_pl, n_sys, e_max)
    v = sum(_velocity(t, *(par[k][j, 0] for k in ("P", "K", "e", "omega", "M0"))) for j in range(n_pl))
    d = dict(t=t, v=v + sigma * _normal(g, n_obs), sigma=sigma, **par)
    if case["offset"]:
        d["offset"] = _uniform(g, -10.0, 10.0, n_sys)
    if case["jitter"]:
        d["jitter"] = _uniform(g, 0.0, 3.0, n_sys)
    return d


def _offsets(n):
    return torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), n.cumsum(0)])


def _ragged(case, g):
    n_sys = case["n_sys"]
    n_pl = torch.randint(1, case["n_pl_max"] + 1, (n_sys,), generator=g, device=DEV)
    n_obs = _uniform(g, math.log(case["obs_lo"]), math.log(case["obs_hi"]), n_sys).exp().round().to(torch.int64)
    obs_off, pl_off = _offsets(n_obs), _offsets(n_pl)
    total, planets = int(obs_off[-1]), int(pl_off[-1])
    system = torch.repeat_interleave(torch.arange(n_sys, device=DEV, dtype=F64), n_obs)
    t = 2454000.0 + 3000.0 * ((system + _uniform(g, 0.0, 1.0, total)).sort().values - system)
    sigma = _uniform(g, 1.0, 5.0, total)
    p = {k: x[0] for k, x in _planets(g, 1, planets, 0.9).items()}
    v = _velocity(t, *(p[k][0] for k in ("P", "K", "e", "omega", "M0")))
    return dict(t=t, v=v + sigma * _normal(g, total), sigma=sigma, obs_off=obs_off, pl_off=pl_off, **p)


def _demc(case, g):
    """A population scattered by 1e-4 about the truth, as after an optimiser."""
    d = _dense(dict(case, n_sys=1, offset=False, jitter=False), g, 0.9)
    n_pl, n_half = case["n_pl"], case["n_half"]
    centre = torch.cat([d[k][:, 0] for k in ("P", "K", "e", "omega", "M0")])
    scale = 1e-4 * centre.abs().clamp(min=0.05)
    x = torch.empty(2, 5 * n_pl + 1, n_half, dtype=F64, device=DEV)
    x[:, :-1] = centre[:, None] + scale[:, None] * _normal(g, 2, 5 * n_pl, n_half)
    x[:, 2 * n_pl:3 * n_pl].clamp_(0.0, 0.95)
    x[:, -1] = 0.5 * _normal(g, 2, n_half)
    eps = torch.cat([0.1 * scale, torch.full((1,), 1e-5, dtype=F64, device=DEV)])
    return d, x, eps


def _astro(case, g):
    n_sys, n_pl, n_obs = case["n_sys"], case["n_pl"], case["n_obs"]
    t = _uniform(g, 2457000.0, 2458826.0, n_obs).sort().values
    sx, sy = _uniform(g, 0.02, 0.1, n_obs), _uniform(g, 0.02, 0.1, n_obs)
    P = _uniform(g, math.log(10.0), math.log(2000.0), n_pl, n_sys).exp().sort(dim=0).values.contiguous()
    e, M0 = _uniform(g, 0.0, 0.9, n_pl, n_sys), _uniform(g, 0.0, TWO_PI, n_pl, n_sys)
    a = _uniform(g, 0.0, math.log(100.0), n_pl, n_sys).exp()
    A, B, F, G = (a * _uniform(g, -1.0, 1.0, n_pl, n_sys) for _ in range(4))
    x, y = sx * _normal(g, n_obs), sy * _normal(g, n_obs)
    for j in range(n_pl):
        X, Y = _orbit(t, P[j, 0], e[j, 0], M0[j, 0])
        x, y = x + B[j, 0] * X + G[j, 0] * Y, y + A[j, 0] * X + F[j, 0] * Y
    return dict(t=t, x=x, y=y, sigma_x=sx, sigma_y=sy, P=P, e=e, M0=M0, A=A, B=B, F=F, G=G,
                x0=_uniform(g, -1.0, 1.0, n_sys), y0=_uniform(g, -1.0, 1.0, n_sys))


def _inputs(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    kind = case["kind"]
    if kind == "kepler":
        return dict(M=_uniform(g, 0.0, TWO_PI, case["n"]), e=_uniform(g, 0.0, 0.9, case["n"]))
    if kind in ("ragged", "static"):
        return _ragged(case, g)
    if kind == "astro":
        return _astro(case, g)
    return _dense(case, g, 0.9 if kind == "chisq" else 0.8)


def prepare(case, seed):
    if case["kind"] == "demc":
        d, x, eps = _demc(case, torch.Generator(device=DEV).manual_seed(seed))
        sampler = kp.DEMC(d["t"], d["v"], d["sigma"], x, eps, seed=seed, jump_every=10, prec=case["prec"])
        return {"case": case, "sampler": sampler, "gen": 0}
    inputs = dict(_inputs(case, seed), prec=case["prec"])
    if case["kind"] == "ragged":
        return {"case": case, "plan": kp.RaggedPlan(**inputs)}
    return {"case": case, "inputs": inputs}


_CALLS = {"chisq": kp.rv_chisq, "grad": kp.rv_chisq_grad, "nll": kp.rv_nll_grad, "gn": kp.rv_chisq_gn,
          "static": kp.rv_chisq_ragged_static, "kepler": kp.kepler_solve, "astro": kp.astro_chisq}


def run(state):
    kind = state["case"]["kind"]
    if kind == "ragged":
        return state["plan"]()
    if kind == "demc":
        n_gen, sampler = state["case"]["n_gen"], state["sampler"]
        sampler.run(state["gen"], n_gen)
        state["gen"] += n_gen
        return sampler.x, sampler.chi2, sampler.n_accept
    return _CALLS[kind](**state["inputs"])


# ------------------------------------------------------------------ floor
def work(case):
    """Bytes: every input and output once.  Operations: those of one Kepler solve and velocity in the
    leanest formulation in use (55 a triple; 136 with derivatives), and the Gram matrix's products."""
    kind = case["kind"]
    if kind == "kepler":
        return {"bytes": 24 * case["n"], "flops": 55 * case["n"]}
    if kind in ("ragged", "static"):
        span = math.log(case["obs_hi"] / case["obs_lo"])
        obs = case["n_sys"] * (case["obs_hi"] - case["obs_lo"]) / span if span > 0 else case["n_sys"] * case["obs_lo"]
        planets = case["n_sys"] * (1 + case["n_pl_max"]) / 2
        return {"bytes": 24 * obs + 40 * planets + 24 * case["n_sys"], "flops": 55 * obs * (1 + case["n_pl_max"]) / 2}
    n_pl, n_obs = case["n_pl"], case["n_obs"]
    if kind == "demc":
        chains = 2 * case["n_half"] * case["n_gen"]
        return {"bytes": chains * (5 * n_pl + 2) * 16, "flops": 55 * chains * n_pl * n_obs}
    n_sys = case["n_sys"]
    triples = n_sys * n_pl * n_obs
    if kind == "astro":
        return {"bytes": 8 * n_sys * (7 * n_pl + 3) + 40 * n_obs, "flops": 80 * triples}
    rows, npar = 5 * n_pl, 5 * n_pl + 1
    vectors = int(case["offset"]) + int(case["jitter"])
    out = {"chisq": 1, "grad": 1 + npar, "nll": 2 + npar, "gn": 1 + npar + npar * (npar + 1) // 2}[kind]
    flops = 55 * triples if kind == "chisq" else 136 * triples
    if kind == "gn":
        flops += n_sys * n_obs * (npar + 1) * (npar + 2)
    return {"bytes": 8 * n_sys * (rows + vectors + out) + 24 * n_obs, "flops": flops}


# ------------------------------------------------------------------ reference in 64 bits
def _solve(M, e):
    """E - e sin E = M for M in [-pi, pi], 0 <= e < 1, by bracketed Halley steps."""
    lo, hi = M - e, M + e
    E = M + 0.85 * e * torch.sign(M)
    for _ in range(9):
        s, c = torch.sin(E), torch.cos(E)
        f, f1 = E - e * s - M, 1.0 - e * c
        E = torch.minimum(torch.maximum(E - f * f1 / (f1 * f1 - 0.5 * f * e * s), lo), hi)
    return E


def _anomaly(t, P, M0):
    q = t / P
    phase = (q - torch.floor(q)) + M0 / TWO_PI
    return TWO_PI * (phase - torch.round(phase)), q


def _orbit(t, P, e, M0):
    M, _ = _anomaly(t, P, M0)
    E = _solve(M, e)
    return torch.cos(E) - e, torch.sqrt((1.0 - e) * (1.0 + e)) * torch.sin(E)


def _velocity(t, P, K, e, w, M0, derivatives=False):
    """v = K [cos(w + f) + e cos w] and, if asked for, its derivatives by (P, K, e, w, M0)."""
    M, q = _anomaly(t, P, M0)
    E = _solve(M, e)
    s, c, b2 = torch.sin(E), torch.cos(E), (1.0 - e) * (1.0 + e)
    b, D, cw, sw = torch.sqrt(b2), 1.0 - e * c, torch.cos(w), torch.sin(w)
    dv_dK = b * (b * cw * c - sw * s) / D
    if not derivatives:
        return K * dv_dK
    sin_wf = (sw * (c - e) + cw * b * s) / D
    dv_dM = -K * sin_wf * b / (D * D)
    dv_de = K * cw - K * sin_wf * s * (2.0 - e * c - e * e) / (b * D * D)
    return K * dv_dK, [dv_dM * (-TWO_PI) * q / P, dv_dK, dv_de, -K * b * (b * sw * c + cw * s) / D, dv_dM]


def _exact_dense(case, d):
    kind, n_sys, n_pl = case["kind"], case["n_sys"], case["n_pl"]
    derivatives = kind != "chisq"
    step = max(1, (1 << (20 if derivatives else 22)) // max(case["n_obs"], 1))
    out = []
    for i in range(0, n_sys, step):
        part = slice(i, min(n_sys, i + step))
        gamma = d["offset"][part, None] if "offset" in d else torch.zeros((), dtype=F64, device=DEV)
        s2 = d["jitter"][part, None] ** 2 if "jitter" in d else torch.zeros((), dtype=F64, device=DEV)
        r, cols = gamma - d["v"], []
        for j in range(n_pl):
            args = [d[k][j, part, None] for k in ("P", "K", "e", "omega", "M0")]
            got = _velocity(d["t"], *args, derivatives=derivatives)
            if derivatives:
                cols += got[1]
                got = got[0]
            r = r + got
        var = d["sigma"] ** 2 + s2
        w = (1.0 / var).expand_as(r)
        chi2 = (w * r * r).sum(1)
        if kind == "chisq":
            out.append((chi2,))
            continue
        cols.append(torch.ones_like(r))
        if kind == "gn":
            J = torch.stack(cols, 1)
            npar = J.shape[1]
            A = torch.matmul(J, (J * w[:, None]).transpose(1, 2).contiguous())
            a, b = torch.triu_indices(npar, npar, device=DEV)
            out.append((chi2, (J * (w * r)[:, None]).sum(2).T, A[:, a, b].T))
            continue
        rows = [(2.0 * w * r * x).sum(1) for x in cols]
        if kind == "nll":
            jitter = d["jitter"][part] if "jitter" in d else torch.zeros_like(chi2)
            chi2 = chi2 + torch.log(var).expand_as(r).sum(1)
            rows.append(2.0 * jitter * (w - (w * r) ** 2).sum(1))
        out.append((chi2, torch.stack(rows)))
    return tuple(torch.cat(x, -1) for x in zip(*out))


def _exact_ragged(case, d):
    n_sys = case["n_sys"]
    n_obs, n_pl = d["obs_off"].diff(), d["pl_off"].diff()
    system = torch.repeat_interleave(torch.arange(n_sys, device=DEV), n_obs)
    chi2 = torch.zeros(n_sys, dtype=F64, device=DEV)
    for i in range(0, system.numel(), 1 << 22):
        part = slice(i, i + (1 << 22))
        which, t = system[part], d["t"][part]
        r = -d["v"][part]
        for j in range(case["n_pl_max"]):
            here = j < n_pl[which]
            p = torch.where(here, d["pl_off"][which] + j, 0)
            r = r + here * _velocity(t, *(d[k][p] for k in ("P", "K", "e", "omega", "M0")))
        chi2.index_add_(0, which, (r / d["sigma"][part]) ** 2)
    return chi2


def _exact_astro(case, d):
    out, step = [], max(1, (1 << 22) // case["n_obs"])
    for i in range(0, case["n_sys"], step):
        part = slice(i, i + step)
        rx, ry = d["x0"][part, None] - d["x"], d["y0"][part, None] - d["y"]
        for j in range(case["n_pl"]):
            P, e, M0, A, B, F, G = (d[k][j, part, None] for k in ("P", "e", "M0", "A", "B", "F", "G"))
            X, Y = _orbit(d["t"], P, e, M0)
            rx, ry = rx + B * X + G * Y, ry + A * X + F * Y
        out.append(((rx / d["sigma_x"]) ** 2 + (ry / d["sigma_y"]) ** 2).sum(1))
    return torch.cat(out)


def exact(case, seed):
    """What run() returns, in plain 64-bit torch (the sampler's states depend on its random draws: none)."""
    kind = case["kind"]
    if kind == "demc":
        return None
    d = _inputs(case, seed)
    if kind == "kepler":
        turns = torch.round(d["M"] / TWO_PI)
        return _solve(d["M"] - TWO_PI * turns, d["e"]) + TWO_PI * turns
    if kind in ("ragged", "static"):
        return _exact_ragged(case, d)
    if kind == "astro":
        return _exact_astro(case, d)
    got = _exact_dense(case, d)
    return got[0] if kind == "chisq" else got
