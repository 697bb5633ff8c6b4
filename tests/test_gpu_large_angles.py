"""Angles far from [-pi, pi].  Binary64 entry points at such an M0: a system's result is
the one for its M0 reduced by whole turns, bit for bit, and the other systems' results
stay.  The standalone solve at any finite M, in both precisions."""
from fractions import Fraction

import mpmath as mp
import numpy as np
import pytest
import torch

import paper_0812_2976_amd as kp
from tests import workloads as W

pytestmark = pytest.mark.gpu
U = 2.0 ** -53
TWO_PI_HI, TWO_PI_LO = 6.283185307179586232, 2.4492935982947064e-16
M0_LARGE = [-1e4, 3e10, 1e15, -1e17, 1e25, 1e31, -1e33, 1e37, 1e60, -1e300, 1.7976931348623157e308]


def _gpu(x):
    return torch.as_tensor(np.ascontiguousarray(x), device="cuda")


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _reduced(x):
    """x less whole turns, the kernels' repeated two-part subtraction."""
    while True:
        n = float(np.rint(x * 0.15915494309189533576888376337251))
        x = _fma(-n, TWO_PI_LO, _fma(-n, TWO_PI_HI, x))
        if abs(x) <= 3.1416:
            return x


def _planes(wl, e):
    """The workload with one planet of system 1 + 2 i at M0_LARGE[i] and eccentricity e, and the same reduced."""
    far, near = wl.M0.copy(), wl.M0.copy()
    for i, x in enumerate(M0_LARGE):
        s, j = 1 + 2 * i, i % far.shape[0]
        wl.e[j, s] = e
        far[j, s], near[j, s] = x, _reduced(x)
    return far, near


CALLS = {"chisq": kp.rv_chisq, "grad": kp.rv_chisq_grad, "nll": kp.rv_nll_grad, "gn": kp.rv_chisq_gn, "model": kp.rv_model}


def _same(a, b):
    a, b = (x if isinstance(x, tuple) else (x,) for x in (a, b))
    for x, y in zip(a, b):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("e", [0.0, 0.6, 0.88, 0.95, 0.9995])
@pytest.mark.parametrize("call", sorted(CALLS))
@pytest.mark.parametrize("n_obs", [70, 300])
def test_m0_of_any_size(call, e, n_obs):
    wl = W.dense("c1", n_sys=2 * len(M0_LARGE) + 1, n_pl=3, n_obs=n_obs, seed=23)
    far, near = _planes(wl, e)
    g = W.to_gpu(wl, torch.device("cuda", 0))
    if call == "model":
        g = {k: x for k, x in g.items() if k not in ("v", "sigma", "jitter")}
    a, b = (CALLS[call](**dict(g, M0=_gpu(m)), prec="fp64") for m in (far, near))
    _same(a, b)
    if call == "model":
        assert (a.abs() <= 2.0 * _gpu(wl.K.sum(0))[:, None]).all()


@pytest.mark.parametrize("e", [0.6, 0.95])
def test_m0_of_any_size_ragged(e):
    wl = W.dense("c1", n_sys=2 * len(M0_LARGE) + 1, n_pl=3, n_obs=70, seed=23)
    far, near = _planes(wl, e)
    n = wl.M0.shape[1]
    flat = lambda x: _gpu(x.T.ravel())
    args = dict(t=_gpu(np.tile(wl.t, n)), v=_gpu(np.tile(wl.v, n)), sigma=_gpu(np.tile(wl.sigma, n)),
                obs_off=_gpu(70 * np.arange(n + 1)), P=flat(wl.P), K=flat(wl.K), e=flat(wl.e), omega=flat(wl.w),
                pl_off=_gpu(3 * np.arange(n + 1)), prec="fp64")
    _same(*(kp.rv_chisq_ragged_static(**args, M0=flat(m)) for m in (far, near)))
    _same(*(kp.RaggedPlan(**args, M0=flat(m))() for m in (far, near)))


@pytest.mark.parametrize("e", [0.6, 0.95])
@pytest.mark.parametrize("n_obs", [70, 300])
def test_m0_of_any_size_astro(e, n_obs):
    wl = W.astro(2 * len(M0_LARGE) + 1, 2, n_obs, seed=29)
    far, near = _planes(wl, e)
    g = W.astro_to_gpu(wl, torch.device("cuda", 0))
    _same(*(kp.astro_chisq(**dict(g, M0=_gpu(m)), prec="fp64") for m in (far, near)))
    g = {k: g[k] for k in ("t", "P", "e", "A", "B", "F", "G", "x0", "y0", "t0")}
    _same(*(kp.astro_model(**g, M0=_gpu(m), prec="fp64") for m in (far, near)))


@pytest.mark.parametrize("m0", [1e17, 1e33, 1e300])
def test_m0_of_any_size_sampler(m0):
    """A population whose M0 have run away: every stored chi-square is the one of the stored state."""
    n_half, n_pl, n_obs = 40, 2, 100
    wl = W.dense("c4", n_sys=1, n_pl=n_pl, n_obs=n_obs, seed=31)
    p = np.concatenate([np.concatenate([getattr(wl, k)[:, 0] for k in ("P", "K", "e", "w", "M0")]), [0.0]])
    x = p[None, :, None] * (1.0 + 1e-4 * np.random.default_rng(1).standard_normal((2, p.size, n_half)))
    x[:, 4 * n_pl:5 * n_pl] *= m0
    s = kp.DEMC(_gpu(wl.t), _gpu(wl.v), _gpu(wl.sigma), _gpu(x), _gpu(1e-8 * np.abs(p) + 1e-9), seed=7, prec="fp64")
    s.generations(0, 4)
    stored, again = s.chi2.clone(), s.chisq()
    assert torch.isfinite(again).all()
    # the same terms, at most n_obs of them and none negative, summed in another order
    assert ((stored - again).abs() <= 2.0 ** -52 * n_obs * again).all()


def _root(M, e):
    """(E, E less M's whole turns) to 40 digits: Newton's steps on the mean anomaly reduced with that many more."""
    with mp.workdps(70):
        x = mp.mpf(M)
        turns = 2 * mp.pi * mp.nint(x / (2 * mp.pi))
        m, e = x - turns, mp.mpf(e)
        lo, hi = m - e, m + e
        E = m + mp.mpf("0.85") * e * mp.sign(m)
        for _ in range(200):
            f = E - e * mp.sin(E) - m
            if f > 0:
                hi = min(hi, E)
            else:
                lo = max(lo, E)
            step = E - f / (1 - e * mp.cos(E))
            step = step if lo <= step <= hi else (lo + hi) / 2
            if abs(step - E) < mp.mpf(10) ** -45:
                break
            E = step
        return E + turns, E


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_kepler_solve_of_any_finite_m(prec):
    """|M| < 2^54 against the 40-digit root: the rounding of sin E (two of its ulps), of the reduced mean
    anomaly and of E (mixed: the bound of a binary32 solve with |Mr|, |Er| <= pi + 1); above, E is M itself."""
    rng = np.random.default_rng(77)
    mag = np.concatenate([10.0 ** rng.uniform(3, 16.25, 300), 10.0 ** rng.uniform(13, 16.25, 100)])
    odd = (2.0 * np.rint(10.0 ** rng.uniform(3, 15, 100)) + 1.0) * np.pi
    M = np.concatenate([mag * rng.choice([-1, 1], mag.size), odd, -odd, [367531048600891.44]])
    M = M[np.abs(M) < 2.0 ** 54]
    e = np.where(rng.random(M.size) < 0.7, rng.uniform(0.0, 0.9, M.size), rng.uniform(0.9, 0.9999, M.size))
    e[-1] = 0.8737577320354846
    E = kp.kepler_solve(_gpu(M), _gpu(e), prec=prec).cpu().numpy()
    for x, ei, got in zip(M, e, E):
        ref, Er = _root(x, ei)
        D, s = float(1 - ei * mp.cos(Er)), abs(float(mp.sin(Er)))
        if prec == "fp64":
            tol = (4 * U * ei * s + 2 * U * abs(float(Er)) + 4 * np.pi * U + abs(x) * 2.0 ** -105) / D + 4 * U * abs(x)
        else:
            u = 2.0 ** -24
            tol = 8 * u * (2 * np.pi + 1) / D + 2 * u * (np.pi + 1) + 4 * u * 0.015 + 1e-9 + 4 * U * abs(x)
        assert abs(float(mp.mpf(got) - ref)) <= tol, (x, ei, got, float(ref))
    big = np.concatenate([[2.0 ** 54, 1e17, 1e25, 1e60, 1e300, 1.7976931348623157e308],
                          10.0 ** rng.uniform(16.3, 308, 1000)])
    big = np.concatenate([big, -big])
    eb = rng.uniform(0.0, 0.9999, big.size)
    assert np.array_equal(kp.kepler_solve(_gpu(big), _gpu(eb), prec=prec).cpu().numpy(), big)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("opts", [None, {"fixed_iter": 30}, {"fixed_iter": -1}])
def test_kepler_solve_with_one_large_m(prec, opts):
    """A large M among ordinary ones changes no other pair's root."""
    rng = np.random.default_rng(78)
    n = 5000
    M, e = _gpu(rng.uniform(-20.0, 20.0, n)), _gpu(rng.uniform(0.0, 0.9999, n))
    clean = kp.kepler_solve(M, e, prec=prec, opts=opts)
    for at, x in ((0, 1e15), (1023, -1e300), (n - 1, 9e9)):
        far = M.clone()
        far[at] = x
        E = kp.kepler_solve(far, e, prec=prec, opts=opts)
        keep = torch.arange(n, device="cuda") != at
        assert torch.equal(E[keep], clean[keep]) and abs(E[at].item() - x) <= 1.0 + 2.0 ** -52 * abs(x)
