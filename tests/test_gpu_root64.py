"""The binary64 path at its default step count: the root from the binary32 start
and binary64 steps (kep_root64.h), at the edges of the table, of the knots and of
the chunk counts, against the oracle and against thirty plain Danby steps
(fixed_iter = 30)."""
import numpy as np
import pytest
import torch

import oracle
import paper_0812_2976_amd as kp
from tests import workloads as W

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _gpu(x):
    return torch.as_tensor(np.ascontiguousarray(x), device="cuda")


def _pairs(kind):
    rng = np.random.default_rng(64)
    if kind == "edges":           # table rows and bands, both sides of its end, knots and half knots of the root
        e = np.concatenate([[0.0, 0.7, 0.85, 0.9], np.nextafter([0.7, 0.85, 0.9], 0.0), np.nextafter([0.7, 0.85, 0.9], 1.0),
                            [0.95, 0.975, 0.9755, 0.99, 0.9955, 0.9999]])
        E = np.arange(-402, 403) / 128.0
        E = E[np.abs(E) <= np.pi]
        ee, EE = np.meshgrid(e, E)
        M, e = (EE - ee * np.sin(EE)).ravel(), ee.ravel()
        return np.concatenate([M, [0.0, -0.0, np.pi, -np.pi, 2 * np.pi]]), np.concatenate([e, np.full(5, 0.9)])
    if kind == "near periapsis":
        return 10.0 ** rng.uniform(-14, -1, 4000) * rng.choice([-1, 1], 4000), 1.0 - 10.0 ** rng.uniform(-6, 0, 4000)
    return rng.uniform(-100.0, 100.0, 5000), rng.uniform(0.0, 0.9, 5000)      # other branches


@pytest.mark.parametrize("kind", ["edges", "near periapsis", "branches"])
def test_kepler_root64(kind):
    """|dE| <= (4 u e |sin E| + 2 u |M|) / (1 - e cos E) + 4 u |E|, u = 2^-53: the rounding of sin E
    (two of its ulps), of the reduced mean anomaly, and of E, with M on the input's branch."""
    M, e = _pairs(kind)
    ref = oracle.kepler(M, e)
    E = kp.kepler_solve(_gpu(M), _gpu(e), prec="fp64").cpu().numpy()
    tol = (4 * U * e * np.abs(np.sin(ref)) + 2 * U * np.abs(M)) / (1.0 - e * np.cos(ref)) + 4 * U * np.abs(ref)
    assert np.all(np.abs(E - ref) <= tol), np.max(np.abs(E - ref) / np.maximum(tol, 1e-300))


@pytest.mark.parametrize("n_sys,n_pl,n_obs,e_range", [(1, 1, 1, (0.0, 0.9)), (37, 8, 64, (0.0, 0.9)),
                                                      (130, 2, 65, (0.85, 0.95)), (65, 3, 129, (0.0, 0.99)),
                                                      (41, 5, 256, (0.9, 0.999)), (5, 1, 257, (0.0, 0.9)),
                                                      (3, 4, 1000, (0.0, 0.9))])
def test_chisq_and_model_against_thirty_steps(n_sys, n_pl, n_obs, e_range):
    """Both within the stated binary64 targets of the oracle (chi2 relative 1e-12, velocities 1e-9 m/s),
    so within twice that of each other."""
    wl = W.dense("c1", n_sys=n_sys, n_pl=n_pl, n_obs=n_obs, seed=11, jitter=True, e_range=e_range)
    g = W.to_gpu(wl, torch.device("cuda", 0))
    chi2 = kp.rv_chisq(**g, prec="fp64").cpu().numpy()
    ref = oracle.chisq(W.oracle_dense(wl))
    thirty = kp.rv_chisq(**g, prec="fp64", opts={"fixed_iter": 30}).cpu().numpy()
    assert W.rel_err_chi2(chi2, ref).max() <= 1e-12
    assert W.rel_err_chi2(chi2, thirty).max() <= 2e-12
    g = {k: x for k, x in g.items() if k not in ("v", "sigma", "jitter")}
    v = kp.rv_model(**g, prec="fp64")
    assert np.abs(v.cpu().numpy() - oracle.rv_model(W.oracle_dense(wl))).max() <= 1e-9
    assert (v - kp.rv_model(**g, prec="fp64", opts={"fixed_iter": 30})).abs().max().item() <= 2e-9


def test_periods_at_the_ends_of_binary64():
    """A period whose reciprocal overflows or is subnormal takes the same values as thirty plain steps;
    at the epoch itself the phase is M0 / (2 pi) for every period."""
    P = np.array([[5e-324, 1e-310, 2.0 ** -1023, 1e-300, 1e300, 1.7e308]])
    one = np.ones_like(P)
    args = dict(t=_gpu(np.array([0.0, 0.0, 0.0])), P=_gpu(P), K=_gpu(50 * one), e=_gpu(0.3 * one), omega=_gpu(0.7 * one),
                M0=_gpu(1.1 * one))
    a = kp.rv_model(**args, prec="fp64").cpu().numpy()
    b = kp.rv_model(**args, prec="fp64", opts={"fixed_iter": 30}).cpu().numpy()
    assert np.all(np.isfinite(a)) and np.abs(a - b).max() <= 2e-9
    args["t"] = _gpu(np.array([0.0, 1.0, 2456000.0]))
    a = kp.rv_model(**args, prec="fp64").cpu().numpy()
    b = kp.rv_model(**args, prec="fp64", opts={"fixed_iter": 30}).cpu().numpy()
    assert np.array_equal(np.isnan(a), np.isnan(b))


@pytest.mark.parametrize("field", ["P", "K", "e", "omega", "M0"])
def test_invalid_planets_are_nan_alone(field):
    wl = W.dense("c1", n_sys=20, n_pl=2, n_obs=70, seed=3)
    g = W.to_gpu(wl, torch.device("cuda", 0))
    clean = kp.rv_chisq(**g, prec="fp64")
    g[field] = g[field].clone()
    g[field][1, 7] = float("nan") if field != "e" else 1.0
    chi2 = kp.rv_chisq(**g, prec="fp64")
    keep = torch.arange(20, device="cuda") != 7
    assert torch.isnan(chi2[7]) and torch.equal(chi2[keep], clean[keep])
