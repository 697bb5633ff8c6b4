"""Binary64 entry points at periods near the ends of binary64: where (t - t0)/P
overflows the result is NaN at every eccentricity, and at the epoch itself, where the
phase is M0/(2 pi) for every period, values and derivatives are finite."""
import numpy as np
import pytest
import torch

import paper_0812_2976_amd as kp

pytestmark = pytest.mark.gpu
TINY = [5e-324, 1e-310, 2.0 ** -1023, 1e-307]


def _gpu(x):
    return torch.as_tensor(np.ascontiguousarray(x), device="cuda")


def _args(P, e, t):
    one = np.ones((1, len(P)))
    return dict(t=_gpu(np.asarray(t, dtype=np.float64)), P=_gpu(one * P), K=_gpu(50 * one), e=_gpu(e * one),
                omega=_gpu(0.7 * one), M0=_gpu(1.1 * one))


@pytest.mark.parametrize("e", [0.3, 0.88, 0.95, 0.9995])
def test_overflowing_phase_is_nan(e):
    """Velocities, positions and chi-squares are NaN exactly where thirty plain steps make them NaN."""
    P = np.array(TINY + [1e-300, 1.0, 1e300])
    d = _args(P, e, [0.0, 1e-8, 2456000.0])
    a, b = (kp.rv_model(**d, prec="fp64", opts=o).cpu().numpy() for o in (None, {"fixed_iter": 30}))
    assert np.isnan(b).any() and np.isfinite(b[:, 0]).all()
    assert np.array_equal(np.isnan(a), np.isnan(b))
    n, nan = len(P), np.isnan(b).any(1)
    obs = dict(v=_gpu(np.zeros(3)), sigma=_gpu(np.ones(3)))
    got = [kp.rv_chisq(**d, **obs, prec="fp64"), kp.rv_chisq_grad(**d, **obs, prec="fp64")[0],
           kp.rv_nll_grad(**d, **obs, prec="fp64")[0], kp.rv_chisq_gn(**d, **obs, prec="fp64")[0],
           kp.rv_chisq_ragged_static(**{k: x[0] for k, x in d.items() if k != "t"}, t=d["t"].repeat(n),
                                     v=_gpu(np.zeros(3 * n)), sigma=_gpu(np.ones(3 * n)), obs_off=_gpu(3 * np.arange(n + 1)),
                                     pl_off=_gpu(np.arange(n + 1)), prec="fp64")]
    for chi2 in got:
        assert np.array_equal(np.isnan(chi2.cpu().numpy()), nan)
    s = {k: d[k] for k in ("t", "P", "e", "M0")}
    s.update({k: torch.ones_like(d["P"]) for k in "ABFG"})
    xy, xy30 = (kp.astro_model(**s, prec="fp64", opts=o).cpu().numpy() for o in (None, {"fixed_iter": 30}))
    assert np.array_equal(np.isnan(xy), np.isnan(xy30)) and np.isnan(xy).any()


@pytest.mark.parametrize("n_obs", [3, 70, 200])
@pytest.mark.parametrize("call", ["grad", "nll", "gn"])
@pytest.mark.parametrize("opts", [None, {"fixed_iter": 30}])
def test_derivatives_at_the_epoch(call, n_obs, opts):
    """All observations at the epoch: nothing depends on P, so every output is the one for P = 1 and the
    derivative by P is zero."""
    f = {"grad": kp.rv_chisq_grad, "nll": kp.rv_nll_grad, "gn": kp.rv_chisq_gn}[call]
    rng = np.random.default_rng(3)
    obs = dict(v=_gpu(rng.normal(0.0, 30.0, n_obs)), sigma=_gpu(rng.uniform(1.0, 5.0, n_obs)))
    tiny, one = (f(**_args(P, 0.4, np.zeros(n_obs)), **obs, prec="fp64", opts=opts)
                 for P in (np.array(TINY), np.ones(len(TINY))))
    for a, b in zip(tiny, one):
        assert torch.isfinite(a).all() and torch.equal(a, b)
    assert (tiny[1][0] == 0).all() and (tiny[1][1] != 0).all()
