"""Chunk counts and last groups of the mixed gradient and Gauss-Newton kernels
(one to four chunks of 64 observations, several groups with a shorter last one),
and the full and last rounds of batches, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_0812_2976_amd as kp
import synth
from tests import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pl", [1, 4, 5, 8])
@pytest.mark.parametrize("n_obs", [64, 129, 192, 193, 257, 385, 449, 512])
def test_gradient_and_products(n_pl, n_obs):
    """The stated targets: gradient rows within 1e-6 max(|g|, S_r), J^T W J within 1e-5 of
    sqrt(C_aa C_bb), chi2 relative 1e-5."""
    wl = W.dense("c4", n_sys=40, n_pl=n_pl, n_obs=n_obs, seed=n_obs, jitter=True)
    g, d = W.to_gpu(wl, torch.device("cuda", 0)), W.oracle_dense(wl)
    c_ref, g_ref = oracle.chisq_grad(d)
    s_r = oracle.chisq_grad_scales(d)[2]
    for call in (kp.rv_chisq_grad, kp.rv_nll_grad):
        chi2, grad = (x.cpu().numpy() for x in call(**g))
        assert np.all(np.abs(grad[:5 * n_pl + 1] - g_ref) <= 1e-6 * np.maximum(np.abs(g_ref), s_r))
        if call is kp.rv_chisq_grad:
            assert W.rel_err_chi2(chi2, c_ref).max() <= 1e-5
    chi2, jtwr, jtwj = (x.cpu().numpy() for x in kp.rv_chisq_gn(**g))
    _, _, j_ref = oracle.gn(d)
    a, b = np.triu_indices(5 * n_pl + 1)
    diag = j_ref[a == b]
    assert np.all(np.abs(jtwj - j_ref) <= 1e-5 * np.sqrt(diag[a] * diag[b]))
    assert np.all(np.abs(2 * jtwr - g_ref) <= 1e-6 * np.maximum(np.abs(g_ref), s_r))
    assert W.rel_err_chi2(chi2, c_ref).max() <= 1e-5


@pytest.mark.parametrize("n_sys", [1, 255, 5119, 5121, 81919, 81921, 100003, 163841])
def test_every_system_once(n_sys):
    """Batches of full and last rounds cover every system exactly once: equal parameters give equal
    results everywhere, for every kernel that hands out batches."""
    wl = W.dense("c4", n_sys=1, n_pl=2, n_obs=20, seed=1)
    t, v, s = (torch.as_tensor(x, device="cuda") for x in (wl.t, wl.v, wl.sigma))
    par = [torch.as_tensor(x, device="cuda").expand(2, n_sys).contiguous() for x in (wl.P, wl.K, wl.e, wl.w, wl.M0)]
    nan = float("nan")
    for prec in ("mixed", "fp64"):
        out = torch.full((n_sys,), nan, dtype=torch.float64, device="cuda")
        kp.rv_chisq(t, v, s, *par, prec=prec, out=out)
        assert torch.all(out == out[0]), prec
        grad = torch.full((11, n_sys), nan, dtype=torch.float64, device="cuda")
        out.fill_(nan)
        kp.rv_chisq_grad(t, v, s, *par, prec=prec, out=out, grad=grad)
        assert torch.all(out == out[0]) and torch.all(grad == grad[:, :1]), prec
        if n_sys <= 100003:
            model = torch.full((n_sys, 20), nan, dtype=torch.float64, device="cuda")
            kp.rv_model(t, *par, prec=prec, out=model)
            assert torch.all(model == model[:1]), prec
        out.fill_(nan)
        ab = [x * 0.1 for x in par[1:2]] * 4
        kp.astro_chisq(t, v, v, s, s, par[0], par[2], par[4], *ab, prec=prec, out=out)
        assert torch.all(out == out[0]), prec


@pytest.mark.parametrize("n_sys,n_pl,n_obs", [(20000, 8, 3), (20000, 8, 65), (9000, 7, 128), (1, 1, 1), (40000, 1, 64)])
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_astrometry_records(n_sys, n_pl, n_obs, prec):
    """Records built over (planet, system) pairs, more than 64 of them in a one-wavefront block, and chunks
    whose last lanes are past the end: a system's result does not depend on the batch it is in."""
    wl = synth.astro(n_sys=n_sys, n_pl=n_pl, n_obs=n_obs, e_range=(0.0, 0.95))
    obs = {k: torch.as_tensor(x, device="cuda") for k, x in
           dict(t=wl.t, x=wl.noise_x, y=wl.noise_y, sigma_x=wl.sx, sigma_y=wl.sy).items()}
    cols = {k: torch.as_tensor(getattr(wl, k), device="cuda") for k in ("P", "e", "M0", "A", "B", "F", "G", "x0", "y0")}
    chi2 = kp.astro_chisq(**obs, **cols, prec=prec)
    assert torch.isfinite(chi2).all()
    assert torch.equal(chi2, kp.astro_chisq(**obs, **cols, prec=prec, opts={"block_threads": 64}))
    few = {k: x[..., -5:].contiguous() for k, x in cols.items()}
    assert torch.equal(chi2[-5:], kp.astro_chisq(**obs, **few, prec=prec))
    cols["G"][n_pl - 1, n_sys // 2] = float("nan")
    bad = kp.astro_chisq(**obs, **cols, prec=prec)
    keep = torch.arange(n_sys, device="cuda") != n_sys // 2
    assert torch.isnan(bad[n_sys // 2]) and torch.equal(bad[keep], chi2[keep])
