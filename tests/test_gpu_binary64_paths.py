"""The binary64 gradient, likelihood, Gauss-Newton products, ragged, sampler and
astrometric kernels at the default step count: chunk and planet-count edges
against the oracle, and against thirty plain Danby steps (fixed_iter = 30)."""
import numpy as np
import pytest
import torch

import oracle
import paper_0812_2976_amd as kp
import synth
from tests import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _gpu(x):
    return torch.as_tensor(np.ascontiguousarray(x), device=DEV)


SHAPES = [(1, 1, 1, (0.0, 0.9)), (3, 8, 63, (0.0, 0.9)), (70, 2, 64, (0.0, 0.9)), (33, 4, 65, (0.85, 0.95)),
          (130, 3, 128, (0.0, 0.9)), (9, 5, 129, (0.0, 0.9)), (17, 7, 300, (0.0, 0.9))]


@pytest.mark.parametrize("n_sys,n_pl,n_obs,e_range", SHAPES)
def test_gradients_and_products(n_sys, n_pl, n_obs, e_range):
    """The stated binary64 targets: gradient rows within 1e-6 (|g| + 1e-6 S_r) of the oracle, J^T W J
    within 1e-9 of sqrt(C_aa C_bb); thirty plain steps give the same within twice that."""
    wl = W.dense("c4", n_sys=n_sys, n_pl=n_pl, n_obs=n_obs, seed=5, jitter=True, e_range=e_range)
    g, d = W.to_gpu(wl, torch.device(DEV, 0)), W.oracle_dense(wl)
    ref, (_, _, s_r, _) = oracle.chisq_grad(d), oracle.chisq_grad_scales(d)
    for opts in (None, {"fixed_iter": 30}):
        chi2, grad = (x.cpu().numpy() for x in kp.rv_chisq_grad(**g, prec="fp64", opts=opts))
        assert W.rel_err_chi2(chi2, ref[0]).max() <= 1e-12
        assert np.all(np.abs(grad - ref[1]) <= 1e-6 * (np.abs(ref[1]) + 1e-6 * s_r))
        nll, gn = (x.cpu().numpy() for x in kp.rv_nll_grad(**g, prec="fp64", opts=opts))
        assert np.all(np.abs(gn[:-1] - ref[1]) <= 1e-6 * (np.abs(ref[1]) + 1e-6 * s_r))
        n_ref, g_ref = oracle.nll_grad(d)[:2]
        assert np.abs(nll - n_ref).max() <= 1e-12 * np.abs(n_ref).max() + 1e-10
        assert np.abs(gn[-1] - g_ref[-1]).max() <= 1e-9 * np.abs(g_ref[-1]).max()
        _, jtwr, jtwj = (x.cpu().numpy() for x in kp.rv_chisq_gn(**g, prec="fp64", opts=opts))
        _, r_ref, c_ref = oracle.gn(d)
        npar = 5 * n_pl + 1
        a, b = np.triu_indices(npar)
        diag = c_ref[[i for i in range(len(a)) if a[i] == b[i]]]
        assert np.all(np.abs(jtwj - c_ref) <= 1e-9 * np.sqrt(diag[a] * diag[b]))
        assert np.all(np.abs(jtwr - r_ref) <= 1e-9 * np.sqrt(diag * np.maximum(ref[0], 1.0)))


@pytest.mark.parametrize("n_obs", [0, 1, 64, 65, 193, 256, 257, 520])
def test_ragged_equals_dense(n_obs):
    """Systems of one size in a CSR batch (a last batch of 1 to 4 systems) equal the dense kernel's, but
    for the order of their sums; plan, direct and plan-free calls agree bit for bit."""
    for n_sys in (1, 6, 4099 if n_obs == 65 else 7):
        wl = W.dense("c1", n_sys=n_sys, n_pl=3, n_obs=max(n_obs, 1), seed=8)
        t, v, s = (x[:n_obs] for x in (wl.t, wl.v, wl.sigma))
        csr = dict(t=_gpu(np.tile(t, n_sys)), v=_gpu(np.tile(v, n_sys)), sigma=_gpu(np.tile(s, n_sys)),
                   obs_off=_gpu(np.arange(n_sys + 1, dtype=np.int64) * n_obs), pl_off=_gpu(np.arange(n_sys + 1, dtype=np.int64) * 3),
                   **{k: _gpu(x.T.ravel()) for k, x in (("P", wl.P), ("K", wl.K), ("e", wl.e), ("omega", wl.w), ("M0", wl.M0))})
        dense = kp.rv_chisq(_gpu(t), _gpu(v), _gpu(s), *(_gpu(x) for x in (wl.P, wl.K, wl.e, wl.w, wl.M0)), prec="fp64")
        plan = kp.RaggedPlan(**csr, prec="fp64")
        got = plan()
        assert torch.equal(got, plan.direct()) and torch.equal(got, kp.rv_chisq_ragged_static(**csr, prec="fp64"))
        assert W.rel_err_chi2(got.cpu().numpy(), dense.cpu().numpy()).max() <= 1e-13
        thirty = kp.rv_chisq_ragged_static(**csr, prec="fp64", opts={"fixed_iter": 30})
        assert W.rel_err_chi2(got.cpu().numpy(), thirty.cpu().numpy()).max() <= 2e-12


@pytest.mark.parametrize("n_sys,n_pl,n_obs,e_range", [(1, 1, 1, (0.0, 0.9)), (70, 2, 128, (0.0, 0.9)),
                                                      (19, 8, 65, (0.85, 0.95)), (40, 3, 300, (0.9, 0.999))])
def test_astrometry_against_thirty_steps(n_sys, n_pl, n_obs, e_range):
    """chi2 within the stated 1e-12 of each, so 2e-12 of each other."""
    wl = synth.astro(n_sys=n_sys, n_pl=n_pl, n_obs=n_obs, e_range=e_range)
    cols = {k: _gpu(getattr(wl, k)) for k in ("t", "P", "e", "M0", "A", "B", "F", "G", "x0", "y0")}
    obs = dict(x=_gpu(wl.noise_x), y=_gpu(wl.noise_y), sigma_x=_gpu(wl.sx), sigma_y=_gpu(wl.sy))
    a = kp.astro_chisq(**cols, **obs, prec="fp64").cpu().numpy()
    b = kp.astro_chisq(**cols, **obs, prec="fp64", opts={"fixed_iter": 30}).cpu().numpy()
    assert W.rel_err_chi2(a, b).max() <= 2e-12
    amp = sum(cols[k].abs() for k in "ABFG") / (1 - cols["e"])
    x = kp.astro_model(**cols, prec="fp64") - kp.astro_model(**cols, prec="fp64", opts={"fixed_iter": 30})
    assert (x.abs().amax(dim=(1, 2)) <= 2e-11 * amp.sum(0)).all()


@pytest.mark.parametrize("n_obs", [1, 64, 129, 300, 600])
def test_sampler_against_thirty_steps(n_obs):
    """The same proposals; a decision can only differ where the acceptance margin is within the
    chi-square's rounding, which no chain of this seed is."""
    wl = W.dense("c1", n_sys=1, n_pl=2, n_obs=n_obs, seed=4)
    x, eps = synth.demc_population({k: getattr(wl, k)[:, 0] for k in ("P", "K", "e", "w", "M0")}, 40, seed=4)
    runs = []
    for opts in (None, {"fixed_iter": 30}):
        s = kp.DEMC(_gpu(wl.t), _gpu(wl.v), _gpu(wl.sigma), _gpu(x), _gpu(eps), seed=9, prec="fp64", opts=opts)
        s.generations(0, 3)
        s.run(3, 9)
        runs.append(s)
    assert torch.equal(runs[0].n_accept, runs[1].n_accept) and torch.equal(runs[0].x, runs[1].x)
    assert W.rel_err_chi2(runs[0].chi2.cpu().numpy(), runs[1].chi2.cpu().numpy()).max() <= 2e-12
