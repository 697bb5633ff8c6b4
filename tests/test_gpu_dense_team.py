"""The dense chi-square's split of observations over wavefronts (teams) and chunk
counts at their edges: against the oracle, and equal, but for the order of
binary64 sums, to the same observations given to one wavefront (block_threads =
64 and at most 256 observations at a time)."""
import numpy as np
import pytest
import torch

import oracle
import paper_0812_2976_amd as kp
from tests import workloads as W

pytestmark = pytest.mark.gpu

# observations at the chunk, group and team edges; system counts from one to several rounds of batches
SHAPES = [(1, 64), (1, 4097), (3, 129), (5, 192), (2, 193), (3, 257), (70, 321), (40, 512), (300, 513), (33, 1024),
          (9, 1025), (2500, 300), (2500, 65), (9, 4500), (6000, 128), (6000, 1)]


@pytest.mark.parametrize("n_sys,n_obs", SHAPES)
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_split_over_wavefronts(n_sys, n_obs, prec):
    n_pl = 1 + (n_sys + n_obs) % 8
    wl = W.dense("c1", n_sys=n_sys, n_pl=n_pl, n_obs=n_obs, seed=n_obs, jitter=True)
    g = W.to_gpu(wl, torch.device("cuda", 0))
    chi2 = kp.rv_chisq(**g, prec=prec)
    obs = ("t", "v", "sigma")
    parts = sum(kp.rv_chisq(**{k: x[i:i + 256] if k in obs else x for k, x in g.items()}, prec=prec,
                            opts={"block_threads": 64}) for i in range(0, n_obs, 256))
    # each sum of at most n_obs positive terms in either order
    assert ((chi2 - parts).abs() <= 2.0 ** -52 * n_obs * parts).all()
    few = min(n_sys, 64)
    ref = oracle.chisq(W.oracle_dense(wl), 0, few)[:few]
    err = np.abs(chi2[:few].cpu().numpy() - ref)
    dv = 1e-4 if prec == "mixed" else 1e-12      # few observations: the velocity's error through chi2 (|dv| <= dv m/s)
    bound = (1e-5 if prec == "mixed" else 1e-12) * np.maximum(ref, 1.0) + 2 * dv * np.sqrt(ref * n_obs) + dv * dv * n_obs
    assert np.all(err <= bound)


@pytest.mark.parametrize("where", ["observation", "jitter", "offset", "planet"])
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_team_domain(where, prec):
    wl = W.dense("c4", n_sys=30, n_pl=2, n_obs=700, seed=2, jitter=True)
    g = W.to_gpu(wl, torch.device("cuda", 0))
    clean = kp.rv_chisq(**g, prec=prec)
    if where == "observation":                   # every system sees it
        g["sigma"] = g["sigma"].clone()
        g["sigma"][690] = -1.0
        assert torch.isnan(kp.rv_chisq(**g, prec=prec)).all()
        return
    key = {"jitter": "jitter", "offset": "offset", "planet": "e"}[where]
    g[key] = g[key].clone()
    g[key].view(-1)[17] = float("nan")
    chi2 = kp.rv_chisq(**g, prec=prec)
    keep = torch.arange(30, device="cuda") != 17
    assert torch.isnan(chi2[17]) and torch.equal(chi2[keep], clean[keep])
