"""Populations large enough for full rounds of batches in the sampler's half step, where
a block's batch of chains is as large as its share of the LDS allows."""
import numpy as np
import pytest
import torch

import paper_0812_2976_amd as kp
from tests import workloads as W

pytestmark = pytest.mark.gpu


def _gpu(x):
    return torch.as_tensor(np.ascontiguousarray(x), device="cuda")


@pytest.mark.parametrize("n_half,n_pl,n_obs,prec", [(70001, 4, 64, "mixed"), (70001, 4, 100, "mixed"), (40003, 8, 33, "mixed"),
                                                    (30001, 8, 64, "fp64"), (30001, 8, 65, "fp64"), (70001, 1, 20, "fp64")])
@pytest.mark.parametrize("opts", [None, {"block_threads": 256}])
def test_stored_chisq_of_a_large_population(n_half, n_pl, n_obs, prec, opts):
    n_gen = 3
    wl = W.dense("c4", n_sys=1, n_pl=n_pl, n_obs=n_obs, seed=n_obs)
    rng = np.random.default_rng(n_half)
    p = np.concatenate([np.concatenate([getattr(wl, k)[:, 0] for k in ("P", "K", "e", "w", "M0")]), [0.0]])
    x = p[None, :, None] * (1.0 + 1e-4 * rng.standard_normal((2, p.size, n_half)))
    runs = []
    for fused in (False, True):
        s = kp.DEMC(_gpu(wl.t), _gpu(wl.v), _gpu(wl.sigma), _gpu(x), _gpu(1e-8 * np.abs(p) + 1e-9), seed=7, prec=prec,
                    opts=opts)
        (s.run if fused else s.generations)(0, n_gen)
        stored = s.chi2.clone()
        again = s.chisq()
        # the same terms, at most n_obs of them and none negative, summed in another order
        assert ((stored - again).abs() <= 2.0 ** -52 * n_obs * again).all()
        runs.append((s.x.clone(), stored, s.n_accept.clone()))
    assert runs[0][2].sum() > 0
    assert all(torch.equal(a, b) for a, b in zip(*runs))
