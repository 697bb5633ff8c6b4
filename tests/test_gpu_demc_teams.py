"""The sampler's half step shares a chain's observations among wavefronts and puts
several teams into a block for large populations: at the edges of both, every
chi-square it stores equals the one that the dense kernel computes for the stored
parameters, and run() takes the same steps as generations()."""
import numpy as np
import pytest
import torch

import paper_0812_2976_amd as kp
from tests import workloads as W

pytestmark = pytest.mark.gpu


def _gpu(x):
    return torch.as_tensor(np.ascontiguousarray(x), device="cuda")


@pytest.mark.parametrize("n_half,n_obs", [(3, 1), (3, 2000), (1023, 65), (1024, 64), (1024, 129), (1030, 257),
                                          (1100, 1100), (2051, 128)])
@pytest.mark.parametrize("opts", [None, {"block_threads": 64}, {"block_threads": 192}, {"block_threads": 256}])
@pytest.mark.parametrize("jitter", [False, True])
def test_stored_chisq(n_half, n_obs, opts, jitter):
    n_pl, n_gen = 1 + n_obs % 3, 4
    wl = W.dense("c4", n_sys=1, n_pl=n_pl, n_obs=n_obs, seed=n_obs)
    rng = np.random.default_rng(n_half)
    p = np.concatenate([np.concatenate([getattr(wl, k)[:, 0] for k in ("P", "K", "e", "w", "M0")]), [0.0]])
    x = p[None, :, None] * (1.0 + 1e-4 * rng.standard_normal((2, p.size, n_half)))
    x[:, n_pl:2 * n_pl] = np.abs(x[:, n_pl:2 * n_pl])
    jit = _gpu(rng.uniform(0.5, 2.0, (2, n_half))) if jitter else None
    runs = []
    for fused in (False, True):
        s = kp.DEMC(_gpu(wl.t), _gpu(wl.v), _gpu(wl.sigma), _gpu(x), _gpu(1e-8 * np.abs(p) + 1e-9), seed=7, jitter=jit,
                    opts=opts)
        (s.run if fused else s.generations)(0, n_gen)
        stored = s.chi2.clone()
        again = s.chisq()
        # the same terms, at most n_obs of them and none negative, summed in another order
        assert ((stored - again).abs() <= 2.0 ** -52 * n_obs * again).all()
        runs.append((s.x.clone(), stored, s.n_accept.clone()))
    assert runs[0][2].sum() > 0
    assert all(torch.equal(a, b) for a, b in zip(*runs))
