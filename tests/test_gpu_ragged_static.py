"""The plan-free ragged chi-square at the edges of its ordering kernels (tiles of
1,024 systems, one block up to 8,192) and of the block-per-item form (its two
block sizes, and the batches past it), with rejected systems among them: against
the binary64 path, which checks each system's offsets by itself."""
import numpy as np
import pytest
import torch

import paper_0812_2976_amd as kp

pytestmark = pytest.mark.gpu


def _batch(n_sys, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    f64 = dict(generator=g, device="cuda", dtype=torch.float64)
    n_pl = torch.randint(1, 9, (n_sys,), generator=g, device="cuda")
    n_obs = torch.randint(0, 300, (n_sys,), generator=g, device="cuda")
    n_obs[::7] = 64 * (n_obs[::7] % 6)                          # whole groups only, and empty systems
    off = [torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), n.cumsum(0)]) for n in (n_obs, n_pl)]
    n, p = int(off[0][-1]), int(off[1][-1])
    args = dict(t=2454000 + 3000 * torch.rand(n, **f64), v=60 * torch.randn(n, **f64), sigma=1 + 4 * torch.rand(n, **f64),
                P=torch.exp(6.9 * torch.rand(p, **f64)), K=1 + 99 * torch.rand(p, **f64), e=0.99 * torch.rand(p, **f64),
                omega=6.28 * torch.rand(p, **f64), M0=6.28 * torch.rand(p, **f64), jitter=3 * torch.rand(n_sys, **f64))
    # no planets, a decreasing observation offset, one past the end
    rng = np.random.default_rng(seed)
    bad = rng.choice(np.arange(1, max(n_sys - 1, 2)), size=min(max(n_sys // 50, 0), 200), replace=False)
    for k, i in enumerate(bad.tolist()):
        if k % 3 == 0:
            off[1][i + 1] = off[1][i]
        elif k % 3 == 1:
            off[0][i] = off[0][i + 1] + 5
        else:
            off[0][i + 1] = n + 1 + k
    return dict(args, obs_off=off[0], pl_off=off[1])


@pytest.mark.parametrize("n_sys", [1, 15, 16, 17, 1023, 1024, 1025, 8192, 8193, 9000, 30011, 44000])
def test_static_against_binary64(n_sys):
    """Velocities within the stated 1e-3 m/s, so chi2 within 2e-3 sum w |r| + 1e-6 sum w, and
    (sum w |r|)^2 <= chi2 sum w with w <= 1."""
    b = _batch(n_sys, n_sys)
    ref = kp.rv_chisq_ragged_static(**b, prec="fp64")
    first = kp.rv_chisq_ragged_static(**b)
    assert torch.equal(torch.isnan(first), torch.isnan(ref))
    ok = ~torch.isnan(ref)
    n = b["obs_off"].diff().double()[ok]
    tol = 2e-3 * torch.sqrt(ref[ok] * n) + 1e-6 * n
    assert ((first[ok] - ref[ok]).abs() <= tol).all()
    for opts in (None, {"block_threads": 64}, {"block_threads": 128}, {"block_threads": 256}):
        again = kp.rv_chisq_ragged_static(**b, opts=opts)         # the same evaluations, summed in another order
        assert torch.equal(torch.isnan(again), torch.isnan(ref))
        assert ((again[ok] - first[ok]).abs() <= 1e-13 * first[ok].abs()).all()
