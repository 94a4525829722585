"""The padding of a cloud's last tile takes no part in the gradient, also where
its position (the origin) is out of float32 range for every component: the
culled backward kernel against the dense one (GMM_CULL=0), at 64 roundings
of 2^-24 of each array's largest entry (a tile's points in any order)."""
import numpy as np
import pytest
import torch

import paper_2307_00071_amd as gmm

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n,k", [(65, 2), (100, 70)])
def test_padding_out_of_float32_range_leaves_the_gradient(n, k, monkeypatch):
    """The last tile's padding sits at the origin, where every component of
    this mixture (sigma 1e-16 m at 1e4 m) has a squared distance beyond
    float32; its far points are one float32 step from a mean, in range."""
    print("case: padding out of range n=%d k=%d" % (n, k), flush=True)
    rng = np.random.default_rng(n)
    mu = np.full((k, 3), 1e4, np.float32) + 64.0 * np.arange(k, dtype=np.float32)[:, None]
    x = mu[rng.integers(0, k, n)].copy()
    x[-3:, 0] = np.nextafter(x[-3:, 0], np.float32(1e9))
    w = np.full(k, 1.0 / k)
    cov = np.tile(1e-32 * np.eye(3), (k, 1, 1))
    args = [torch.as_tensor(a, dtype=torch.float32, device=DEV) for a in (x, w, mu, cov)]

    def run():
        g = gmm.loglik_backward(*args, need=("pts", "w", "mu"), check=False)
        return {a: b.double() for a, b in g.items() if b is not None}

    g1 = run()
    monkeypatch.setenv("GMM_CULL", "0")
    g0 = run()
    for key in ("pts", "w", "mu"):
        assert bool(torch.isfinite(g0[key]).all())
        d, scale = float((g1[key] - g0[key]).abs().max()), float(g0[key].abs().max())
        print(key, d, scale, flush=True)
        assert d <= 64 * 2.0 ** -24 * scale, (key, d, scale)
