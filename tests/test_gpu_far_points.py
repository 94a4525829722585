"""Points far from every component (float32 weight sum below 2^-100), alone,
in clusters and as whole clouds, in the culled scoring and backward kernels
against the dense ones (GMM_CULL=0).

Both evaluate each pair's float32 term alike, so they differ by the order of
float32 sums alone: of K terms for a point (at most K 2^-24 of the sum of
their sizes) and of 64 points for a component.  Bars: K 2^-24 with at least
64 terms, of each array's largest entry (lse: of the point's value, plus
the bar itself for the logarithm of the sum)."""
import numpy as np
import pytest
import torch

import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _cloud(n, pattern, mu, rng):
    x = mu[rng.integers(0, len(mu), n)] + 0.3 * rng.standard_normal((n, 3))
    far = {"none": [], "one": [n // 2], "tail": range(n - n // 3, n),
           "every third": range(0, n, 3), "all": range(n)}[pattern]
    far = np.asarray(list(far), np.int64)
    x[far] += np.array([9.0, -7.0, 8.0]) + 2.0 * rng.standard_normal((len(far), 3))
    return x.astype(np.float32)


@pytest.mark.parametrize("pattern", ["none", "one", "tail", "every third", "all"])
@pytest.mark.parametrize("n,k", [(1, 1), (63, 5), (129, 16), (1000, 64), (3001, 130), (2000, 300),
                                 (700, 512)])
def test_far_points_match_the_dense_kernels(n, k, pattern, monkeypatch):
    print("case: far points n=%d k=%d %s" % (n, k, pattern), flush=True)
    rng = np.random.default_rng(n + k)
    w, mu, cov = synth.random_theta(k, k, spread=3.0, smin=0.05, smax=0.3)
    x = torch.from_numpy(_cloud(n, pattern, mu, rng)).to(DEV)
    th = [torch.as_tensor(a, dtype=torch.float32, device=DEV) for a in (w, mu, cov)]
    pose = torch.tensor([0.05, -0.02, 0.03, 0.1, 0.0, -0.1], device=DEV)

    def run():
        L, lse = gmm.loglik(x, *th, pose6=pose, return_lse=True)
        g = gmm.loglik_backward(x, *th, pose6=pose)
        return float(L), lse.double(), {a: b.double() for a, b in g.items()}

    L1, lse1, g1 = run()
    monkeypatch.setenv("GMM_CULL", "0")
    L0, lse0, g0 = run()
    bar = max(k, 64) * 2.0 ** -24
    assert bool(((lse1 - lse0).abs() <= bar * (1.0 + lse0.abs())).all())
    assert abs(L1 - L0) <= bar * (n + abs(L0))
    for key in g0:
        d, scale = float((g1[key] - g0[key]).abs().max()), float(g0[key].abs().max())
        print(key, d, scale, flush=True)
        assert d <= bar * scale, (key, d, scale)
