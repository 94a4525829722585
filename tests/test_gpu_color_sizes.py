"""Conditional intensity with the components split over the waves of a block
(fewer components than waves, remainders, the largest K) and blocks of 64
locations that hold near and far ones and end inside a block; joint sampling
at the smallest and largest K.  The bars are those of test_gpu_gmm4.py."""
import numpy as np
import pytest
import torch

import paper_2307_00071_amd as gmm
from oracle import gmm4 as o4
from tests.test_gpu_gmm4 import _cond_check, _fitted4, _to

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 7, 33, 512])
def test_conditional_over_split_components(K):
    print("case: conditional K=%d" % K, flush=True)
    X, th = _fitted4(K=K, n=max(2000, 30 * K), seed=3)
    locs = np.ascontiguousarray(X[:, :3])
    locs[::5] += np.float32(40.0)      # every block has far locations
    for m in (1, 63, 64, 65, 1999):
        _cond_check(np.ascontiguousarray(locs[:m]), th)
    _cond_check(np.ascontiguousarray(locs[:1000:5]), th)   # far ones alone


@pytest.mark.parametrize("K", [1, 2, 255, 257, 1024])
def test_joint_sample_over_component_counts(K):
    print("case: joint sample K=%d" % K, flush=True)
    rng = np.random.default_rng(K)
    w = rng.random(K).astype(np.float32)
    w[K // 2 + 1:: 3] = 0.0
    mu = rng.normal(0, 2, (K, 4)).astype(np.float32)
    A = rng.normal(0, 0.3, (K, 4, 4))
    cov = (A @ A.transpose(0, 2, 1) + 0.05 * np.eye(4)).astype(np.float32)
    m = 3000
    u = rng.random(m)
    u[0], u[1] = 0.0, 1.0 - 2.0 ** -53
    z = rng.standard_normal((m, 4)).astype(np.float32)
    out, comp = gmm.joint_dist_sample(_to(w), _to(mu), _to(cov), m, u=u, z=z)
    torch.cuda.synchronize()
    ro, rc = o4.joint_sample(w.astype(np.float64), mu.astype(np.float64), cov.astype(np.float64),
                             u, z.astype(np.float64))
    np.testing.assert_array_equal(comp.cpu().numpy(), rc)
    ulp = np.spacing(np.abs(ro).astype(np.float32)).astype(np.float64)
    assert np.all(np.abs(out.cpu().numpy() - ro) <= 2 * ulp + 1e-30)
