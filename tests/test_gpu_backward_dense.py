"""The dense backward kernel: the one that runs above 512 components, with
GMM_CULL=0 and under a forced dense tile shape, against the FP64 oracle at
the bars of the registration tests, and the rule that selects it."""
import pytest
import torch

import paper_2307_00071_amd as gmm
from tests.test_gpu_registration import _check, _registration_problem, _to

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(777, 1), (5000, 16), (20011, 64), (3000, 129), (3000, 300)])
def test_dense_kernel_matches_the_oracle(n, k, monkeypatch):
    print("case: dense backward n=%d k=%d" % (n, k), flush=True)
    monkeypatch.setenv("GMM_CULL", "0")
    _check(*_registration_problem(n, k, seed=k, fit_n=max(4000, 4 * k)))


@pytest.mark.parametrize("n,k", [(2500, 513), (4000, 550)])
def test_more_components_than_the_culled_kernel_takes(n, k):
    print("case: backward n=%d k=%d" % (n, k), flush=True)
    _check(*_registration_problem(n, k, seed=3, fit_n=8 * k))


@pytest.mark.parametrize("shape", ["b1024t128", "b512t128", "b512t64"])
def test_a_forced_dense_shape_takes_the_dense_kernel(shape, monkeypatch):
    """Every point reaches the gradients whatever tile the forward has, and
    the gradients are those of GMM_CULL=0 to the bit (one kernel, sums in a
    fixed order)."""
    print("case: backward forced %s" % shape, flush=True)
    src, pose, th = _registration_problem(20011, 64, seed=11, fit_n=8000)
    args, kw = (_to(src), *(_to(a) for a in th)), dict(pose6=_to(pose))
    with monkeypatch.context() as m:
        m.setenv("GMM_CULL", "0")
        want = gmm.loglik_backward(*args, **kw)
    monkeypatch.setenv("GMM_TILE_SHAPE", shape)
    got = gmm.loglik_backward(*args, **kw)
    for key in want:
        assert torch.equal(got[key], want[key]), key
    _check(src, pose, th)
