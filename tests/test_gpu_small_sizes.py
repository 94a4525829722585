"""The one-launch fit at the sizes where its tiles, point subsets, label
groups and exchange (one hop up to 4,096 values of all rows, two beyond)
change, from labels, from a mixture and with the stopping rule, against a
launch pair per pass (GMM_SMALL=0).

Bars, those of the comparison of the two forms in test_gpu_fit.py: the
log-likelihood 1e-5 of max(|L|, N) at every iteration (the forms refer a
component's float32 constant to different bounds, and a float32 mean is up to
1e-6 m from its FP64 value, 3e-5 of the thinnest standard deviation), the same
iterations run, and the parameters 1e-4 of each array's norm.
"""
import numpy as np
import pytest
import torch

import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("start", ["labels", "theta0", "tol"])
@pytest.mark.parametrize("n,k", [(3, 1), (255, 9), (256, 16), (257, 2), (2049, 8), (6500, 16),
                                 (13000, 7), (30001, 11), (65536, 3), (65535, 16)])
def test_one_launch_fit_sizes(n, k, start, monkeypatch):
    print("case: one-launch n=%d k=%d %s" % (n, k, start), flush=True)
    X = synth.gaussian_blobs(n + k, n_per=-(-n // 8))[0]
    rng = np.random.default_rng(k)
    X = np.ascontiguousarray(X[rng.permutation(len(X))[:n]])
    lab = synth.kmeanspp_labels(X, k, 1)
    pts, labt = torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV)
    kw = {"iters": 6, "reg_covar": 1e-3}
    if start == "theta0":
        r = gmm.fit(pts, k, iters=0, labels=labt)
        kw["theta0"] = (r.weights, r.means, r.covariances)
    else:
        kw["labels"] = labt
    if start == "tol":
        kw.update(iters=40, tol=1e-3)

    def run():
        r = gmm.fit(pts, k, **kw)
        return [t.double().cpu().numpy() for t in (r.weights, r.means, r.covariances, r.loglik)]

    one = run()
    monkeypatch.setenv("GMM_SMALL", "0")
    two = run()
    assert np.array_equal(np.isnan(one[3]), np.isnan(two[3]))
    ok = ~np.isnan(one[3])
    assert np.all(np.abs(one[3] - two[3])[ok] <= 1e-5 * np.maximum(np.abs(two[3]), n)[ok])
    for a, b in zip(one[:3], two[:3]):
        assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b)
