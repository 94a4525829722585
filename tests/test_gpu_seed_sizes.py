"""k-means++ seeding at the edges of its three forms: the plain rounds
(up to 2,048 chunks of 256 points), the culled rounds with 512 and with
1,024 threads (the line at 8,192 chunks, the end at 16,384) and the pair of
kernels past them.  Points lie in runs of neighbours, so that the culled
rounds skip chunks.  Indices and labels are whole numbers: no tolerance;
the picks are checked along their own trajectory as in the seeding tests."""
import numpy as np
import pytest
import torch

import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import _lib
from tests.test_gpu_kinit import _both

pytestmark = pytest.mark.gpu
C = 256


@pytest.mark.parametrize("n", [1, 255, C, C + 1, 16 * C + 1, 2048 * C - 1, 2048 * C,
                               2048 * C + 1, 2064 * C + 3, 8192 * C, 8192 * C + 1,
                               16384 * C, 16384 * C + 1])
def test_seeding_at_the_edges_of_its_forms(n):
    import ctypes
    K = min(n, 9)
    print("case: seeding n=%d K=%d" % (n, K), flush=True)
    rng = np.random.default_rng(n)
    X = rng.uniform(-8, 8, (n, 3)).astype(np.float32)
    X = np.ascontiguousarray(X[np.lexsort((X[:, 1], X[:, 0].round()))])
    X[n // 3:n // 2] = X[n // 3]     # chunks of one repeated point
    u = rng.random(K)
    cen, lab, rc, rl = _both(X, K, u)
    np.testing.assert_array_equal(cen, rc)
    np.testing.assert_array_equal(lab, rl)
    # without labels: the same centres
    lib = _lib.load()
    Xt = torch.from_numpy(X).to("cuda:0")
    ut = torch.from_numpy(u).to("cuda:0")
    c2 = torch.empty(K, dtype=torch.int64, device="cuda:0")
    st = lib.gmm_kmeanspp(ctypes.c_void_p(Xt.data_ptr()), n, K, ctypes.c_void_p(ut.data_ptr()),
                          ctypes.c_void_p(c2.data_ptr()), None, None, 0, None)
    torch.cuda.synchronize()
    assert st == 0
    np.testing.assert_array_equal(c2.cpu().numpy(), cen)


def test_seeding_with_a_bad_point_in_a_culled_cloud():
    print("case: seeding, one point not finite", flush=True)
    X = torch.rand(2049 * C, 3, device="cuda:0")
    X[-1, 1] = float("inf")
    with pytest.raises(_lib.GmmError) as e:
        gmm.kmeanspp(X, 5, seed=0)
    assert e.value.status == 3
