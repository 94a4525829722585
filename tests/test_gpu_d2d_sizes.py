"""Registration of two mixtures at the sizes where the launch scheme changes
(sources of at most 256 components take two launches an iteration) and where
threads, waves and row groups run out: against the oracle's registration, at
the bars of the FP64 comparison (history 1e-11 of max(1, |f|) per entry,
transform 1e-9, equal counts)."""
import numpy as np
import pytest

from oracle import d2d as od
from tests.test_gpu_d2d import _dev, _mixture, _moved
import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("iso,aniso", [(4, 6), (0, 7), (3, 0)])
@pytest.mark.parametrize("m,n", [(2, 1), (1, 65), (64, 255), (255, 64), (256, 257), (257, 40),
                                 (38, 300)])
def test_register_sizes(m, n, iso, aniso):
    print("case: d2d m=%d n=%d iso=%d aniso=%d" % (m, n, iso, aniso), flush=True)
    big = _mixture(m + 3 * n, max(m, n))
    pose = synth.random_pose(m, max_angle=0.1, max_trans=0.1)
    src = tuple(a[:m] for a in big)
    tgt = _moved(tuple(a[:n] for a in big), od.expso3(pose[:3]), pose[3:])
    To, ho, co = od.register(np.eye(4), src, tgt, iso, aniso)
    T, h, c = gmm.d2d_register(_dev(src), _dev(tgt), iters_iso=iso, iters_aniso=aniso)
    f = np.array([v for _, v in ho])
    h = h.cpu().numpy()
    want = [0, 0]
    for stage, k in zip([i for i, it in enumerate((iso, aniso)) if it > 0], co):
        want[stage] = k
    assert c.cpu().tolist() == want
    assert np.all(np.isnan(h[len(f):])) and not np.any(np.isnan(h[:len(f)]))
    assert np.abs(h[:len(f)] - f).max() <= 1e-11 * max(1.0, np.abs(f).max())
    assert np.abs(T.cpu().numpy() - To).max() <= 1e-9
