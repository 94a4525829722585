"""Registration of two mixtures on both sides of the lines between its two
launch schemes (16 to 128 source components with at most eight target
components each take two launches an iteration): against the oracle's
registration, at the bars of the FP64 comparison (history 1e-11 of
max(1, |f|) per entry, transform 1e-9, equal counts)."""
import numpy as np
import pytest

from oracle import d2d as od
from tests.test_gpu_d2d import _dev, _mixture, _moved
import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(15, 30), (16, 1), (16, 128), (16, 129), (37, 64), (38, 64),
                                 (74, 300), (128, 16), (128, 1024), (128, 1025), (129, 16)])
def test_register_on_both_sides_of_the_lines(m, n):
    print("case: d2d m=%d n=%d" % (m, n), flush=True)
    big = _mixture(m + 3 * n, max(m, n))
    pose = synth.random_pose(m, max_angle=0.1, max_trans=0.1)
    src = tuple(a[:m] for a in big)
    tgt = _moved(tuple(a[:n] for a in big), od.expso3(pose[:3]), pose[3:])
    To, ho, co = od.register(np.eye(4), src, tgt, 3, 5)
    T, h, c = gmm.d2d_register(_dev(src), _dev(tgt), iters_iso=3, iters_aniso=5)
    f = np.array([v for _, v in ho])
    h = h.cpu().numpy()
    assert c.cpu().tolist() == list(co)
    assert np.all(np.isnan(h[len(f):])) and not np.any(np.isnan(h[:len(f)]))
    assert np.abs(h[:len(f)] - f).max() <= 1e-11 * max(1.0, np.abs(f).max())
    assert np.abs(T.cpu().numpy() - To).max() <= 1e-9
