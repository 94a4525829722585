"""Conditional intensity on both sides of the line between one wave and four
waves a group of 64 locations (16,384 locations per component), near and far
locations mixed in every group and a last group that is not full.  The bars
are those of test_gpu_gmm4.py."""
import numpy as np
import pytest
import torch

import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import _lib
from tests.test_gpu_gmm4 import _cond_check, _fitted4, _to

pytestmark = pytest.mark.gpu


def _locations(X, m):
    locs = np.resize(X[:, :3], (m, 3)).astype(np.float32)
    locs[::5] += np.float32(40.0)
    return np.ascontiguousarray(locs)


@pytest.mark.parametrize("K,m", [(1, 16383), (1, 16384), (1, 16449), (2, 32767), (2, 32769),
                                 (5, 81919), (5, 82000)])
def test_conditional_on_both_sides_of_the_split(K, m):
    print("case: conditional split K=%d m=%d" % (K, m), flush=True)
    X, th = _fitted4(K=K, n=2000, seed=3)
    _cond_check(_locations(X, m), th)


def test_a_location_that_is_not_finite_beyond_the_split():
    print("case: conditional split, NaN", flush=True)
    X, th = _fitted4(K=2, n=2000, seed=3)
    locs = _locations(X, 33000)
    locs[32999, 1] = np.nan
    with pytest.raises(_lib.GmmError, match="finite"):
        gmm.color_conditional(_to(locs), *(_to(a) for a in th))
    torch.cuda.synchronize()
