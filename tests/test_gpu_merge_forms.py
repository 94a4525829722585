"""The merge of the mean-shift modes where its passes change form: chains of
decisions longer than one launch's passes, more undecided predecessors within
h than a wave keeps, more modes than a wave keeps lists for, and modes that
fall in one cell.  The kept set is a whole answer: no tolerance."""
import numpy as np
import pytest

from tests.test_gpu_gbms import _check_merge_properties, _run

pytestmark = pytest.mark.gpu


def _line(h, bins, d):
    """One mode per bin, weights falling along the line: every decision
    waits for the one before."""
    rng = np.random.default_rng(bins)
    x = np.repeat(np.arange(bins) * 0.9 * h, bins + 40 - np.arange(bins))
    X = rng.uniform(-1e-3 * h, 1e-3 * h, (len(x), d))
    X[:, 0] += x
    return X


def _cloud(kind, h):
    rng = np.random.default_rng(5)
    if kind == "line":
        return _line(h, 300, 3)
    if kind == "short line":
        return _line(h, 70, 4)
    if kind == "one cluster":
        return rng.normal(0, 2.2 * h, (6000, 4))
    return rng.uniform(0, 38 * h, (60000, 3))    # "many"


@pytest.mark.parametrize("kind,max_iter", [("line", 0), ("short line", 0), ("one cluster", 300),
                                           ("one cluster", 0), ("many", 0), ("many", 3)])
def test_merge_decides_the_greedy_set(kind, max_iter):
    print("case: merge %s max_iter=%d" % (kind, max_iter), flush=True)
    h = 0.1
    modes, w, info = _run(_cloud(kind, h), h, max_iter)
    st = info["seed_status"]
    assert st.min() >= 1                   # every mode decided
    if kind == "many":
        assert len(st) > 4 * 4096
    if kind == "line":
        assert (st != 3).sum() > 250
    _check_merge_properties(h, info)
    np.testing.assert_array_equal(modes, info["seed_modes"][st == 1])
    np.testing.assert_array_equal(w, info["seed_weights"][st == 1])
