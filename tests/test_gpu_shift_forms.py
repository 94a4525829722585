"""Mean shift with a block per seed (lists of pieces kept over several
iterations) against one wave per seed: cells around a piece of 64 points,
around what the waves keep, and far larger; long chains of small steps.  Both
forms take the same points into each mean, so weights and iteration counts
are equal and a mode differs by the rounding of a sum of at most n numbers,
(n + 1) 2^-53 max |x| in each form."""
import numpy as np
import pytest
import torch

import paper_2307_00071_amd as gmm

pytestmark = pytest.mark.gpu


def _cloud(d, m, h):
    """A ramp of slowly changing density (long chains) and a cluster of m
    points inside one cell."""
    rng = np.random.default_rng(100 * d + m)
    ramp = rng.uniform(-0.2 * h, 0.2 * h, (3000, d))
    ramp[:, 0] = 30 * h * (np.arange(3000) / 3000.0) ** 0.9
    ramp[:, 1] += 12 * h
    cell = rng.uniform(-0.45 * h, 0.45 * h, (m, d))
    return np.concatenate([cell, ramp]).astype(np.float32)


@pytest.mark.parametrize("d", [3, 4])
@pytest.mark.parametrize("m", [1, 63, 64, 65, 511, 513, 4096, 4200, 30000])
def test_a_block_per_seed_agrees_with_a_wave_per_seed(monkeypatch, d, m):
    print("case: mean shift forms d=%d m=%d" % (d, m), flush=True)
    h = 0.1
    X = _cloud(d, m, h)
    Xt = torch.from_numpy(X).to("cuda:0")
    out = {}
    for form in ("1", "4"):
        monkeypatch.setenv("GMM_MS_SEED_WAVES", form)
        modes, weights, info = gmm.meanshift(Xt, h, seeds=True)
        out[form] = [t.cpu().numpy() for t in (info["seed_modes"], info["seed_weights"],
                                               info["seed_iters"])] + [len(weights)]
    a, b = out["1"], out["4"]
    assert a[2].max() > 20
    np.testing.assert_array_equal(a[1], b[1])
    np.testing.assert_array_equal(a[2], b[2])
    assert a[3] == b[3]
    tol = 2 * (len(X) + 1) * 2.0 ** -53 * float(np.abs(X).max())
    np.testing.assert_allclose(a[0], b[0], rtol=0, atol=tol)
