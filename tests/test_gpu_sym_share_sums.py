"""FP64 evaluations whose half ring takes several launches: a particle's slots are added
in four shares, so the error stays that of four short sums.

Tolerance: with particles in random order a sum over K slots grows evenly, and its
roundings, each rms r = 2^-53 / sqrt(3) of the sum so far at most, add up to
r sqrt(K / 3) of the result in one run and to r sqrt(K / 48) in four shares.  204800
particles have K = 200 distances of 512: 8.2 r and 2.0 r; the bar is their geometric
mean, 4.1 r.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_chunked_ring_sums_in_shares():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nb
    n, eps = 204800, 1e-3
    g = np.random.default_rng(5)
    x = g.standard_normal((3, n)) * np.exp(g.standard_normal(n))
    m, v = g.random(n) / n, g.standard_normal((3, n))
    rows = np.sort(g.choice(n, 512, replace=False))
    a, _ = nb.nbody_accel_jerk(*(torch.from_numpy(t).cuda() for t in (x, v, m)), eps=eps, precision="fp64")
    ref = oracle.accel_rows(x, m, rows, eps=eps)
    err = a.cpu().numpy()[:, rows] - ref
    rms = np.sqrt(((err ** 2).sum(0) / (ref ** 2).sum(0)).mean())
    assert rms < 4.1 * 2.0 ** -53 / np.sqrt(3.0), rms
