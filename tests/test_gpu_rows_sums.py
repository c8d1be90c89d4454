"""The row kernels' FP64 sums over lanes and waves are compensated, as the tile kernels'
sums over blocks and slices are.

The potential shows it, since all its terms have one sign.  Its relative error against
sums in extended precision, rms over many particles: the last rounding alone gives
2^-53 sqrt(E[1/s^2] / 3) = 4.7e-17 with the mantissa s spread evenly over [1, 2) in its
logarithm; each further rounding of a whole sum adds as much in squares, the roundings of
128th parts and less that are added plainly about a twentieth.  So sqrt(2) times the one
rounding, 6.7e-17, separates the two (512 rows leave 3 % of scatter): plain sums over
four waves and the levels above give 8e-17.
"""
import numpy as np
import pytest

import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1000, 2048, 5000, 8191])
def test_row_potential_has_one_rounding(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nb
    x, _, m = ics.plummer(n, seed=n)
    phi = nb.nbody_potential(*(torch.tensor(t, device="cuda:0") for t in (x, m)), eps=0.01).cpu().numpy()
    rows = np.random.default_rng(n).choice(n, 512, replace=False)
    xl = x.astype(np.longdouble)
    err = []
    for i in rows:
        d = xl - xl[:, i:i + 1]
        t = m / np.sqrt((d * d).sum(0) + np.longdouble(0.01 * 0.01))
        t[i] = 0
        ref = -t.sum()
        err.append(float((phi[i] - ref) / ref))
    rms = float(np.sqrt(np.mean(np.square(err))))
    print("n=%d rms relative error of phi %.2e" % (n, rms))
    assert rms <= 6.7e-17
