"""Close pairs in each sub-block of 16 particles of a tile of 64, and in two tiles of a
workgroup, through the symmetric FP32C kernels' repair, which visits only the sub-blocks
that a lane flagged.

n = 1025 makes three blocks of 512; particle i lies in the first, particle j in the second,
at the sub-block and lane offset under test.  The pair carries half of the cluster's mass
and is 1e-5 apart at eps = 0.01, around (3, -2, 5): its force is about ten times the
field's, and without the repair the rounding of its positions (2^-24 * 5 on a displacement
of 1e-5, a few percent) would show at 1e-2.  Bars: 1e-5 for the acceleration and 2e-5 for
the Jacobian product, which the other tests of these kernels use.
"""
import numpy as np
import pytest

import ics
from parity_stats import cond_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nbm
    nbm.load()
    return nbm


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("pairs", [[(37, 512)], [(200, 512 + 64 + 31)], [(311, 512 + 128 + 32)], [(3, 1023)],
                                   [(70, 520), (70 + 256, 520 + 48)]])
def test_sym_repair_visits_flagged_sub_blocks(nb, oracle_mod, pairs):
    n = 1025
    x, v, m = ics.plummer(n, seed=5)
    x = x + np.array([[3.0], [-2.0], [5.0]])
    rng = np.random.default_rng(6)
    for i, j in pairs:
        off = rng.standard_normal(3)
        x[:, j] = x[:, i] + 1e-5 * off / np.linalg.norm(off)
        m[i] = m[j] = 0.5
    w, acc = rng.standard_normal((3, n)), rng.standard_normal((3, n))
    kw = dict(eps=0.01, precision="fp32c")
    nb.nbody_set_config(pairs=2, split=1)
    try:
        gx, gm = (t.cpu().numpy() for t in nb.nbody_accel_vjp(dev(x), dev(m), dev(w), **kw))
        a = [nb.nbody_accel_jerk(dev(x), dev(v), dev(m), **kw)[0].cpu().numpy(),
             nb.nbody_accel_jerk_snap(dev(x), dev(v), dev(acc), dev(m), **kw)[0].cpu().numpy()]
    finally:
        nb.nbody_set_config()
    rows = np.array(pairs).ravel()
    ref = oracle_mod.accel(x, m, eps=0.01)
    for q in a:
        err = np.linalg.norm(q - ref, axis=0) / np.linalg.norm(ref, axis=0)
        print("pairs %s accel err: pair rows %.2e all %.2e" % (pairs, err[rows].max(), err.max()))
        assert err[rows].max() <= 1e-5
    rgx, rgm = oracle_mod.accel_vjp(x, m, w, eps=0.01)
    sx, sm = oracle_mod.accel_vjp_scale_rows(x, m, w, np.arange(n), eps=0.01)
    ex, em = cond_err(gx, rgx, sx).max(), cond_err(gm, rgm, sm).max()
    print("pairs %s vjp cond gx %.2e gm %.2e" % (pairs, ex, em))
    assert ex <= 2e-5 and em <= 2e-5
