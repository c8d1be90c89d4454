"""The jerk and snap of close pairs through the symmetric FP32C kernels' repair, which is
written for each evaluation: the pairs and lanes of test_gpu_sym_near.py, all components.

The pair's particles are 1e-5 apart with eps = 1e-5 around (3, -2, 5) and hold half of the
mass each, so that their terms are some 1e9 of the field's and all depend on the
displacement, which positions rounded to FP32 give to a few percent.  Errors are relative
to the sum of the magnitudes of the pair's own terms (the row's scale); about 40 roundings
of 6e-8 make 2.4e-6, the bar is the VJP's 2e-5.  Plain FP32, without the repair, has to
exceed it tenfold.
"""
import numpy as np
import pytest

import ics

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
def test_sym_repair_of_jerk_and_snap(nb, oracle_mod, pairs):
    n, eps = 1025, 1e-5
    x, v, m = ics.plummer(n, seed=5)
    x = x + np.array([[3.0], [-2.0], [5.0]])
    rng = np.random.default_rng(6)
    acc = rng.standard_normal((3, n))
    for i, j in pairs:
        off = rng.standard_normal(3)
        x[:, j] = x[:, i] + 1e-5 * off / np.linalg.norm(off)
        m[i] = m[j] = 0.5
    rows = np.array(pairs).ravel()
    ref = oracle_mod.accel_jerk_snap_rows(x, v, acc, m, rows, eps=eps)
    scale = np.empty((3, rows.size))
    norm = np.linalg.norm
    for k, (i, j) in enumerate(pairs):
        d, w, u = x[:, j] - x[:, i], v[:, j] - v[:, i], acc[:, j] - acc[:, i]
        s = d @ d + eps * eps
        t, al = 0.5 * s ** -1.5, abs(d @ w) / s
        jerk = norm(w) + 3 * al * norm(d)
        snap = norm(u) + 6 * al * jerk + 3 * ((w @ w + norm(d) * norm(u)) / s + al * al) * norm(d)
        scale[:, 2 * k] = scale[:, 2 * k + 1] = t * norm(d), t * jerk, t * snap
    worst = {}
    for prec in ("fp32c", "fp32"):
        nb.nbody_set_config(pairs=2, split=1)
        try:
            got = [nb.nbody_accel_jerk(dev(x), dev(v), dev(m), eps=eps, precision=prec),
                   nb.nbody_accel_jerk_snap(dev(x), dev(v), dev(acc), dev(m), eps=eps, precision=prec)]
        finally:
            nb.nbody_set_config()
        worst[prec] = [[norm(q.cpu().numpy()[:, rows] - ref[c], axis=0) / scale[c] for c, q in enumerate(g)] for g in got]
        print("pairs %s %s: worst %s" % (pairs, prec, [["%.1e" % e.max() for e in g] for g in worst[prec]]), flush=True)
    for g, g32 in zip(worst["fp32c"], worst["fp32"]):
        for e, e32 in zip(g, g32):
            assert e.max() <= 2e-5
            assert e32.min() > 2e-4
