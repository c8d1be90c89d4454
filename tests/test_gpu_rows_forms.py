"""The row kernels against the tile kernels' other forms (two and four particles a lane,
one slice, many) and against the symmetric ones, with the tolerances of test_gpu_rows.py
for the ordered forms; the symmetric FP32C force has other terms and takes its 1e-5."""
import numpy as np
import pytest

import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32c": 1e-9, "fp32": 1e-9}


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("n", [130, 3001])
@pytest.mark.parametrize("form", [dict(ipl=2), dict(ipl=4, split=1), dict(split=1), dict(split=40), dict(pairs=2)])
@pytest.mark.parametrize("prec", ["fp64", "fp32c", "fp32"])
def test_rows_match_every_form(n, form, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nb
    if form.get("pairs") and prec != "fp64":
        tol = {"fp32c": 1e-5, "fp32": 1e-4}[prec]
    else:
        tol = TOL[prec]
    x, v, m = ics.plummer(n, seed=n)
    rng = np.random.default_rng(n)
    tx, tv, tm, tw, ta = dev(x), dev(v), dev(m), dev(rng.standard_normal(x.shape)), dev(rng.standard_normal(x.shape))
    kw = dict(eps=0.02, precision=prec)
    run = lambda: [nb.nbody_accel(tx, tm, **kw), *nb.nbody_accel_vjp(tx, tm, tw, **kw),
                   *nb.nbody_accel_jerk(tx, tv, tm, **kw), *nb.nbody_accel_jerk_snap(tx, tv, ta, tm, **kw)]
    rows = run()
    nb.nbody_set_config(**form)
    try:
        other = run()
    finally:
        nb.nbody_set_config()
    print("rows n=%d %s against %r" % (n, prec, form), flush=True)
    for k, (p, q) in enumerate(zip(rows, other)):
        assert (p - q).abs().max().item() <= tol * q.abs().max().item(), k
