"""KDK runs on the symmetric FP64 force, whose last kernel kicks, drifts and stages the next
step, against the same steps one call at a time with the force evaluated apart: bitwise, since
both do the same operations on the same values.

Sizes: one block (no half ring), an odd and an even ring with a ragged last block, a ring cut
into several launches (slot sums on the side stream).  The trajectory of nbody_traj_grad's
recompute (positions of every step) goes through the same loop.
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


@pytest.mark.parametrize("n,launches", [(100, 0), (512, 0), (1300, 0), (2047, 0), (3000, 3), (9001, 0)])
@pytest.mark.parametrize("steps", [1, 2, 5])
def test_fused_steps_match_single_evaluations(nb, n, launches, steps):
    x, v, m = (dev(q) for q in ics.plummer(n, seed=n))
    dt, kw = 1.0 / 64, dict(eps=0.02, precision="fp64")
    nb.nbody_set_config(pairs=2, split=launches)
    try:
        for valid in (False, True):
            xs, vs = x.clone(), v.clone()
            a = nb.nbody_accel(x, m, **kw)
            got = [x.clone(), v.clone(), a.clone() if valid else torch.full_like(x, float("nan"))]
            nb.nbody_step(*got, m, dt, steps, acc_valid=valid, **kw)
            for k in range(steps):
                nb.nbody_step(xs, vs, a, m, dt, 1, acc_valid=True, **kw)
            want = nb.nbody_accel(got[0], m, **kw)
            assert torch.equal(got[0], xs) and torch.equal(got[2], a) and torch.equal(got[2], want), (n, valid)
            # a closing and an opening half-kick of two calls are the two of one step
            assert torch.equal(got[1], vs), (n, valid)
    finally:
        nb.nbody_set_config()


@pytest.mark.parametrize("n", [1300, 9001])
def test_recomputed_trajectory_gradient(nb, n):
    """Checkpoints every 3 of 7 steps (the sweep recomputes positions through the loop)
    against a checkpoint at every step (nothing recomputed): the same values, so bitwise."""
    x, v, m = (dev(q) for q in ics.plummer(n, seed=n + 1))
    dt, steps, kw = 1.0 / 64, 7, dict(eps=0.02, precision="fp64")
    gx, gv = torch.randn_like(x), torch.randn_like(v)
    nb.nbody_set_config(pairs=2)
    try:
        out = []
        for every in (1, 3):
            xs, vs, a = x.clone(), v.clone(), nb.nbody_accel(x, m, **kw)
            cx, cv = [], []
            for k in range(steps):
                if k % every == 0:
                    cx.append(xs.clone())
                    cv.append(vs.clone())
                nb.nbody_step(xs, vs, a, m, dt, 1, acc_valid=True, **kw)
            out.append(nb.nbody_traj_grad(torch.stack(cx), torch.stack(cv), every, steps, m, dt, gx, gv, **kw))
        for p, q in zip(*out):
            assert torch.isfinite(p).all() and torch.equal(p, q)
    finally:
        nb.nbody_set_config()
