"""nbody_step captured into a HIP graph before any call has sized the workspace: at the
sizes of the row kernels neither nbody_accel nor nbody_step with nsteps <= 1 needs
scratch, so a program that warms up with one of those has none when it captures a call
of several steps.  Replays, with eager work between them, equal the eager call bitwise.
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


@pytest.mark.parametrize("n,prec", [(100, "fp64"), (1000, "fp64"), (1000, "fp32"), (1000, "fp32c"), (16384, "fp32c")])
@pytest.mark.parametrize("steps,valid", [(2, True), (3, True), (4, False)])
def test_step_captured_without_a_workspace(nb, n, prec, steps, valid):
    x, v, m = ics.plummer(n, seed=n)
    tm, dt, kw = dev(m), 1.0 / 256, dict(eps=0.05, precision=prec)
    print("step capture n=%d %s steps=%d valid=%s" % (n, prec, steps, valid), flush=True)
    torch.cuda.synchronize()
    nb.nbody_finalize()  # no workspace
    s = [dev(x), dev(v), torch.empty(3, n, dtype=torch.float64, device="cuda:0")]
    nb.nbody_step(*s, tm, dt, 0, **kw)
    start = [t.clone() for t in s]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        nb.nbody_step(*s, tm, dt, steps, acc_valid=valid, **kw)
    ref = [t.clone() for t in start]
    nb.nbody_step(*ref, tm, dt, steps, acc_valid=valid, **kw)  # this one sizes the workspace
    for k in range(3):
        for t, u in zip(s, start):
            t.copy_(u)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(t, u) for t, u in zip(s, ref)), k
        (s[0] + 1.0).sum().item()
