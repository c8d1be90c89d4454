"""nbody_accel_vjp with its outputs over its inputs (C callers that keep one array for
the cotangent and its product), at the sizes that the row kernels serve otherwise.

The call has to take the tile kernels, which store after the last read: with their
form forced (ipl = 1, the automatic one below 16384 particles) the result of the call
with outputs of its own is bitwise the same, and that is the reference.
"""
import ctypes

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


def vjp(nb, x, m, w, gx, gm, prec):
    from paper_2605_02744_amd._binding import nbody_params
    lib, p = nb.load(), nbody_params(1.0, 0.01, nb.PRECISIONS[prec], 0)
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in (x, m, w, gx, gm)]
    st = lib.nbody_accel_vjp(m.shape[0], *ptr, ctypes.byref(p), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == nb.NBODY_OK, lib.nbody_last_error()


@pytest.mark.parametrize("n", [5, 100, 257, 1000, 8191])
@pytest.mark.parametrize("prec", ["fp64", "fp32c", "fp32"])
def test_vjp_outputs_over_inputs(nb, n, prec):
    x, _, m = ics.random_cloud(n, seed=n)
    w = np.random.default_rng(n).standard_normal(x.shape)
    print("vjp in place n=%d %s" % (n, prec), flush=True)
    nb.nbody_set_config(ipl=1)
    try:
        rx, rm = nb.nbody_accel_vjp(dev(x), dev(m), dev(w), eps=0.01, precision=prec)
    finally:
        nb.nbody_set_config()
    # gx over w and gm over m; gx over x; gx over x but for one particle's offset
    tx, tm, tw = dev(x), dev(m), dev(w)
    vjp(nb, tx, tm, tw, tw, tm, prec)
    assert torch.equal(tw, rx) and torch.equal(tm, rm)
    tx, tm, tw, gm = dev(x), dev(m), dev(w), torch.empty_like(rm)
    vjp(nb, tx, tm, tw, tx, gm, prec)
    assert torch.equal(tx, rx) and torch.equal(gm, rm)
    buf = torch.empty(3 * n + 1, dtype=torch.float64, device="cuda:0")
    buf[:3 * n] = dev(x).ravel()
    tx, gx = buf[:3 * n].view(3, n), buf[1:].view(3, n)
    vjp(nb, tx, dev(m), dev(w), gx, gm, prec)
    assert torch.equal(gx, rx) and torch.equal(gm, rm)
