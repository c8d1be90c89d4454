"""nbody_accel_noalloc on each kernel that serves it: the row kernels, which need no
scratch; the ordered tile kernels between them and the symmetric ones, whose slices of
the j-range lie in the fixed array; and a set split of 1024, whose slices would not fit
(1.1 MB each for 40000 particles) and are cut to as many as do.  Against nbody_accel,
bitwise where both run the same slices, else to the force tolerances."""
import ctypes

import numpy as np
import pytest

import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = {"fp32c": 1e-5, "fp32": 1e-4, "fp64": 1e-12}


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("n,prec,cfg,same", [
    (1000, "fp64", {}, True), (1000, "fp32c", {}, True), (16384, "fp32c", {}, True),
    (24577, "fp32c", {}, True), (49151, "fp32c", {}, True), (30000, "fp32", {}, True),
    (40000, "fp32c", dict(split=1024), False), (40000, "fp32", dict(split=1024), False),
    (40000, "fp64", dict(split=1024, pairs=1), False)])
def test_noalloc_kernels(n, prec, cfg, same):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nb
    from paper_2605_02744_amd._binding import nbody_params
    lib = nb.load()
    x, _, m = ics.plummer(n, seed=n)
    tx, tm = dev(x), dev(m)
    ta = torch.full((3, n), float("nan"), dtype=torch.float64, device="cuda:0")
    p = nbody_params(1.0, 0.01, nb.PRECISIONS[prec], 0)
    print("noalloc n=%d %s %r" % (n, prec, cfg), flush=True)
    nb.nbody_set_config(**cfg)
    try:
        st = lib.nbody_accel_noalloc(n, *(ctypes.c_void_p(t.data_ptr()) for t in (tx, tm, ta)), ctypes.byref(p),
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == nb.NBODY_OK, lib.nbody_last_error()
        ref = nb.nbody_accel(tx, tm, eps=0.01, precision=prec)
    finally:
        nb.nbody_set_config()
    if same:
        assert torch.equal(ta, ref)
    assert ((ta - ref).norm(dim=0) / ref.norm(dim=0)).max().item() <= TOL[prec]
