"""The row kernels (small systems: one launch per evaluation or step) against the
tile kernels (a forced j-split), which the other tests hold to the oracle.

Sizes sit at the edges: fewer rows than a workgroup, one short of and one past a
workgroup's rows (4 in FP64, 16 or 32 in FP32C) and a block of j (256, 64), the
sizes where the launch shape changes and the largest systems served.

FP64: both sides are FP64 sums of the same terms; what differs is the order of the
sums and the last roundings of a term.  Each is within a few tens of units of
1.1e-16 of the sum of its terms' magnitudes, which for these clusters is at most
~100 times the component's largest value over the particles: 1e-12 of that largest
value holds with a factor of a few to spare; the trajectories of three short steps
carry the same relative error.

FP32C and FP32: both sides sum the same FP32 terms of a block of 64 j in the same
order and combine k blocks in more than FP32, the tile kernel in an FP32 pair whose
low half is off by at most k^2 2^-48 / 2 of the sums (3e-12 for 43 blocks).  1e-9 of
the largest value leaves room for sums that cancel a hundredfold, and is far below
6e-8, what one FP32 rounding in a term or in the order of a sum would show.
"""
import numpy as np
import pytest

import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32c": 1e-9, "fp32": 1e-9}
PRECS = ["fp64", "fp32c", "fp32"]
SIZES = [1, 2, 5, 63, 65, 255, 257, 1022, 2049, 4097, 8191]


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nbm
    nbm.load()
    return nbm


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def both(nb, f, prec="fp64"):
    """f() on the row kernels and on the tile kernels."""
    rows = [t.clone() for t in f()]
    nb.nbody_set_config(ipl=1, split=3)
    try:
        tiles = [t.clone() for t in f()]
    finally:
        nb.nbody_set_config()
    for k, (p, q) in enumerate(zip(rows, tiles)):
        assert torch.isfinite(p).all(), k
        scale = q.abs().max().item()
        assert (p - q).abs().max().item() <= TOL[prec] * max(scale, 1e-300), (k, (p - q).abs().max().item(), scale)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("eps", [0.01, 0.0])
@pytest.mark.parametrize("prec", PRECS)
def test_row_evaluations_match_tiles(nb, n, eps, prec):
    x, v, m = ics.two_component(n, seed=70 + n) if n > 20 else ics.random_cloud(n, seed=70 + n)
    rng = np.random.default_rng(n)
    tx, tm = dev(x), dev(m)
    tv, tw, ta = (dev(rng.standard_normal(x.shape)) for _ in range(3))
    kw = dict(G=1.3, eps=eps, precision=prec, exclude_self=eps == 0.0)
    print("rows n=%d eps=%g %s" % (n, eps, prec), flush=True)
    both(nb, lambda: [nb.nbody_accel(tx, tm, **kw)], prec)
    both(nb, lambda: nb.nbody_accel_vjp(tx, tm, tw, **kw), prec)
    both(nb, lambda: nb.nbody_accel_jerk(tx, tv, tm, **kw), prec)
    both(nb, lambda: nb.nbody_accel_jerk_snap(tx, tv, ta, tm, **kw), prec)
    if prec == "fp64":
        both(nb, lambda: [nb.nbody_potential(tx, tm, G=1.3, eps=eps)])


@pytest.mark.parametrize("n", [8193, 24576])
@pytest.mark.parametrize("rescue", [0, 2])
def test_row_force32_largest_systems(nb, n, rescue):
    """The FP32C force above the other evaluations' sizes, with rows flagged for
    the FP64 rescue and without it, and close pairs in both halves of a block."""
    x, _, m = ics.plummer(n, seed=77)
    x = x + np.array([[2.0], [-1.0], [3.0]])
    x[:, 40:60] = x[:, 4040:4060] + 1e-4
    x[:, 70:90] = x[:, 100:120] + 1e-4
    tx, tm = dev(x), dev(m)
    got = []
    for split in (0, 3):
        nb.nbody_set_config(ipl=1 if split else 0, split=split, rescue=rescue)
        try:
            got.append(nb.nbody_accel(tx, tm, eps=1e-3, precision="fp32c").clone())
        finally:
            nb.nbody_set_config()
    print("row force n=%d rescue=%d" % (n, rescue), flush=True)
    assert (got[0] - got[1]).abs().max().item() <= TOL["fp32c"] * got[1].abs().max().item()


@pytest.mark.parametrize("n", [3, 257, 1022])
@pytest.mark.parametrize("steps,valid", [(0, False), (1, False), (1, True), (2, False), (2, True), (3, False), (3, True)])
@pytest.mark.parametrize("prec", PRECS)
def test_row_steps_match_tiles(nb, n, steps, valid, prec):
    """Every buffer parity of the fused steps, with and without a valid state."""
    x, v, m = ics.random_cloud(n, seed=80 + n)
    tm, dt = dev(m), 1.0 / 256
    kw = dict(eps=0.05, precision=prec)

    def state(k, start):
        s = [dev(x), dev(v)] + [torch.full((3, n), 7.0, dtype=torch.float64, device="cuda:0") for _ in range(k)]
        if valid:
            start(*s)
        return s

    def kdk():
        s = state(1, lambda *s: nb.nbody_step(*s, tm, dt, 0, **kw))
        nb.nbody_step(*s, tm, dt, steps, acc_valid=valid, **kw)
        return s

    def h4():
        s = state(2, lambda *s: nb.nbody_step_hermite(*s, tm, dt, 0, **kw))
        nb.nbody_step_hermite(*s, tm, dt, steps, acc_valid=valid, **kw)
        return s

    def h6():
        s = state(4, lambda *s: nb.nbody_step_hermite6(*s, tm, dt, 0, **kw))
        nb.nbody_step_hermite6(*s, tm, dt, steps, acc_valid=valid, **kw)
        return s[:5]  # the crackle divides differences of the others by dt^3

    print("row steps n=%d steps=%d valid=%s %s" % (n, steps, valid, prec), flush=True)
    both(nb, kdk, prec)
    both(nb, h4, prec)
    both(nb, h6, prec)


@pytest.mark.parametrize("steps,every", [(0, 4), (1, 4), (5, 5), (6, 4), (7, 3)])
@pytest.mark.parametrize("prec", ["fp64", "fp32c"])
def test_row_gradient_matches_tiles(nb, steps, every, prec):
    """The adjoint sweep with the update in the VJP's launch: even and odd step
    counts, one and several segments."""
    n = 257
    x, v, m = ics.random_cloud(n, seed=90)
    rng = np.random.default_rng(90)
    w = [dev(rng.standard_normal((3, n))) for _ in range(2)]

    def grad():
        t = [dev(a).requires_grad_(True) for a in (x, v, m)]
        out = nb.trajectory(*t, 1.0 / 128, steps, every=every, eps=0.05, precision=prec)
        return list(o.detach() for o in out) + list(torch.autograd.grad(out, t, w, allow_unused=True))

    print("row gradient steps=%d every=%d %s" % (steps, every, prec), flush=True)
    both(nb, grad, prec)


@pytest.mark.parametrize("n", [1, 511, 513, 1024, 2500, 8192, 9001])
@pytest.mark.parametrize("launches", [0, 2])
def test_symmetric_potential_matches_tiles(nb, n, launches):
    """One block, odd and even numbers of blocks of 512, ragged ends, a half ring
    in one and two launches, with and without softening; the energy's potential
    is the same one."""
    x, v, m = ics.two_component(n, seed=60 + n) if n > 20 else ics.random_cloud(n, seed=60 + n)
    tx, tv, tm = dev(x), dev(v), dev(m)
    for eps in (0.01, 0.0):
        print("potential n=%d launches=%d eps=%g" % (n, launches, eps), flush=True)
        got = {}
        for form in (dict(pairs=2, split=launches), dict(split=3)):
            nb.nbody_set_config(**form)
            try:
                got[form["split"] == 3] = [nb.nbody_potential(tx, tm, G=0.7, eps=eps).clone(),
                                           nb.nbody_energy(tx, tv, tm, G=0.7, eps=eps)[1:2].clone()]
            finally:
                nb.nbody_set_config()
        for p, q in zip(got[False], got[True]):
            assert torch.isfinite(p).all()
            assert (p - q).abs().max().item() <= TOL["fp64"] * max(q.abs().max().item(), 1e-300), (p - q).abs().max().item()
