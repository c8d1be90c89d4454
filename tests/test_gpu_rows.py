"""The FP64 row kernels (systems below 8192 particles: one launch per evaluation
or step, workgroups of four rows, lanes over blocks of 256 particles) against
the tile kernels (a forced j-split), which the other tests hold to the oracle.

Sizes sit at the edges: fewer rows than a workgroup, one short of and one past a
workgroup's four rows and a block of 256, and the largest system served.  Both
sides are FP64 sums of the same terms; what differs is the order of the sums and
the last roundings of a term.  Each is within a few tens of units of 1.1e-16 of
the sum of its terms' magnitudes, which for these clusters is at most ~100 times
the component's largest value over the particles: 1e-12 of that largest value
holds with a factor of a few to spare; the trajectories of three short steps
carry the same relative error.
"""
import numpy as np
import pytest

import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12
SIZES = [1, 2, 5, 255, 257, 1022, 2049, 8191]


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nbm
    nbm.load()
    return nbm


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def both(nb, f):
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
        assert (p - q).abs().max().item() <= TOL * max(scale, 1e-300), (k, (p - q).abs().max().item(), scale)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("eps", [0.01, 0.0])
def test_row_evaluations_match_tiles(nb, n, eps):
    x, v, m = ics.two_component(n, seed=70 + n) if n > 20 else ics.random_cloud(n, seed=70 + n)
    rng = np.random.default_rng(n)
    tx, tm = dev(x), dev(m)
    tv, tw, ta = (dev(rng.standard_normal(x.shape)) for _ in range(3))
    kw = dict(G=1.3, eps=eps, precision="fp64", exclude_self=eps == 0.0)
    print("rows n=%d eps=%g" % (n, eps), flush=True)
    both(nb, lambda: [nb.nbody_accel(tx, tm, **kw)])
    both(nb, lambda: nb.nbody_accel_vjp(tx, tm, tw, **kw))
    both(nb, lambda: nb.nbody_accel_jerk(tx, tv, tm, **kw))
    both(nb, lambda: nb.nbody_accel_jerk_snap(tx, tv, ta, tm, **kw))
    both(nb, lambda: [nb.nbody_potential(tx, tm, G=1.3, eps=eps)])


@pytest.mark.parametrize("n", [3, 257, 1022])
@pytest.mark.parametrize("steps,valid", [(0, False), (1, False), (1, True), (2, False), (2, True), (3, False), (3, True)])
def test_row_steps_match_tiles(nb, n, steps, valid):
    """Every buffer parity of the fused steps, with and without a valid state."""
    x, v, m = ics.random_cloud(n, seed=80 + n)
    tm, dt = dev(m), 1.0 / 256
    kw = dict(eps=0.05, precision="fp64")

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

    print("row steps n=%d steps=%d valid=%s" % (n, steps, valid), flush=True)
    both(nb, kdk)
    both(nb, h4)
    both(nb, h6)


@pytest.mark.parametrize("steps,every", [(0, 4), (1, 4), (5, 5), (6, 4), (7, 3)])
def test_row_gradient_matches_tiles(nb, steps, every):
    """The adjoint sweep with the update in the VJP's launch: even and odd step
    counts, one and several segments."""
    n = 257
    x, v, m = ics.random_cloud(n, seed=90)
    rng = np.random.default_rng(90)
    w = [dev(rng.standard_normal((3, n))) for _ in range(2)]

    def grad():
        t = [dev(a).requires_grad_(True) for a in (x, v, m)]
        out = nb.trajectory(*t, 1.0 / 128, steps, every=every, eps=0.05, precision="fp64")
        return list(o.detach() for o in out) + list(torch.autograd.grad(out, t, w, allow_unused=True))

    print("row gradient steps=%d every=%d" % (steps, every), flush=True)
    both(nb, grad)


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
            assert (p - q).abs().max().item() <= TOL * max(q.abs().max().item(), 1e-300), (p - q).abs().max().item()
