"""The FP64 symmetric ensemble items (the automatic FP64 choice for layouts whose
systems span several blocks of 64) against the ordered items (mode 3).

Layouts hold systems of one particle, one short of and one past a block, odd and
even numbers of blocks, and one large enough for several parts.  Both sides sum
the same FP64 terms in another order: 1e-12 of each system's largest component
(a few tens of units of 1.1e-16 of the terms' magnitudes) for the accelerations,
and for the states of three short steps.
"""
import numpy as np
import pytest

import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12
LAYOUTS = {
    "edges": [1, 63, 64, 65, 127, 128, 129, 191, 193, 700],
    "large": [2500, 64, 1025],
}


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nbm
    nbm.load()
    return nbm


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def run(nb, off, epsv, x, v, m, chunks, mode, **kw):
    tx, tv, tm = dev(x), dev(v), dev(m)
    ta = torch.full_like(tx, 7.0)
    nb.nbody_set_config(bsplit=mode)
    try:
        for k, c in enumerate(chunks):
            nb.nbody_step_batched(off, epsv, tx, tv, ta, tm, 1.0 / 512, c, precision="fp64", acc_valid=k > 0, **kw)
    finally:
        nb.nbody_set_config()
    return tx.cpu().numpy(), tv.cpu().numpy(), ta.cpu().numpy()


@pytest.mark.parametrize("layout", sorted(LAYOUTS))
@pytest.mark.parametrize("steps", [0, 1, 3])
@pytest.mark.parametrize("soft", [True, False])
def test_sym64_matches_ordered_items(nb, layout, steps, soft):
    sizes = LAYOUTS[layout]
    off, epsv, x, v, m = ics.ensemble(len(sizes), seed=91, sizes=sizes)
    if not soft:
        epsv = np.zeros_like(epsv)
    kw = dict(G=1.1, exclude_self=not soft)
    print("sym64 ensemble %s steps=%d soft=%s" % (layout, steps, soft), flush=True)
    got = run(nb, off, epsv, x, v, m, [steps], 0, **kw)
    ref = run(nb, off, epsv, x, v, m, [steps], 3, **kw)
    assert not np.array_equal(got[2], ref[2])  # another order of sums: the symmetric items ran
    for p, q in zip(got, ref):
        assert np.isfinite(p).all()
        for s, e in zip(off[:-1], off[1:]):
            assert np.abs(p[:, s:e] - q[:, s:e]).max() <= TOL * max(np.abs(q[:, s:e]).max(), 1e-300), (s, e)


def test_sym64_resumable_bitwise_and_graph(nb):
    sizes = LAYOUTS["edges"]
    off, epsv, x, v, m = ics.ensemble(len(sizes), seed=92, sizes=sizes)
    ref = run(nb, off, epsv, x, v, m, [6], 0)
    for chunks in ([6], [2, 4], [0, 1, 5]):
        for p, q in zip(ref, run(nb, off, epsv, x, v, m, chunks, 0)):
            assert np.array_equal(p, q), chunks
    tx, tv, tm = dev(x), dev(v), dev(m)
    ta = torch.empty_like(tx)
    kw = dict(precision="fp64")
    nb.nbody_step_batched(off, epsv, tx, tv, ta, tm, 1.0 / 512, 2, **kw)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream(), capture_error_mode="relaxed"):
        nb.nbody_step_batched(off, epsv, tx, tv, ta, tm, 1.0 / 512, 2, acc_valid=True, **kw)
    for k in range(2):
        g.replay()
        torch.cuda.synchronize()
        _ = (tx.sum() + 1.0).item()
    for p, q in zip(ref, (tx, tv, ta)):
        assert np.array_equal(p, q.cpu().numpy())
