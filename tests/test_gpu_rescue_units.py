"""The FP64 rescue's units: groups of rows times runs of j for one system (a few rows cut
into many runs, many rows into few or none), groups of rows of all systems of an ensemble
shared by one grid (few and many systems, systems without a listed row).

The rows that the rescue changed, found against the same call without it, have to be FP64
sums: within 1e-12 of the sum of their terms' magnitudes of a plain FP64 sum (both are off
by at most a few hundred units of 1.1e-16 of it, the square root of the number of terms),
where FP32C terms are off by some 1e-8 of it.
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


def check_rows(x, m, eps, a, rows):
    for i in rows:
        d = x - x[:, i:i + 1]
        t = m * d / ((d * d).sum(0) + eps * eps) ** 1.5
        err, bar = np.abs(a[:, i] - t.sum(1)), 1e-12 * np.abs(t).sum(1)
        assert (err <= bar).all(), (i, err, bar)


@pytest.mark.parametrize("n,form,eps", [(1025, dict(ipl=1, split=3), 1e-4), (1023, dict(ipl=1, split=1), 1e-4),
                                        (9000, dict(pairs=2), 1e-4), (9000, dict(pairs=2), 5e-3),
                                        (40001, dict(), 2e-3), (65536, dict(), 5e-3),
                                        (140001, dict(), 1e-2), (140001, dict(ipl=1, split=3), 1e-3)])
def test_single_system_rows(nb, n, form, eps):
    x, _, m = ics.plummer(n, seed=n)
    tx, tm = dev(x), dev(m)
    on, off = [], []
    for rescue, q in ((1, on), (2, off)):
        nb.nbody_set_config(rescue=rescue, **form)
        try:
            # twice: the counts and sums of a call leave nothing to the next
            q += [nb.nbody_accel(tx, tm, eps=eps, precision="fp32c").cpu().numpy() for _ in range(2)]
        finally:
            nb.nbody_set_config()
    assert np.array_equal(on[0], on[1])
    rows = np.flatnonzero((on[0] != off[0]).any(0))
    print("n=%d %s eps=%g: %d rows" % (n, form, eps, rows.size), flush=True)
    assert 0 < rows.size < n / 10
    check_rows(x, m, eps, on[0], rows[:: max(1, rows.size // 40)])


@pytest.mark.parametrize("mode", [3, 4])
@pytest.mark.parametrize("sizes", [[3000], [1, 700, 64], list(range(40, 340))])
def test_ensemble_rows(nb, mode, sizes):
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    parts = [ics.plummer(k, seed=7 + k) for k in sizes]
    x = np.concatenate([p[0] for p in parts], axis=1)
    v = np.concatenate([p[1] for p in parts], axis=1)
    m = np.concatenate([p[2] for p in parts])
    eps = np.full(len(sizes), 1e-4)
    got = []
    for rescue in (1, 2):
        nb.nbody_set_config(bsplit=mode, rescue=rescue)
        try:
            a = torch.empty((3, x.shape[1]), dtype=torch.float64, device="cuda:0")
            nb.nbody_step_batched(off, eps, dev(x), dev(v), a, dev(m), 0.01, 0, precision="fp32c")
            got.append(a.cpu().numpy())
        finally:
            nb.nbody_set_config()
    rows = np.flatnonzero((got[0] != got[1]).any(0))
    print("mode %d %d systems: %d rows" % (mode, len(sizes), rows.size), flush=True)
    assert 0 < rows.size < x.shape[1] / 2
    for i in rows[:: max(1, rows.size // 60)]:
        c = np.searchsorted(off, i, side="right") - 1
        s = slice(off[c], off[c + 1])
        check_rows(x[:, s], m[s], 1e-4, got[0][:, s], [i - off[c]])
