"""What the tuners report, set with nbody_set_config: where the fastest form has no
setting of its own (the row kernels, the FP64 symmetric ensemble items), the reported one
set as reported gives that form, and anything else that is set the form it names.  The
forms are told apart by the last bits of FP64 results, whose sums run in another order."""
import json

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


def with_config(nb, f, **cfg):
    nb.nbody_set_config(**cfg)
    try:
        return f()
    finally:
        nb.nbody_set_config()


def test_tuned_force_set_as_reported(nb, tmp_path):
    n = 1003
    x, v, m = (dev(t) for t in ics.plummer(n, seed=9))
    force = lambda: nb.nbody_accel(x, m, eps=0.01, precision="fp64")
    vjp = lambda: nb.nbody_accel_vjp(x, m, v, eps=0.01, precision="fp64")[0]
    rows, rows_vjp = force(), vjp()
    path = str(tmp_path / "tune.jsonl")
    best = nb.nbody_tune(n, "fp64", path)
    print("tuned n=%d: %r" % (n, best))
    assert json.loads(open(path).read().splitlines()[-1])["rows"] == 1
    assert torch.equal(force(), rows)
    assert torch.equal(with_config(nb, force, **best), rows)
    assert torch.equal(with_config(nb, vjp, **best), rows_vjp)
    other = dict(best, split=best["split"] + 1)
    assert not torch.equal(with_config(nb, force, **other), rows)
    assert not torch.equal(with_config(nb, vjp, **other), rows_vjp)


def test_tuned_fp64_ensemble_set_as_reported(nb):
    sizes = [1500, 2111, 1730, 1999]
    off, epsv, x, v, m = ics.ensemble(len(sizes), seed=13, sizes=sizes)
    tx, tv, tm = dev(x), dev(v), dev(m)

    def accel():
        ta = torch.empty_like(tx)
        nb.nbody_step_batched(off, epsv, tx, tv, ta, tm, 1.0 / 512, 0, precision="fp64")
        return ta

    sym = accel()
    best = nb.nbody_tune_batched(off, epsv, tx, tv, tm, 1.0 / 512, 4, precision="fp64", allow_cooperative=False)
    best = {k: best[k] for k in ("bsplit", "bpass", "bitem")}
    print("tuned FP64 ensemble: %r" % best)
    assert torch.equal(accel(), sym)  # ten times as fast as the ordered items here
    assert torch.equal(with_config(nb, accel, **best), sym)
    other = dict(bsplit=0, bpass=2) if best["bsplit"] == 3 else dict(bsplit=3)
    assert not torch.equal(with_config(nb, accel, **other), sym)
