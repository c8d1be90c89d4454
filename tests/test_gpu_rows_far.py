"""The FP32C row force where most pairs are corrected and several rows of a workgroup
rescued: a cluster far from the origin (the repair radius and the error estimate grow with
|x|; at 100, 3 to 7 % of the rows are rescued), one of two such parts
(blocks of many corrections next to blocks of few, in one wave), at the edges of the launch
shapes (16 rows with marks in the pair loop, 16, 32, 16 in half workgroups, 32).

Against the tile kernels, which sum the same FP32 terms and corrections in the same order:
1e-9 of the largest value, as for the other row kernels' FP32C results; the rows rescued in
FP64 agree far better.
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


def with_config(nb, f, **cfg):
    nb.nbody_set_config(**cfg)
    try:
        return f()
    finally:
        nb.nbody_set_config()


@pytest.mark.parametrize("n", [70, 1000, 2048, 2049, 4097, 8193, 12288, 12289, 16384])
@pytest.mark.parametrize("rescue", [0, 2])
@pytest.mark.parametrize("far", ["all", "half"])
def test_row_force_far_from_the_origin(nb, n, rescue, far):
    x, _, m = ics.plummer(n, seed=n)
    x[:, :n if far == "all" else (n // 2 + 17)] += 100.0
    tx, tm = dev(x), dev(m)
    print("far force n=%d rescue=%d %s" % (n, rescue, far), flush=True)
    for eps, excl in ((0.01, False), (0.0, True)):
        f = lambda: nb.nbody_accel(tx, tm, eps=eps, precision="fp32c", exclude_self=excl)
        rows, tiles = with_config(nb, f, rescue=rescue), with_config(nb, f, rescue=rescue, ipl=1)
        assert torch.isfinite(rows).all()
        assert (rows - tiles).abs().max().item() <= 1e-9 * tiles.abs().max().item()


def test_row_force_far_from_the_origin_is_not_slower(nb):
    """9011 particles around 100: 147 us against the tile kernels' 151 (214 with turns for
    every correction, row by row rescues and two whole workgroups on some CUs)."""
    x, _, m = ics.plummer(9011, seed=1)
    tx, tm = dev(x + 100.0), dev(m)
    out = torch.empty_like(tx)

    def shortest_ms():
        ms = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                nb.nbody_accel(tx, tm, eps=0.01, precision="fp32c", out=out)
            b.record()
            b.synchronize()
            ms.append(a.elapsed_time(b) / 20)
        return min(ms)

    rows, tiles = shortest_ms(), with_config(nb, shortest_ms, ipl=1)
    print("force of 9011 around 100: rows %.3f ms, tiles %.3f ms" % (rows, tiles))
    assert rows <= 1.2 * tiles
