"""The plans that the symmetric ensemble items keep per layout (their slots take up to 1
GiB each): a bound on what they hold together, plans given back and built again with
the same results, a captured plan that stays; and FP64 layouts whose slots find no room,
which take the ordered items from then on, also under capture."""
import numpy as np
import pytest

import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
GIB = 1 << 30


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nbm
    nbm.load()
    yield nbm
    nbm.nbody_finalize()


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def held(nb, free0):
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return free0 - torch.cuda.mem_get_info()[0]


def test_plans_are_bounded_and_captured_ones_stay(nb):
    n = 66000  # 0.1875 n^2 bytes of slots: 780 MiB
    x, _, m = ics.plummer(n, seed=4)
    tx, tm = dev(x), dev(m)
    ta, tv = torch.empty_like(tx), torch.zeros_like(tx)

    def accel(k, out):  # layout k: all particles but k in one system, then one of k
        nb.nbody_step_batched([0, n - k, n], [0.01, 0.02], tx, tv, out, tm, 1.0 / 512, 0, precision="fp64")
        return out

    torch.cuda.synchronize()
    nb.nbody_finalize()
    first = accel(1, ta).clone()
    small = dict(off=[0, 500, 1100], eps=[0.01, 0.02])
    sx, sv, sm = tx[:, :1100].contiguous(), torch.zeros(3, 1100, dtype=torch.float64, device="cuda:0"), tm[:1100].contiguous()
    sa = torch.empty_like(sx)
    nb.nbody_step_batched(small["off"], small["eps"], sx, sv, sa, sm, 1.0 / 512, 0, precision="fp64")
    ref = sa.clone()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        nb.nbody_step_batched(small["off"], small["eps"], sx, sv, sa, sm, 1.0 / 512, 0, precision="fp64")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free0 = torch.cuda.mem_get_info()[0]
    for k in range(2, 17):
        accel(k, ta)
        print("layout %d: %.2f GiB held" % (k, held(nb, free0) / GIB), flush=True)
    assert held(nb, free0) <= 9 * GIB  # 15 layouts of 0.76
    sa.zero_()
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(sa, ref)
    assert torch.equal(accel(1, ta), first)


def test_no_room_for_the_slots(nb):
    """With 256 to 512 MiB of the card's memory left, a layout whose slots take 980 MiB."""
    n = 74000
    x, v, m = ics.plummer(n, seed=5)
    tx, tv, tm = dev(x), dev(v), dev(m)
    off, eps = [0, n], [0.01]
    ta = torch.empty_like(tx)
    nb.nbody_set_config(bsplit=3)
    try:
        nb.nbody_step_batched(off, eps, tx, tv, ta, tm, 1.0 / 512, 0, precision="fp64")
    finally:
        nb.nbody_set_config()
    ordered = ta.clone()
    torch.cuda.synchronize()
    nb.nbody_finalize()
    torch.cuda.empty_cache()
    fill, chunk = [], 256 << 20
    try:
        while len(fill) < 2048:
            try:
                fill.append(torch.empty(chunk, dtype=torch.uint8, device="cuda:0"))
            except torch.OutOfMemoryError:
                break
        assert len(fill) < 2048
        print("%d chunks of 256 MiB fit" % len(fill), flush=True)
        del fill[-1:]
        torch.cuda.empty_cache()
        nb.nbody_step_batched(off, eps, tx, tv, ta, tm, 1.0 / 512, 0, precision="fp64")
        assert torch.equal(ta, ordered)
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g):
            nb.nbody_step_batched(off, eps, tx, tv, ta, tm, 1.0 / 512, 0, precision="fp64")
        for _ in range(3):
            ta.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(ta, ordered)
        del g
    finally:
        fill.clear()
        torch.cuda.empty_cache()
        torch.cuda.synchronize()
        nb.nbody_finalize()
