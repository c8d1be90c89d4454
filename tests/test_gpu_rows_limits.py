"""Where the row kernels' force ends: above, the automatic choice is the tile kernels
with their own j-split.  The row kernels need hardly any scratch, the tile kernels' slices need
megabytes of it at these sizes: after a release of the workspace the free device memory
tells which ran."""
import numpy as np
import pytest

import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,rows", [("fp32", 16383, True), ("fp32", 16384, False), ("fp32", 20000, False),
                                         ("fp32c", 16384, True), ("fp32c", 16385, False), ("fp32c", 24576, False)])
def test_force_route_at_the_limits(prec, n, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_02744_amd as nb
    x, _, m = (torch.tensor(np.ascontiguousarray(t), device="cuda:0") for t in ics.plummer(n, seed=n))
    a, tiles = torch.empty_like(x), torch.empty_like(x)

    def scratch(out):
        torch.cuda.synchronize()
        nb.nbody_finalize()
        free = torch.cuda.mem_get_info()[0]
        nb.nbody_accel(x, m, eps=0.01, precision=prec, out=out)
        torch.cuda.synchronize()
        return free - torch.cuda.mem_get_info()[0]

    nb.nbody_accel(x, m, eps=0.01, precision=prec, out=a)  # the code object is loaded
    used = scratch(a)
    nb.nbody_set_config(ipl=1)
    try:
        tile_used = scratch(tiles)
    finally:
        nb.nbody_set_config()
    print("force %s n=%d: scratch %d, tiles' %d bytes" % (prec, n, used, tile_used))
    assert tile_used > 1 << 20
    assert used < tile_used // 2 if rows else used == tile_used
    assert (a - tiles).abs().max().item() <= 1e-9 * tiles.abs().max().item()
