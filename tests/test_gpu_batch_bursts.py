"""GPU test of a batch's bursts of one, two, three and more steps in any order: the tiles are cut
anew between short and longer ones, and every grid keeps the bits it gets alone."""
import numpy as np
import pytest

from gpu_helpers import gpu_run
from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu

GRIDS = [(20, 15, 0, "paper"), (131, 77, 2, "halfway"), (300, 211, 1, "paper"), (700, 501, 0, "halfway")]


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("bursts", [[1, 2, 3, 4, 3, 2, 1], [10, 1, 23, 3], [1] * 5])
def test_bursts_of_any_length(prec, bursts):
    from paper_1912_09327_amd.batch import Batch
    from paper_1912_09327_amd.grid import Grid
    geos, grids = [], []
    for nx, ny, per, wall in GRIDS:
        rng = np.random.default_rng(nx)
        geos.append((I.random_obstacles(nx, ny, 0.1, rng), *I.random_state(nx, ny, rng)))
        grids.append(Grid(nx, ny, prec=prec, wall=wall, periodic=per))
        grids[-1].set_geometry(*geos[-1])
    budgets = [sum(bursts)] * 3 + [sum(bursts) - 1]  # one grid ends inside the last burst
    b = Batch(sum(g.nbytes for g in grids) + (1 << 20), len(grids))
    try:
        slots = [b.admit(g, n) for g, n in zip(grids, budgets)]
        for k in bursts:
            b.run(k)
            b.shape()
        for s, n in zip(slots, budgets):
            assert b.slot_info(s)[1] == n
            b.evict(s)
        for g, geo, n, (nx, ny, per, wall) in zip(grids, geos, budgets, GRIDS):
            ref = gpu_run(*geo, n, prec, wall, per, kernel=dict(kernel="gather"))
            for a, c in zip(g.read_moments(), ref):
                assert np.array_equal(a, c), (nx, ny)
    finally:
        b.close()
        for g in grids:
            g.close()
