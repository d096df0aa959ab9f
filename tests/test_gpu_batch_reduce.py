"""GPU test of the batch's per-grid diagnostics: grids of one node more and less than a
reduction chunk (4096 nodes) and than a block (256), narrower and wider than a block, give
the residual that each gives alone, and refresh its snapshot."""
import numpy as np
import pytest

from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s"])
def test_batch_residuals_equal_those_of_the_grids_alone(prec):
    """A maximum over the same values does not depend on the order: equal bits."""
    from paper_1912_09327_amd.batch import Batch
    from paper_1912_09327_amd.grid import Grid
    shapes = [(64, 64), (63, 65), (17, 241), (3, 3), (4097, 3), (300, 7), (255, 17), (256, 33), (257, 100)]
    b = Batch(1 << 30, len(shapes))
    pairs = []
    try:
        for k, (nx, ny) in enumerate(shapes):
            rho, jx, jy = I.random_state(nx, ny, np.random.default_rng(40 + k))
            flags = None if k % 2 else (np.random.default_rng(60 + k).random((ny, nx)) < 0.1).astype(np.uint8)
            gs = [Grid(nx, ny, prec=prec, periodic=3) for _ in range(2)]
            for g in gs:
                g.set_geometry(flags, rho, jx, jy)
            pairs.append((b.admit(gs[0], 1000), gs[0], gs[1]))
        for n in (7, 5):
            b.run(n)
            b.poll()
            for slot, _, alone in pairs:
                alone.step(n)
                assert b.slot_info(slot)[2] == alone.reduce()["residual"]
    finally:
        b.close()
        for _, g, h in pairs:
            g.close()
            h.close()
