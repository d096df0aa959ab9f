"""GPU tests of the batch's tile class (the default shape): every grid of a mix gets the
bits it gets alone, with budgets and bursts that are no multiple of a launch's steps, and
mixes small and large enough that every region shape is taken."""
import numpy as np
import pytest

from gpu_helpers import gpu_run
from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu

# nx, ny, periodic bits, wall rule, share of solid nodes, budget
SMALL = [(20, 15, 0, "paper", 0.0, 57), (33, 70, 1, "halfway", 0.1, 100), (61, 31, 3, "paper", 0.0, 41),
         (131, 77, 2, "halfway", 0.1, 1)]
MIXES = [SMALL, SMALL + [(700, 501, 1, "paper", 0.05, 33)],
         SMALL + [(1501, 1400, 0, "halfway", 0.01, 26), (1300, 1201, 1, "paper", 0.0, 9)]]


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("mix", range(len(MIXES)))
def test_tile_class_alone_vs_mix_bitwise(prec, mix):
    from paper_1912_09327_amd.batch import Batch
    from paper_1912_09327_amd.grid import Grid
    F = (1e-5, -2e-6)
    geos, grids = [], []
    for nx, ny, per, wall, frac, budget in MIXES[mix]:
        rng = np.random.default_rng(nx)
        geos.append((I.random_obstacles(nx, ny, frac, rng) if frac else None, *I.random_state(nx, ny, rng)))
        grids.append(Grid(nx, ny, prec=prec, wall=wall, periodic=per, force=F,
                          scale=(0.125, 0.0625) if nx == 61 else (0.0, 0.0)))
        grids[-1].set_geometry(*geos[-1])
    b = Batch(sum(g.nbytes for g in grids) + (1 << 20), len(grids))
    try:
        slots = [b.admit(g, m[5]) for g, m in zip(grids, MIXES[mix])]
        assert b.shape()["rows"] == [0] * 5
        while len(b.poll()) < len(grids):
            b.run(23)
        for s, m in zip(slots, MIXES[mix]):
            assert b.slot_info(s)[1] == m[5]
            b.evict(s)
        for g, geo, m in zip(grids, geos, MIXES[mix]):
            nx, ny, per, wall, _, budget = m
            ref = gpu_run(*geo, budget, prec, wall, per, F, kernel=dict(kernel="gather"),
                          scale=(0.125, 0.0625) if nx == 61 else (0.0, 0.0))
            for a, c in zip(g.read_moments(), ref):
                assert np.array_equal(a, c), m
    finally:
        b.close()
        for g in grids:
            g.close()
