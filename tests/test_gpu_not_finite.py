"""GPU tests of values that are not finite in the 2-D kernels that take several steps a launch: the
same nodes become infinite or NaN as with one thread per node (or, on population grids, one step a
launch), across the edges of regions, in their halo and beside walls."""
import numpy as np
import pytest

from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu

# edges of regions: those of 64 columns with halos of 4 to 10, and the grid's own
SPOTS = ((56, 28), (117, 60), (0, 0), (180, 95))


def _case(prec, walls, nx=190, ny=101):
    rng = np.random.default_rng(3)
    rho, jx, jy = I.random_state(nx, ny, rng)
    flags = I.random_obstacles(nx, ny, 0.1, rng) if walls else None
    for x, y in SPOTS:
        jx[y, x] = 1e200 if prec == "f64" else 1e39
        if walls:
            flags[max(0, y - 1):y + 2, max(0, x - 1):x + 2] = I.FLUID
            flags[y + 1, x] = I.SOLID
    return flags, rho, jx, jy


def _run(case, prec, wall, per, splits, kernel, **more):
    from paper_1912_09327_amd.grid import Grid
    flags, rho, jx, jy = case
    ny, nx = rho.shape
    g = Grid(nx, ny, prec=prec, wall=wall, periodic=per, **more)
    try:
        if kernel:
            g.set_kernel(kernel)
        g.set_geometry(flags, rho, jx, jy)
        for n in splits:
            g.step(n)
        return g.read_moments(), g.reduce(8)["nonfinite"]
    finally:
        g.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("walls,wall,per", [(False, "paper", 3), (True, "paper", 0), (True, "halfway", 1)])
@pytest.mark.parametrize("kind", ["single", "multiphase", "populations"])
def test_not_finite(kind, walls, wall, per, prec):
    more = dict(multiphase=(-4.2, 1.0)) if kind == "multiphase" else dict(populations=True, tau=0.8) if kind == "populations" else {}
    case = _case(prec, walls)
    a, na = _run(case, prec, wall, per, [1] * 7 if kind == "populations" else [7], None if kind == "populations" else "gather", **more)
    b, nb = _run(case, prec, wall, per, [7], None, **more)
    assert na == nb and na > len(SPOTS)
    for x, y in zip(a, b):
        assert np.array_equal(x, y, equal_nan=True)
    assert np.isfinite(a[1]).any()


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("wall", ["paper", "halfway"])
def test_not_finite_in_a_batch(prec, wall):
    """The grid beside it stays what it is alone."""
    from paper_1912_09327_amd.batch import Batch
    from paper_1912_09327_amd.grid import Grid
    case = _case(prec, True)
    clean = (case[0], np.ones_like(case[1]), np.zeros_like(case[1]), 1e-3 * (case[0] == I.FLUID))
    grids = []
    for flags, rho, jx, jy in (case, clean):
        grids.append(Grid(190, 101, prec=prec, wall=wall, periodic=1))
        grids[-1].set_geometry(flags, rho, jx, jy)
    b = Batch(1 << 28, 2)
    try:
        slots = [b.admit(g, 100) for g in grids]
        b.run(7)
        assert [b.slot_info(s)[0] for s in slots] == [4, 1]  # non-finite, running
        for s in slots:
            b.evict(s)
        for g, c in zip(grids, (case, clean)):
            ref, _ = _run(c, prec, wall, 1, [7], "gather")
            for x, y in zip(ref, g.read_moments()):
                assert np.array_equal(x, y, equal_nan=True)
    finally:
        b.close()
        for g in grids:
            g.close()
