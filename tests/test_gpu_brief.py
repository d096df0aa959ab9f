"""GPU tests of calls of one and two steps, which may take another kernel than longer ones (a launch
a step, or a strip): any mix of short and long calls gives the bits of one long call, and of the
one-thread-per-node kernel where a grid has it."""
import numpy as np
import pytest

from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu

SPLITS = ([1] * 13, [2] * 6 + [1], [5, 1, 2, 2, 1, 2], [13])


def _runs(nx, ny, prec, wall, per, flags, more, scale=(0.0, 0.0)):
    from paper_1912_09327_amd.grid import Grid
    geo = I.random_state(nx, ny, np.random.default_rng(nx), 1e-3, 1e-3)
    out = []
    for splits in SPLITS:
        g = Grid(nx, ny, prec=prec, wall=wall, periodic=per, force=(1e-5, -2e-6), scale=scale, **more)
        try:
            g.set_geometry(flags, *geo)
            for n in splits:
                g.step(n)
            out.append(g.read_moments())
        finally:
            g.close()
    return geo, out


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("wall,per", [("paper", 3), ("paper", 0), ("halfway", 1)])
@pytest.mark.parametrize("nx,ny", [(64, 32), (130, 77), (384, 384), (517, 400), (1030, 1100)])
def test_populations_short_calls(nx, ny, prec, wall, per):
    flags = I.random_obstacles(nx, ny, 0.1, np.random.default_rng(ny)) if wall == "halfway" else None
    _, out = _runs(nx, ny, prec, wall, per, flags, dict(populations=True, tau=0.8), (0.125, 0.0625) if nx == 130 else (0.0, 0.0))
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("multiphase", [False, True])
@pytest.mark.parametrize("nx,ny", [(702, 715), (900, 1100), (1001, 980), (1024, 1500)])
def test_periodic_short_calls(nx, ny, multiphase, prec):
    """Around the sizes where short calls change over to strips (one of odd width, which has none)."""
    geo, out = _runs(nx, ny, prec, "paper", 3, None, dict(multiphase=(-4.2, 1.0)) if multiphase else {},
                     (0.125, 0.0625) if nx == 900 else (0.0, 0.0))
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("prec", ["f32", "f16s"])
def test_large_periodic_short_calls(prec):
    """Four columns a lane: from 12 million nodes in FP32 (three steps too), 20 in 16-bit storage."""
    from paper_1912_09327_amd.grid import Grid
    nx, ny = (4096, 3000) if prec == "f32" else (5000, 4100)
    jx = np.zeros((ny, nx))
    jx[100:140, 40:200] = 1e-2 * np.random.default_rng(1).standard_normal((40, 160))
    jx[ny - 30:, nx - 90:] = 1e-2 * np.random.default_rng(2).standard_normal((30, 90))
    out = []
    for splits in ([1, 1, 1, 2, 2, 3, 3], [13]):
        g = Grid(nx, ny, prec=prec, periodic=3, snapshot=False)
        try:
            if len(splits) == 1:
                g.set_kernel("gather")
            g.set_geometry(None, None, jx, None)
            for n in splits:
                g.step(n)
            out.append([g.read_window(*w) for w in ((20, 80, 200, 80), (nx - 120, ny - 60, 120, 60), (0, 0, 40, 40))])
        finally:
            g.close()
    for a, b in zip(*out):
        for u, v in zip(a, b):
            assert np.array_equal(u, v)
