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
