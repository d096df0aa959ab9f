"""GPU tests of the stored-population kernels that take several steps per launch: any
split of the steps (each with its own halo) gives the same bits, on grids small and
large enough that every region shape is taken, and FP64 agrees with the oracle."""
import numpy as np
import pytest

from oracle import bgk
from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu


def _case(kind, nx, ny):
    rng = np.random.default_rng(nx + ny)
    rho, jx, jy = I.random_state(nx, ny, rng)
    if kind == "cavity":
        flags, r0, x0, y0, _ = I.cavity(nx, 0.08, ny)
        flags[ny // 2, nx // 3] = I.SOLID
        lid = flags == I.FIXED
        rho[lid], jx[lid], jy[lid] = r0[lid], x0[lid], y0[lid]
        return flags, rho, jx, jy, 0
    if kind == "obstacles":
        return I.random_obstacles(nx, ny, 0.1, rng), rho, jx, jy, 1
    return None, rho, jx, jy, 3


def _run(case, prec, wall, splits, scale=(0.0, 0.0)):
    from paper_1912_09327_amd.grid import Grid
    flags, rho, jx, jy, per = case
    ny, nx = rho.shape
    g = Grid(nx, ny, prec=prec, wall=wall, periodic=per, force=(1e-5, -2e-6), scale=scale, populations=True, tau=0.8)
    try:
        g.set_geometry(flags, rho, jx, jy)
        for n in splits:
            g.step(n)
        return g.read_populations(), g.kernel()
    finally:
        g.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("kind,wall", [("periodic", "paper"), ("cavity", "paper"), ("cavity", "halfway"),
                                       ("obstacles", "halfway")])
def test_bgk_tile_splits_give_the_same_bits(prec, kind, wall):
    shapes = set()
    for nx, ny, n in ((9, 5, 25), (31, 33, 90), (131, 77, 25), (517, 400, 25), (1100, 1030, 13)):
        case = _case(kind, nx, ny)
        scale = (0.125, 0.0625) if nx == 131 else (0.0, 0.0)
        a, (cfg, name) = _run(case, prec, wall, [n], scale)
        b, _ = _run(case, prec, wall, [1] * n, scale)
        assert np.array_equal(a, b), (nx, ny)
        assert "k_bgk_tile" in name
        shapes.add((cfg["vec"], cfg["rows"]))
    assert len(shapes) >= 2, shapes


@pytest.mark.parametrize("wall", ["paper", "halfway"])
def test_bgk_tile_f64_matches_oracle_across_tiles(wall):
    """A porous grid of several regions, odd sides, against the brute-force solver."""
    nx, ny, n = 151, 67, 20
    flags, rho, jx, jy, per = _case("obstacles", nx, ny)
    got, _ = _run((flags, rho, jx, jy, per), "f64", wall, [n])
    o = bgk.BGK(rho, jx, jy, flags, per, (1e-5, -2e-6), bgk.WALL_PAPER if wall == "paper" else bgk.WALL_HALFWAY, 0.8)
    o.run(n, arrays=True)
    m = flags == I.FLUID
    assert np.abs(got - o.f)[:, m].max() <= 1e-12
