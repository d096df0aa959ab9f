"""GPU tests of the tile kernels (several steps per launch on regions held in registers):
every built shape must give the bits of single steps of the gather kernel."""
import numpy as np
import pytest

from gpu_helpers import JTOL, TOL, field_errors, gpu_run, oracle_run
from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu

GATHER = dict(kernel="gather")
# (columns, rows, wavefronts) of the regions built with and without walls
FREE = {"f64": [(32, 32, 8), (64, 32, 8), (64, 64, 8)],
        "f32": [(32, 32, 16), (64, 32, 16), (64, 64, 16), (128, 64, 8)]}
WALLED = {"f64": [(32, 32, 8), (64, 32, 8)],
          "f32": [(32, 32, 16), (64, 32, 16), (64, 64, 8)]}
FREE["f16s"] = FREE["bf16s"] = FREE["f32"]
WALLED["f16s"] = WALLED["bf16s"] = WALLED["f32"]


def _case(kind, nx, ny, seed):
    rng = np.random.default_rng(seed)
    rho, jx, jy = I.random_state(nx, ny, rng)
    if kind == "cavity":
        flags, r0, x0, y0, _ = I.cavity(nx, 0.08, ny)
        flags[ny // 2, nx // 3] = I.SOLID
        lid = flags == I.FIXED
        rho[lid], jx[lid], jy[lid] = r0[lid], x0[lid], y0[lid]
        return flags, rho, jx, jy, 0
    if kind == "obstacles":            # periodic in x, walls at y = -1 and y = ny
        return I.random_obstacles(nx, ny, 0.12, rng), rho, jx, jy, 1
    return None, rho, jx, jy, {"periodic": 3, "open": 0, "open_x": 2}[kind]


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("kind", ["periodic", "cavity", "obstacles", "open", "open_x"])
@pytest.mark.parametrize("wall", ["paper", "halfway"])
def test_tile_bitwise_equals_single_steps(prec, kind, wall):
    """Odd and even sides, grids that fit a region whole, smaller than a halo, of several
    tiles; a walled grid with interior regions; launches of 1, 4, 5 and 15 steps with
    remainders; a storage scale other than one."""
    if kind == "periodic" and wall == "halfway":
        pytest.skip("no walls")
    F = (1e-5, -2e-6)
    for nx, ny in ((61, 31), (64, 32), (9, 5), (131, 77), (300, 203)):
        flags, rho, jx, jy, per = _case(kind, nx, ny, nx + ny)
        scale = (2.0 ** -3, 2.0 ** -4) if nx == 131 else (0.0, 0.0)
        base = gpu_run(flags, rho, jx, jy, 23, prec, wall, per, F, kernel=GATHER, scale=scale)
        for w, rows, waves in (FREE if kind == "periodic" else WALLED)[prec]:
            for steps in (1, 4, 5, 15):
                cfg = dict(kernel="strip", vec=w, rows=rows, waves=waves, fuse=steps)
                got = gpu_run(flags, rho, jx, jy, 23, prec, wall, per, F, kernel=cfg, scale=scale)
                for a, b in zip(base, got):
                    assert np.array_equal(a, b), (nx, ny, w, rows, steps)


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s"])
def test_tile_bursts_splitting_and_whole_grids(prec):
    """Graph bursts, split calls, and a grid that fits one region taking 64 steps a launch."""
    from paper_1912_09327_amd.grid import Grid
    flags, rho, jx, jy, per = _case("cavity", 30, 31, 3)
    ref = gpu_run(flags, rho, jx, jy, 231, prec, "paper", per, kernel=GATHER)
    g = Grid(30, 31, prec=prec, periodic=per)
    try:
        for steps in (64, 6):
            g.set_geometry(flags, rho, jx, jy)
            g.set_kernel("strip", vec=32, rows=32, waves=8 if prec == "f64" else 16, fuse=steps)
            for n in (1, 64, 3, 128, 21, 2, 4, 5, 1, 2):
                g.step(n)
            for a, b in zip(ref, g.read_moments()):
                assert np.array_equal(a, b), steps
    finally:
        g.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("wall", ["paper", "halfway"])
def test_default_kernel_matches_oracle_on_odd_sides(prec, wall):
    """The library's choice on a porous grid of odd width, periodic in x."""
    from paper_1912_09327_amd.grid import Grid
    nx, ny = 173, 91
    flags, rho, jx, jy, per = _case("obstacles", nx, ny, 5)
    ref = oracle_run(flags, rho, jx, jy, 40, wall, per, (2e-5, 1e-5))
    g = Grid(nx, ny, prec=prec, wall=wall, periodic=per, force=(2e-5, 1e-5))
    try:
        g.set_geometry(flags, rho, jx, jy)
        assert "k_step_tile" in g.kernel()[1]
        g.step(40)
        ex, ej = field_errors(g.read_moments(), ref, flags)
    finally:
        g.close()
    assert ex <= TOL[prec] and ej <= JTOL[prec], (ex, ej)


def test_tile_refusals():
    from paper_1912_09327_amd import _capi as C
    from paper_1912_09327_amd.grid import Grid
    g = Grid(200, 100, prec="f32", periodic=3)
    try:
        g.set_geometry(None)
        for cfg in (dict(vec=32, rows=32, waves=16, fuse=16),     # the halo leaves nothing
                    dict(vec=32, rows=32, waves=16, fuse=65),
                    dict(vec=32, rows=32, waves=16, fuse=0),
                    dict(vec=64, rows=64, waves=8, fuse=4)):      # built with walls only (FP32)
            with pytest.raises(C.Lbt1Error) as e:
                g.set_kernel("strip", **cfg)
            assert e.value.status == C.EINVAL, cfg
        g.set_kernel("strip", vec=32, rows=32, waves=16, fuse=15)
        cfg, name = g.kernel()
        assert cfg == dict(kernel=2, vec=32, rows=32, waves=16, fuse=15) and "k_step_tile" in name
    finally:
        g.close()
    h = Grid(64, 64, prec="f32", periodic=3, multiphase=(-5.5, 1.0))
    try:
        h.set_geometry(None)
        with pytest.raises(C.Lbt1Error) as e:                     # a halo of two nodes a step
            h.set_kernel("strip", vec=32, rows=32, waves=8, fuse=8)
        assert e.value.status == C.EINVAL
        h.set_kernel("strip", vec=32, rows=32, waves=8, fuse=7)
    finally:
        h.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("kind", ["periodic", "obstacles", "open", "open_x"])
@pytest.mark.parametrize("wall", ["paper", "halfway"])
def test_multiphase_tile_bitwise_equals_single_steps(prec, kind, wall):
    """Every built shape against the gather kernel: drops over walls and grid edges, odd
    sides, grids smaller than a region, several tiles, a storage scale other than one."""
    from paper_1912_09327_amd import _capi as C
    from paper_1912_09327_amd.grid import Grid
    if kind == "periodic" and wall == "halfway":
        pytest.skip("no walls")
    for nx, ny in ((61, 31), (64, 32), (9, 5), (131, 77)):
        flags, _, _, _, per = _case(kind, nx, ny, nx)
        rng = np.random.default_rng(ny)
        y, x = np.mgrid[0:ny, 0:nx]
        rho = 0.11 + 1.1 * (1 - np.tanh((np.hypot(x - nx / 2, y - ny / 2) - min(nx, ny) / 4) / 2))
        rho *= 1 + 0.01 * rng.standard_normal(rho.shape)
        if flags is not None:
            rho[flags == I.SOLID] = 0.6
        jx, jy = (rho * 0.01 * rng.standard_normal(rho.shape) for _ in range(2))
        g = Grid(nx, ny, prec=prec, wall=wall, periodic=per, force=(1e-5, -2e-6), multiphase=(-5.5, 1.0),
                 scale=(0.125, 0.0625) if nx == 131 else (0.0, 0.0))
        try:
            g.set_geometry(flags, rho, jx, jy)
            assert "k_sc_tile" in g.kernel()[1]
            g.set_kernel("gather")
            g.step(9)
            base = g.read_moments()
            for w, rows in ((32, 32), (64, 32)) + (((64, 64),) if kind == "periodic" else ()):
                for steps in (1, 2, 5):
                    g.set_kernel("strip", vec=w, rows=rows, waves=8, fuse=steps)
                    g.set_geometry(flags, rho, jx, jy)
                    g.step(9)
                    for a, b in zip(base, g.read_moments()):
                        assert np.array_equal(a, b, equal_nan=True), (nx, ny, w, rows, steps)
        finally:
            g.close()
