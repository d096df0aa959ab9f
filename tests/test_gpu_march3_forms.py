"""GPU tests of the forms in which the 3-D kernel goes through the planes, against one thread per
node, bit for bit: the ring over a periodic axis (thin grids), chunks of many planes with obstacles
(the flags run ahead of the moments for the whole chunk), and values that are not finite."""
import numpy as np
import pytest

from paper_1912_09327_amd import inputs as I
from test_gpu_3d import _case
from test_gpu_march3 import _run

pytestmark = pytest.mark.gpu

PRECS = ["f64", "f32", "f16s", "bf16s"]
F = (1e-5, 2e-6, -3e-6)


def _same(flags, rho, js, n, q, prec, wall, per, force=F):
    a = _run("gather", flags, rho, js, n, q, prec, wall, per, force)
    b = _run("tile", flags, rho, js, n, q, prec, wall, per, force)
    for x, y in zip(a, b):
        assert np.array_equal(x, y, equal_nan=True)
    return b


def _obstacles(shape, seed, share=0.12):
    rng = np.random.default_rng(seed)
    flags = (rng.random(shape) < share).astype(np.uint8)
    flags[rng.random(shape) < 0.02] = I.FIXED
    return flags


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("kind,per", [("periodic", 7), ("obstacles", 7), ("walls in x", 6), ("walls in y", 5), ("walls", 4)])
@pytest.mark.parametrize("ny,nx", [(3, 3), (12, 64), (13, 63), (25, 65), (24, 130)])
def test_ring_of_two_planes(ny, nx, kind, per, prec, q):
    """Around the edges of its tiles (64 columns, 12 rows); two planes, so the one above a node is
    the one below it as well."""
    shape = (2, ny, nx)
    _, rho, js, _ = _case("periodic", shape, 21)
    flags = _obstacles(shape, 22) if kind == "obstacles" else None
    for wall in ("paper", "halfway") if per != 7 or flags is not None else ("paper",):
        _same(flags, rho, js, 5, q, prec, wall, per)


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("nz", [3, 4, 8])
@pytest.mark.parametrize("wall", [None, "paper", "halfway"])
def test_ring_of_several_planes(nz, prec, q, wall):
    """Wide enough that all planes in one block are fewer than chunks and their neighbours."""
    shape = (nz, 500, 520)
    _, rho, js, _ = _case("periodic", shape, 23)
    flags = None if wall is None else _obstacles(shape, 24)
    _same(flags, rho, js, 3, q, prec, wall or "paper", 7)


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("wall", ["paper", "halfway"])
def test_long_chunks_with_obstacles(prec, q, wall):
    """200 x 180 x 150 in chunks of 17 to 38 planes, obstacles everywhere."""
    shape = (150, 180, 200)
    rng = np.random.default_rng(25)
    rho = 1.0 + 1e-2 * rng.standard_normal(shape, dtype=np.float32).astype(np.float64)
    js = [1e-2 * rng.standard_normal(shape, dtype=np.float32).astype(np.float64) for _ in range(3)]
    _same(_obstacles(shape, 26), rho, js, 2, q, prec, wall, 0 if wall == "paper" else 4)


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("wall", [None, "paper", "halfway"])
@pytest.mark.parametrize("nz", [1, 2, 21])
def test_not_finite(nz, prec, q, wall):
    """A momentum past the storage's range (FP64: whose square is past it) at a tile's edge: the same
    nodes become infinite or NaN, whatever lies around them."""
    shape = (nz, 45, 140)
    _, rho, js, _ = _case("periodic", shape, 27)
    flags = None
    if wall:
        flags = _obstacles(shape, 28)
        flags[nz // 2, 28:31, 62:66] = I.FLUID
        flags[nz // 2, 29, 66] = I.SOLID
    js[0][nz // 2, 28, 63] = 1e200 if prec == "f64" else 1e39
    js[1][nz // 2, 30, 64] = -1e200 if prec == "f64" else -1e39
    out = _same(flags, rho, js, 4, q, prec, wall or "paper", 7)
    bad = ~np.isfinite(out[1])
    assert bad.sum() > 4 and np.isfinite(out[1][:, :20]).all()
