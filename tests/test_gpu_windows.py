"""GPU tests of the ways a readout fetches its rows (whole rows in pieces, rows one by one, packed
on the device): each gives the values of the whole field, for windows of every shape, for one field
without the others, and for grids whose rows a piece does not hold whole numbers of."""
import ctypes

import numpy as np
import pytest

from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu

SUBSETS = [(0,), (1,), (2,), (0, 2), (1, 2), (0, 1, 2)]


def _window(g, x0, y0, w, h, want):
    from paper_1912_09327_amd import _capi as C
    out = [np.full((h, w), np.nan) if q in want else None for q in range(3)]
    C.check(C.lib.lbt1_read_window(g.handle, x0, y0, w, h, *[None if a is None else a.ctypes.data_as(C._dp) for a in out]))
    return out


# a column, a point, a row, narrow and wide windows; a piece of whole rows is 1 MiB
@pytest.mark.parametrize("nx,ny,prec,more", [
    (3000, 700, "f32", {}), (3000, 700, "f64", dict(planar=True)), (1501, 640, "f16s", {}),
    (1000, 300, "bf16s", dict(populations=True, tau=0.8)), (400, 333, "f64", dict(populations=True, tau=0.8)),
    (65536, 5, "f64", {}), (65536, 5, "f32", dict(planar=True)), (65, 9000, "f32", {})])
def test_every_way_gives_the_field(nx, ny, prec, more):
    from paper_1912_09327_amd.grid import Grid
    g = Grid(nx, ny, prec=prec, periodic=3, **more)
    try:
        rng = np.random.default_rng(nx)
        g.set_geometry(None, *I.random_state(nx, ny, rng))
        g.step(2)
        whole = g.read_moments()
        check = g.reduce(1 | 2)  # the reduction's workspace serves the readout in between
        for x0, y0, w, h in ((nx // 2, 0, 1, ny), (nx - 1, 1, 1, ny - 2), (7, 3, 1, 1), (0, ny // 2, nx, 1), (3, 1, 50, ny - 2),
                             (nx // 8, 0, nx // 4, ny), (1, 0, nx - 1, ny), (nx - 13, ny - 2, 13, 2)):
            for want in SUBSETS:
                for a, b in zip(whole, _window(g, x0, y0, w, h, want)):
                    assert b is None or np.array_equal(a[y0:y0 + h, x0:x0 + w], b), (x0, y0, w, h, want)
        assert g.reduce(1 | 2)["mass"] == check["mass"]
    finally:
        g.close()


@pytest.mark.parametrize("shape,prec", [((31, 45, 200), "f32"), ((3, 700, 130), "f64"), ((40, 33, 65), "f16s"),
                                        ((2, 3, 16384), "f64")])
def test_3d_fields_one_by_one(shape, prec):
    from paper_1912_09327_amd import _capi as C
    from paper_1912_09327_amd.grid3d import Grid3D
    nz, ny, nx = shape
    rng = np.random.default_rng(7)
    g = Grid3D(nx, ny, nz, q=19, prec=prec, periodic=7)
    try:
        g.set_geometry(None, 1 + 1e-2 * rng.standard_normal(shape), *[1e-2 * rng.standard_normal(shape) for _ in range(3)])
        whole = g.read_moments()
        for want in ((0,), (3,), (1, 2), (0, 3)):
            out = [np.full(shape, np.nan) if q in want else None for q in range(4)]
            C.check(C.lib.lbt1_grid3d_read_moments(
                g.handle, *[None if a is None else a.ctypes.data_as(ctypes.POINTER(ctypes.c_double)) for a in out]))
            for a, b in zip(whole, out):
                assert b is None or np.array_equal(a, b), want
    finally:
        g.close()


def test_a_column_does_not_move_the_grid():
    """The section probe of the stopping rules: well under the time that the field's 805 MB take."""
    import time
    from paper_1912_09327_amd.grid import Grid
    n = 8192
    g = Grid(n, n, prec="f32", periodic=3, snapshot=False)
    try:
        g.set_geometry()
        g.read_window(n // 2, 1, 1, n - 2)
        t0 = time.perf_counter()
        for _ in range(3):
            rho, jx, _ = g.read_window(n // 2, 1, 1, n - 2)
        assert (time.perf_counter() - t0) / 3 < 0.02  # 0.1 ms; 280 ms with whole rows
        assert np.all(rho == 1.0) and np.all(jx == 0.0)
    finally:
        g.close()
