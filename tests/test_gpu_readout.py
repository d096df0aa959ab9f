"""GPU tests of the host side of setting and reading fields: the 16-bit conversions against
numpy's, and every way a window is fetched against the whole field."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _values(n, rng):
    """Momenta over the whole range of binary16: normal, subnormal, ties, their neighbours,
    values that round to infinity left out (set_geometry would store them, the step not)."""
    h = np.arange(n, dtype=np.uint16) % 0x7bff
    lo, hi = h.view(np.float16).astype(float), (h + 1).view(np.float16).astype(float)
    mid = 0.5 * (lo + hi)
    v = np.where(np.arange(n) % 3 == 0, mid, np.where(np.arange(n) % 3 == 1, np.nextafter(mid, 1), np.nextafter(mid, 0)))
    return np.where(np.arange(n) % 2 == 0, v, -v) * rng.choice([1.0, 1.0, 1e-3], n)


def _to_bf16(v):
    """bfloat16 of doubles, one rounding, half to even."""
    u = v.view(np.uint64)
    r = (u + ((u >> np.uint64(45)) & np.uint64(1)) + np.uint64((1 << 44) - 1)) & ~np.uint64((1 << 45) - 1)
    return r.view(np.float64)


@pytest.mark.parametrize("prec", ["f16s", "bf16s"])
def test_conversions_match_numpy(prec):
    from paper_1912_09327_amd.grid import Grid
    nx, ny = 256, 250
    rng = np.random.default_rng(3)
    v = _values(nx * ny, rng).reshape(ny, nx)
    g = Grid(nx, ny, prec=prec, periodic=3)
    try:
        g.set_geometry(None, np.ones((ny, nx)), v, -v)
        _, jx, jy = g.read_moments()
    finally:
        g.close()
    ref = v.astype(np.float16).astype(float) if prec == "f16s" else _to_bf16(v)
    assert np.array_equal(jx, ref) and np.array_equal(jy, -ref)


@pytest.mark.parametrize("prec", ["f64", "f16s"])
@pytest.mark.parametrize("more", [dict(), dict(planar=True), dict(populations=True, tau=0.8)])
def test_windows_are_the_field(prec, more):
    from paper_1912_09327_amd import inputs as I
    from paper_1912_09327_amd.grid import Grid
    nx, ny = 301, 180
    g = Grid(nx, ny, prec=prec, periodic=3, **more)
    try:
        g.set_geometry(None, *I.random_state(nx, ny, np.random.default_rng(5)))
        g.step(3)
        whole = g.read_moments()
        for x0, y0, w, h in ((0, 0, 1, ny), (nx - 1, 0, 1, ny), (17, 3, 1, 1), (0, 5, nx, 1), (40, 50, 200, 100),
                             (299, 179, 2, 1), (100, 0, 75, ny), (100, 0, 76, 2)):
            for a, b in zip(whole, g.read_window(x0, y0, w, h)):
                assert np.array_equal(a[y0:y0 + h, x0:x0 + w], b), (x0, y0, w, h)
    finally:
        g.close()
