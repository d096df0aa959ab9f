"""GPU tests of the 3-D kernel that marches through the planes (k_step3_march): at the edges of
its tiles (64 columns, 28, 20 or 12 rows), on grids of one, two and many planes and with chunks
of planes, it gives the bits of one thread per node; FP64 is held to the oracle."""
import numpy as np
import pytest

import oracle
from gpu_helpers import JTOL, TOL
from paper_1912_09327_amd import inputs as I
from test_gpu_3d import _case, _errors

pytestmark = pytest.mark.gpu


def _run(kernel, flags, rho, js, n, q, prec, wall, per, F):
    from paper_1912_09327_amd.grid3d import Grid3D
    nz, ny, nx = rho.shape
    g = Grid3D(nx, ny, nz, q=q, prec=prec, wall=wall, periodic=per, force=F)
    try:
        g.set_kernel(kernel)
        g.set_geometry(flags, rho, *js)
        g.step(n)
        return g.read_moments()
    finally:
        g.close()


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("kind,wall", [("periodic", "paper"), ("box", "paper"), ("box", "halfway"),
                                       ("plates", "halfway"), ("open", "paper"), ("open", "halfway")])
@pytest.mark.parametrize("shape", [(1, 29, 65), (2, 31, 64), (3, 57, 63), (37, 61, 197), (70, 13, 129)])
def test_march_bitwise_equals_gather(shape, kind, wall, prec, q):
    if kind == "box" and min(shape) < 3:
        pytest.skip("a box needs three nodes along every axis")
    flags, rho, js, per = _case(kind, shape, 11)
    F = (1e-5, 2e-6, -3e-6)
    a = _run("gather", flags, rho, js, 5, q, prec, wall, per, F)
    b = _run("tile", flags, rho, js, 5, q, prec, wall, per, F)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("kind,per", [("walls in z", 3), ("walls in y", 5), ("walls in x", 6), ("porous", 7)])
def test_march_partly_periodic_bitwise(kind, per, q):
    """One non-periodic axis at a time, and obstacles (with a FIXED node) in a periodic grid."""
    shape = (33, 45, 130)
    _, rho, js, _ = _case("periodic", shape, 13)
    flags = None
    if kind == "porous":
        flags = (np.random.default_rng(5).random(shape) < 0.15).astype(np.uint8)
        flags[7, 9, 64] = I.FIXED
    for wall in ("paper", "halfway"):
        a = _run("gather", flags, rho, js, 6, q, "f32", wall, per, (1e-5, 0.0, 0.0))
        b = _run("tile", flags, rho, js, 6, q, "f32", wall, per, (1e-5, 0.0, 0.0))
        for x, y in zip(a, b):
            assert np.array_equal(x, y), wall


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("kind,wall", [("periodic", "paper"), ("box", "paper"), ("box", "halfway"), ("open", "halfway")])
def test_march_f64_matches_oracle(kind, wall, q):
    """Several tiles along every axis; the tolerance of the other 3-D tests."""
    shape = (37, 61, 133)
    flags, rho, js, per = _case(kind, shape, 12)
    F = (1e-5, -2e-6, 3e-6)
    got = _run("tile", flags, rho, js, 12, q, "f64", wall, per, F)
    oracle.set_threads(16)
    ref = oracle.run3(rho, *js, 12, q, flags, per, F, oracle.WALL_PAPER if wall == "paper" else oracle.WALL_HALFWAY)
    ex, ej = _errors(got, ref, flags)
    assert ex <= TOL["f64"] and ej <= JTOL["f64"], (ex, ej)


@pytest.mark.parametrize("walls", [False, True])
def test_march_stores_past_the_caches_bitwise(walls):
    """A state of 256 MiB and more is stored with the non-temporal hint."""
    shape = (256, 256, 256)
    rng = np.random.default_rng(14)
    rho = 1.0 + 1e-2 * rng.random(shape, dtype=np.float32).astype(np.float64)
    js = [1e-2 * rng.random(shape, dtype=np.float32).astype(np.float64) for _ in range(3)]
    per = 6 if walls else 7
    a = _run("gather", None, rho, js, 2, 19, "f32", "paper", per, (0.0, 0.0, 0.0))
    b = _run("tile", None, rho, js, 2, 19, "f32", "paper", per, (0.0, 0.0, 0.0))
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("kind", ["periodic", "box"])
@pytest.mark.parametrize("shape", [(3, 5, 3), (2, 9, 65), (4, 33, 200), (33, 45, 131)])
def test_reductions_over_ragged_rows(shape, kind, prec):
    """Sums, counts and the residual against the stored snapshot, from the read moments, for rows
    that do not end with a thread's run of values: sums of n terms in FP64 in another order
    differ by at most n 2^-53 of the sum of magnitudes."""
    from paper_1912_09327_amd.grid3d import Grid3D
    if kind == "box" and min(shape) < 3:
        pytest.skip("a box needs three nodes along every axis")
    flags, rho, js, per = _case(kind, shape, 15)
    nz, ny, nx = shape
    g = Grid3D(nx, ny, nz, q=19, prec=prec, periodic=per)
    try:
        g.set_geometry(flags, rho, *js)
        old = g.read_moments()
        for n in (3, 4):
            g.step(n)
            new, d = g.read_moments(), g.reduce()
            m = np.ones(shape, bool) if flags is None else flags == I.FLUID
            assert d["fluid"] == int(m.sum()) and d["nonfinite"] == 0
            tol = rho.size * 2.0**-53
            assert abs(d["mass"] - new[0][m].sum()) <= 2 * tol * new[0][m].sum()
            for a in range(3):
                assert abs(d["mom"][a] - new[1 + a][m].sum()) <= 2 * tol * np.abs(new[1 + a][m]).sum()
            ref = max(np.abs(new[a] / new[0] - old[a] / old[0])[m].max() for a in (1, 2, 3))
            assert abs(d["residual"] - ref) <= 8 * 2.0**-53
            old = new
    finally:
        g.close()
