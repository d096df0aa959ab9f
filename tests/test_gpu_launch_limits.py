"""GPU test of the largest launches: a launch holds less than 2^32 threads, so a shape whose tiles
need more is refused, and the autotuner does not pick one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_region_shapes_past_a_launch_are_refused():
    """65536 x 4100 in regions of 32 x 32 on 1024 threads: 12 steps store 8 x 8 nodes of each,
    4.2 million blocks."""
    from paper_1912_09327_amd import _capi as C
    from paper_1912_09327_amd.grid import Grid
    nx, ny = 65536, 4100
    jx = np.zeros((ny, nx))
    spots = ((5, 7), (nx // 2, ny // 2), (nx - 70, ny - 40))
    rng = np.random.default_rng(1)
    for x, y in spots:
        jx[y:y + 30, x:x + 60] = 0.01 * rng.standard_normal((30, 60))
    windows = [(max(0, x - 20), max(0, y - 20), 70, 40) for x, y in spots]
    got = {}
    for how in ("gather", "tuned"):
        g = Grid(nx, ny, prec="f16s", periodic=3, snapshot=False)
        try:
            g.set_geometry(None, None, jx, None)
            if how == "tuned":
                with pytest.raises(C.Lbt1Error) as e:
                    g.set_kernel("strip", vec=32, rows=32, waves=16, fuse=12)
                assert e.value.status == C.EINVAL
                cfg, ms = g.autotune(6, 1)
                # 12 bytes a node and launch at 8 TB/s, over the steps of a launch
                assert ms > nx * ny * 12 / 8e12 * 1e3 / max(cfg["fuse"], 1), (cfg, ms)
            else:
                g.set_kernel("gather")
            g.step(12)
            got[how] = [g.read_window(*w) for w in windows]
        finally:
            g.close()
    for a, b in zip(got["gather"], got["tuned"]):
        for u, v in zip(a, b):
            assert np.array_equal(u, v)
    assert all(np.abs(a[1]).max() > 0 for a in got["gather"])
