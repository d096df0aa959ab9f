"""GPU tests of a batch that empties and takes grids of another storage precision: sizes, lists
and launch sizes are the same, so only the precision tells the burst graphs apart."""
import numpy as np
import pytest

from gpu_helpers import gpu_run
from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu

SIDES = (61, 64, 200)
# the two 16-bit formats first: they share every launch size and differ in the kernels alone
ORDER = ("f16s", "bf16s", "f32", "f16s", "f64", "f32")


@pytest.mark.parametrize("shape", [None, dict(fuse=0), dict(fuse=1), dict(lds=1)])
def test_emptied_batch_takes_another_precision(shape):
    from paper_1912_09327_amd.batch import Batch
    from paper_1912_09327_amd.grid import Grid
    geos = [I.cavity(n, 0.05) for n in SIDES]
    ref = {p: [gpu_run(*g[:4], 13, p, "paper", g[4], kernel=dict(kernel="gather")) for g in geos] for p in set(ORDER)}
    b = Batch(1 << 30, len(SIDES))
    try:
        if shape:
            b.set_shape(**shape)
        for prec in ORDER:
            grids = [Grid(n, n, prec=prec, periodic=g[4]) for n, g in zip(SIDES, geos)]
            for g, geo in zip(grids, geos):
                g.set_geometry(*geo[:4])
            slots = [b.admit(g, 1000) for g in grids]
            b.run(13)
            for s in slots:
                b.evict(s)
            for g, want in zip(grids, ref[prec]):
                for a, c in zip(g.read_moments(), want):
                    assert np.array_equal(a, c), (prec, g.nx)
                g.close()
    finally:
        b.close()
