"""GPU tests of steps recorded into a caller's graph: every replay goes on from where the one before
it ended, with the program's own steps and synchronizations in between, whatever number of steps a
launch of the grid's kernel takes."""
import numpy as np
import pytest

from paper_1912_09327_amd import inputs as I

pytestmark = pytest.mark.gpu

GRIDS = [("f64", 64, 32, {}), ("f32", 256, 256, {}), ("f32", 300, 211, dict(populations=True, tau=0.8)),
         ("f32", 200, 200, dict(multiphase=(-5.5, 1.0))), ("f64", 701, 503, {}), ("f16s", 180, 77, {})]


@pytest.mark.parametrize("prec,nx,ny,more", GRIDS)
@pytest.mark.parametrize("walls", [False, True])
def test_recorded_steps_replay(prec, nx, ny, more, walls):
    import torch
    from paper_1912_09327_amd.grid import Grid
    s = torch.cuda.Stream()
    geo = I.random_state(nx, ny, np.random.default_rng(nx))
    flags = I.channel(nx, ny)[0] if walls else None
    grids = [Grid(nx, ny, prec=prec, periodic=1 if walls else 3, stream=s, **more) for _ in range(2)]
    try:
        for n in (2, 3, 5, 10, 12, 25, 64, 131):
            for g in grids:
                g.set_geometry(flags, *geo)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=s, capture_error_mode="relaxed"):
                grids[0].step(n)
            for rep in range(4):
                with torch.cuda.stream(s):
                    graph.replay()
                grids[1].step(n)
                if rep == 1:  # the program's own steps (an even number of launches: the parity stays)
                    for g in grids:
                        g.step(1)
                        g.step(1)
                torch.cuda.synchronize()
                for a, b in zip(grids[0].read_moments(), grids[1].read_moments()):
                    assert np.array_equal(a, b, equal_nan=True), (n, rep)
    finally:
        for g in grids:
            g.close()
