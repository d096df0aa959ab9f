"""The tile kernels' work decomposition, modelled on the CPU (k_step_tile): for every region
shape built and every number of steps, each node is stored by exactly one block, every
load lies in the grid's rows (a chunk of two columns in the row pitch), and a stored node
is at least as many nodes from the region's edge as the launch takes steps, unless that
edge is a grid edge that is not periodic."""
import numpy as np
import pytest

# columns a thread, columns, rows of a region
SHAPES = [(1, 32, 32), (1, 64, 32), (1, 64, 64), (2, 128, 64)]


def tile_map(nx, ny, per, w, rows, halo):
    """halo: the steps of a launch, twice as many for multiphase grids."""
    even = (halo + 1) // 2 * 2
    hx = 0 if not per & 1 and nx <= w else even if w > 64 else halo
    hy = 0 if not per & 2 and ny <= rows else halo
    return hx, hy, w - 2 * hx, rows - 2 * hy


def lattice(first, count, n, periodic):
    """Positions first .. first + count - 1 on an axis of n nodes, as the kernel steps them."""
    out = [first if 0 <= first < n else first % n if periodic else -1]
    for c in range(1, count):
        if periodic:
            out.append(0 if out[-1] + 1 == n else out[-1] + 1)
        else:
            out.append(first + c if 0 <= first + c < n else -1)
    return np.array(out)


@pytest.mark.parametrize("cpl,w,rows", SHAPES)
@pytest.mark.parametrize("nx,ny", [(3, 3), (31, 32), (64, 33), (65, 20), (129, 64), (130, 131), (200, 77)])
@pytest.mark.parametrize("per", [0, 1, 2, 3])
def test_tiles_store_every_node_once_and_in_time(cpl, w, rows, nx, ny, per):
    pitch = (nx + 63) // 64 * 64
    px, py = bool(per & 1), bool(per & 2)
    for steps in (1, 2, 3, 4, 6, 8, 15, 64):
        hx, hy, ox, oy = tile_map(nx, ny, per, w, rows, steps)
        if ox < 1 or oy < 1:
            continue
        assert hx % cpl == 0 and ox % cpl == 0
        count = np.zeros((ny, nx), int)
        for ty in range(-(-ny // oy)):
            for tx in range(-(-nx // ox)):
                x, y = tx * ox - hx, ty * oy - hy
                for t in range(0, w, cpl):  # a thread's columns: stepped from its first
                    cols = lattice(x + t, cpl, nx, px)
                    assert ((cols >= 0) | (not px)).all() and (cols < nx).all()
                    if cpl > 1 and not (px and nx % cpl):  # loaded as one chunk
                        k = max(cols[0], 0)
                        assert k % cpl == 0 and k + cpl <= pitch
                assert (lattice(y, rows, ny, py) < ny).all()
                xs = np.arange(max(0, tx * ox), min(nx, (tx + 1) * ox))
                ys = np.arange(max(0, ty * oy), min(ny, (ty + 1) * oy))
                count[np.ix_(ys, xs)] += 1
                # distance of the stored nodes from the region's edges
                for lo, hi, first, size, n, periodic in ((xs[0], xs[-1], x, w, nx, px), (ys[0], ys[-1], y, rows, ny, py)):
                    assert lo - first >= steps or (not periodic and first >= 0 and first == 0)
                    assert first + size - 1 - hi >= steps or (not periodic and first + size >= n)
        assert (count == 1).all(), (steps,)
