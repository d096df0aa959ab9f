"""CPU tests of the index arithmetic of k_step3_march, modelled on the host: every node is
stored once, every load stays inside the grid, and every store that is not the block's lies
past the end of its buffer."""
import numpy as np
import pytest

W, NOWHERE = 64, 1 << 30


def wrap(c, n):
    return np.mod(c, n)


def chunking(nx, ny, nz, rows, slots):
    tx, ty = -(-nx // W), -(-ny // (rows - 2))
    best, zc = None, 0
    for chunks in range(1, nz + 1):
        c = -(-nz // chunks)
        cost = -(-tx * ty * -(-nz // c) // slots) * (c + 2)
        if best is None or cost < best:
            best, zc = cost, c
    return tx, ty, -(-ny // ty), zc


@pytest.mark.parametrize("rows", [14, 22, 30])
@pytest.mark.parametrize("nx,ny,nz", [(3, 3, 1), (64, 28, 2), (65, 29, 3), (200, 57, 40), (24, 224, 25), (130, 20, 64)])
@pytest.mark.parametrize("size", [2, 4, 8])
def test_march_tiles_store_every_node_once(nx, ny, nz, rows, size):
    tx, ty, oy, zc = chunking(nx, ny, nz, rows, 256)
    assert oy <= rows - 2 and oy * ty >= ny
    rs = 4 * -(-nx // 64) * 64
    tiles = tx * ty * -(-nz // zc)
    per = -(-tiles // 8)
    count = np.zeros((nz, ny, nx), np.int32)
    taken = np.zeros(tiles, np.int32)
    r = np.arange(rows)
    for b in range(8 * per):
        t = (b & 7) * per + (b >> 3)
        if t >= tiles:
            continue
        taken[t] += 1
        z, rest = divmod(t, tx * ty)
        y, x = divmod(rest, tx)
        col, row = x * W + np.arange(W), y * oy - 1 + r
        z0, z1 = z * zc, min(nz, (z + 1) * zc)
        # the offset of a load inside its plane
        off = wrap(row, ny)[:, None] * rs + wrap(col, nx)[None, :]
        assert off.min() >= 0 and off.max() + 3 * (rs // 4) < rs * ny and off.max() * size < 2**32 * (size // 4 or 1)
        # the offset of a store inside the rows of the tile
        mine = (col < nx)[None, :] & ((r >= 1) & (r <= oy) & (row < ny))[:, None]
        to = np.where(mine, ((r - 1)[:, None] * rs + col[None, :]) * size, NOWHERE)
        end = rows * rs * size
        assert end <= NOWHERE and (to[mine] < end).all()
        ys = y * oy + (r - 1)
        assert (ys[r >= 1] >= 0).all()
        for zz in range(z0, z1):
            count[zz, np.repeat(row, W).reshape(rows, W)[mine], np.tile(col, rows).reshape(rows, W)[mine]] += 1
    assert (taken == 1).all() and (count == 1).all()


def test_march_flag_planes_run_ahead_of_the_moments():
    """Slots of the planes' SOLID bits (four) and of the halo columns' (four): what a plane's
    iteration reads was written before the barrier it follows and is not yet written over."""
    zb, ze = -1, 20
    for z in range(zb, ze + 1):
        halo_writes, main_reads = (z + 3) & 3, {(z + 2) & 3}
        own_reads = (z + 1) & 3  # the halo columns' own, for the emissions of the next plane
        assert halo_writes not in main_reads | {own_reads}
        rows_written, rows_read_late = (z + 2) & 3, (z + 1) & 3  # the second: by a wavefront one barrier behind
        assert rows_written != rows_read_late
