"""CPU model of the LDS that k_step3_march passes between wavefronts: which slot of which array is
written and read between which barriers, by the wavefronts of rows and by those of the halo columns,
in the prologue and plane by plane.  Every read must find the plane it is meant for, written in an
earlier interval (or by the reader itself), and no slot may be written by one wavefront in an
interval in which another reads it.  The sizes of the rings are read from the source."""
import os
import re

import pytest

SRC = open(os.path.join(os.path.dirname(__file__), "..", "paper_1912_09327_amd", "csrc", "lbt1_3d.hpp")).read()


def _size(pattern):
    m = re.findall(pattern, SRC)
    assert len(m) == 1, pattern
    return int(m[0])


EDGE = _size(r"uint8_t edge\[(\d+)\]")
SOLID = _size(r"uint8_t solid\[(\d+)\]")
SIDE = _size(r"C side\[(\d+)\]")


class Clash(Exception):
    pass


class Lds:
    def __init__(self, sizes):
        self.sizes, self.now, self.old = sizes, [], {}

    def write(self, role, name, plane):
        self.now.append(("w", role, name, plane % self.sizes[name], plane))

    def read(self, role, name, plane):
        self.now.append(("r", role, name, plane % self.sizes[name], plane))

    def barrier(self):
        """Ends an interval.  Wavefronts of one role run freely against each other, except that a
        halo wavefront reads only edge bits it wrote itself."""
        for k, (op, role, name, slot, plane) in enumerate(self.now):
            if op != "r":
                continue
            own = [e for e in self.now[:k] if e[0] == "w" and e[1] == role == "side" and e[2:4] == (name, slot)]
            others = [e for e in self.now if e[0] == "w" and e[2:4] == (name, slot) and not (e[1] == role == "side")]
            if others:
                raise Clash(f"{name} slot {slot}: plane {plane} read while plane {others[0][4]} is written")
            found = own[-1][4] if own else self.old.get((name, slot))
            if found != plane:
                raise Clash(f"{name} slot {slot}: plane {plane} read, {found} found")
        for op, _, name, slot, plane in self.now:
            if op == "w":
                self.old[(name, slot)] = plane
        self.now = []


def march(form, walls, copies, planes, sizes, ahead=3):
    """form: "chunk" or "ring"; copies: of the row sums (two, or one and a second barrier)."""
    lds = Lds(dict(sizes, sums=copies))
    zb, ze = (0, planes - 1) if form == "ring" else (-1, planes)
    zf = zb - 1 if form == "ring" else zb

    def side_pre(z):  # before the barrier of plane z
        if z < ze:
            if walls:
                lds.read("side", "edge", z + 1)
            lds.write("side", "side", z + 1)
        if walls:
            lds.write("side", "edge", z + ahead)

    def rows_pre(z):
        lds.read("rows", "side", z)
        if walls:
            lds.read("rows", "edge", z + 2)
            lds.write("rows", "solid", z + 2)
        lds.write("rows", "sums", z)

    def rows_post(z):
        if walls:
            lds.read("rows", "solid", z + 2)
        lds.read("rows", "sums", z)

    if walls:
        for z in range(zf, zb + 3):
            lds.write("side", "edge", z)
        lds.read("side", "edge", zb)
    lds.write("side", "side", zb)
    lds.barrier()
    if walls:
        for z in range(zf, zb + 2):
            lds.read("rows", "edge", z)
            lds.write("rows", "solid", z)
        lds.barrier()
        for z in range(zf, zb + 2):
            lds.read("rows", "solid", z)
    for z in range(zb, ze + 1):
        side_pre(z)
        rows_pre(z)
        lds.barrier()
        rows_post(z)
        if copies == 1:
            lds.barrier()
    lds.barrier()


SIZES = dict(edge=EDGE, solid=SOLID, side=SIDE)


@pytest.mark.parametrize("form,copies", [("chunk", 2), ("chunk", 1), ("ring", 1)])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("planes", [1, 2, 3, 5, 40])
def test_every_plane_is_found(form, copies, walls, planes):
    if form == "ring" and planes < 2:
        pytest.skip("a ring has two planes or more")
    march(form, walls, copies, planes, SIZES)


@pytest.mark.parametrize("form,copies,change", [
    ("chunk", 2, dict(edge=2)), ("chunk", 2, dict(solid=2)), ("chunk", 2, dict(side=1)), ("ring", 1, dict(edge=3)),
    ("ring", 1, dict(solid=3)), ("ring", 1, dict(side=1))])
def test_a_shorter_ring_is_noticed(form, copies, change):
    with pytest.raises(Clash):
        march(form, True, copies, 5, dict(SIZES, **change))


def test_an_earlier_or_later_write_is_noticed():
    for ahead in (2, 4):
        with pytest.raises(Clash):
            march("chunk", True, 2, 8, SIZES, ahead=ahead)
    with pytest.raises(Clash):  # one copy of the sums needs its second barrier
        lds = Lds(dict(sums=1))
        lds.write("rows", "sums", 0)
        lds.barrier()
        lds.read("rows", "sums", 0)
        lds.write("rows", "sums", 1)
        lds.barrier()
