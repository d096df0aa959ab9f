"""Performance cases: the work a user of this framework has it do, through its public handles.

A pass is what a program repeats: advance a grid (or a batch) by a number of steps, then
the residual / non-finite check that the stopping rules are built on.  The check copies the
current state into the grid's residual snapshot, so the state after the pass is read in
place from the grid's device memory, laid out as include/lbt1.h documents.  A "request" is
a whole call on host data: create the grid, set its geometry, step, read the moments back.

Kinds: periodic (random field), cavity (lid-driven), channel (body force, round
obstacles, periodic in x), request (a channel from host arrays to host arrays), batch
(many uneven cavities), populations (stored-population BGK), drop (Shan-Chen), periodic3d
and box3d (D3Q19 / D3Q27).
"""
import math

import numpy as np
import torch

VALUE_BYTES = {"f64": 8, "f32": 4, "f16s": 2, "bf16s": 2}
TORCH = {"f64": torch.float64, "f32": torch.float32, "f16s": torch.float16, "bf16s": torch.bfloat16}
FLUID, SOLID, FIXED = 0, 1, 2
DROP_G = (-5.5, 1.0)


# ------------------------------------------------------------------------------- cases
def listed():
    return [
        # the Poiseuille test of the paper at its smallest: launches and latency
        dict(name="channel 64x32 f64", kind="channel", nx=64, ny=32, prec="f64", wall="paper", disks=0.0, steps=200),
        # the lid-driven cavity of the benchmark, checked every 100 steps
        dict(name="cavity 256 f32", kind="cavity", nx=256, ny=256, prec="f32", wall="paper", steps=100),
        # a grid with walls that fills the chip, sides no multiple of any tile
        dict(name="cavity 3000x2500 f32", kind="cavity", nx=3000, ny=2500, prec="f32", wall="paper", steps=100),
        # one served request: a porous channel of odd side in the server's storage, host to host
        dict(name="request porous 701 f16s", kind="request", nx=701, ny=701, prec="f16s", wall="halfway", disks=0.2,
             steps=1000),
        # the benchmark's periodic field, checked at the benchmark's cadence: the largest
        dict(name="periodic 8192 f32", kind="periodic", nx=8192, ny=8192, prec="f32", steps=99),
        # the same in 16-bit storage
        dict(name="periodic 4096 f16s", kind="periodic", nx=4096, ny=4096, prec="f16s", steps=100),
        # an odd-sided field in double precision
        dict(name="periodic 1501x1203 f64", kind="periodic", nx=1501, ny=1203, prec="f64", steps=100),
        # uneven cavities stepped together, as the server and the batch benchmark do
        dict(name="batch 40 cavities f16s", kind="batch", grids=40, lo=32, hi=512, prec="f16s", steps=100),
        # the standard method at tau != 1, as the method comparison runs it
        dict(name="populations 2048 f32", kind="populations", nx=2048, ny=2048, prec="f32", tau=0.8, periodic=True,
             steps=50),
        # the multiphase drop test
        dict(name="drop 1024 f32", kind="drop", nx=1024, ny=1024, prec="f32", channel=False, steps=100),
        # three dimensions: the periodic field, and the lid-driven box with ragged sides
        dict(name="periodic3d 256 q19 f32", kind="periodic3d", nx=256, ny=256, nz=256, q=19, prec="f32", steps=20),
        dict(name="box3d 200x180x150 q19 f32", kind="box3d", nx=200, ny=180, nz=150, q=19, prec="f32", wall="paper",
             steps=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["periodic", "periodic", "cavity", "cavity", "channel", "request", "batch", "populations", "drop",
                       "periodic3d", "box3d"])
    wall = rng.choice(["paper", "halfway"])
    prec = rng.choice(["f32", "f32", "f64", "f16s", "bf16s"])
    if kind == "periodic":
        return dict(kind=kind, nx=_log_int(rng, 48, 4096), ny=_log_int(rng, 48, 4096), prec=prec,
                    steps=rng.choice([60, 99, 100]))
    if kind == "cavity":
        return dict(kind=kind, nx=_log_int(rng, 32, 3000), ny=_log_int(rng, 32, 3000), prec=prec, wall=wall, steps=100)
    if kind == "channel":
        return dict(kind=kind, nx=_log_int(rng, 64, 2048), ny=_log_int(rng, 32, 2048), prec=rng.choice(["f32", "f64"]),
                    wall=wall, disks=rng.choice([0.0, 0.1, 0.3]), steps=100)
    if kind == "request":
        n = _log_int(rng, 32, 1500)
        return dict(kind=kind, nx=n, ny=n, prec="f16s", wall=wall, disks=round(rng.uniform(0.1, 0.3), 2),
                    steps=_log_int(rng, 500, 2000))
    if kind == "batch":
        return dict(kind=kind, grids=rng.randint(8, 40), lo=32, hi=rng.choice([128, 512]),
                    prec=rng.choice(["f16s", "f32"]), steps=100)
    if kind == "populations":
        return dict(kind=kind, nx=_log_int(rng, 50, 2048), ny=_log_int(rng, 50, 2048), prec=prec,
                    tau=round(rng.uniform(0.7, 1.5), 2), periodic=rng.random() < 0.6, steps=50)
    if kind == "drop":
        return dict(kind=kind, nx=_log_int(rng, 64, 2048), ny=_log_int(rng, 64, 2048), prec=rng.choice(["f32", "f64"]),
                    channel=rng.random() < 0.3, steps=50)
    dims = [_log_int(rng, 24, 224) for _ in range(3)]
    c = dict(kind=kind, nx=dims[0], ny=dims[1], nz=dims[2], q=rng.choice([19, 27]), prec=prec, steps=20)
    if kind == "box3d":
        c["wall"] = wall
    return c


# ------------------------------------------------------------------------------ inputs
def _normal(shape, seed):
    """Seeded standard normals made on the GPU, as host doubles."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).double().cpu().numpy()


def _disks(nx, ny, fraction, rng):
    """Rows 0 and ny - 1 solid, and round obstacles (periodic in x) over about `fraction` of the rest."""
    flags = np.zeros((ny, nx), np.uint8)
    flags[0], flags[-1] = SOLID, SOLID
    top = max(3.0, min(12.0, min(nx, ny) / 8.0))
    while fraction > 0 and (flags[1:-1] == SOLID).mean() < fraction:
        for _ in range(max(1, nx * ny // 5000)):
            r, cx, cy = rng.uniform(2.0, top), rng.uniform(0, nx), rng.uniform(1, ny - 2)
            ys = np.arange(max(1, int(cy - r)), min(ny - 2, int(cy + r) + 1) + 1)
            xs = np.arange(int(cx - r), int(cx + r) + 2)
            yy, xx = np.meshgrid(ys, xs, indexing="ij")
            hit = (xx - cx) ** 2 + (yy - cy) ** 2 <= r * r
            flags[yy[hit], np.mod(xx[hit], nx)] = SOLID
    return flags


def _cavity_inputs(nx, ny, lid):
    flags = np.zeros((ny, nx), np.uint8)
    flags[0], flags[:, 0], flags[:, -1] = SOLID, SOLID, SOLID
    flags[-1, 1:-1] = FIXED
    jx = np.zeros((ny, nx))
    jx[-1, 1:-1] = lid
    return flags, jx


def _inputs(case, seed):
    """Host arrays and settings of a single-grid case: flags, rho, momentum list, periodic bits, force."""
    kind, rng = case["kind"], np.random.default_rng(seed)
    if kind.endswith("3d"):
        shape, lid = (case["nz"], case["ny"], case["nx"]), float(rng.uniform(0.02, 0.08))
        g = _normal((4,) + shape, seed)
        rho = 1.0 + 1e-3 * g[0]
        j = [rho * 0.01 * g[1 + a] for a in range(3)]
        if kind == "periodic3d":
            return None, rho, j, 7, (0.0, 0.0, 0.0)
        flags = np.full(shape, SOLID, np.uint8)
        flags[1:-1, 1:-1, 1:-1] = FLUID
        flags[-1, 1:-1, 1:-1] = FIXED
        rho[flags != FLUID] = 1.0
        for a in range(3):
            j[a][flags != FLUID] = 0.0
        j[0][flags == FIXED] = lid
        return flags, rho, j, 0, (0.0, 0.0, 0.0)
    nx, ny = case["nx"], case["ny"]
    if kind == "cavity" or (kind == "populations" and not case["periodic"]):
        flags, jx = _cavity_inputs(nx, ny, float(rng.uniform(0.01, 0.1)))
        return flags, np.ones((ny, nx)), [jx, np.zeros((ny, nx))], 0, (0.0, 0.0)
    if kind in ("channel", "request"):
        u = float(rng.uniform(0.01, 0.1))
        force = (8.0 / 6.0 * u / (ny - 1) ** 2, 0.0)  # centre velocity u in an empty channel
        return _disks(nx, ny, case["disks"], rng), np.ones((ny, nx)), [np.zeros((ny, nx)) for _ in range(2)], 1, force
    if kind == "drop":
        y, x = np.mgrid[0:ny, 0:nx]
        R = min(nx, ny) / 4 * rng.uniform(0.9, 1.1)
        d = np.hypot(x - nx / 2 + rng.uniform(-2, 2), y - ny / 2 + rng.uniform(-2, 2))
        rho = 0.104 + (2.307 - 0.104) * 0.5 * (1 - np.tanh((d - R) / 2))
        flags, per = None, 3
        if case["channel"]:
            flags, per = _disks(nx, ny, 0.0, rng), 1
            rho[flags == SOLID] = 0.3
        return flags, rho, [np.zeros((ny, nx)) for _ in range(2)], per, (0.0, 0.0)
    g = _normal((3, ny, nx), seed)
    rho = 1.0 + 1e-3 * g[0]
    return None, rho, [rho * (0.01 * g[1]), rho * (0.01 * g[2])], 3, (0.0, 0.0)


def _batch_inputs(case, seed):
    """Side and lid speed of every cavity of a batch (one set of sides for every seed)."""
    sides = np.random.default_rng(1000 * case["grids"] + case["hi"])
    span = np.exp(sides.uniform(math.log(case["lo"]), math.log(case["hi"]), case["grids"]))
    return [int(round(s)) for s in span], np.random.default_rng(seed).uniform(0.01, 0.1, case["grids"])


# ----------------------------------------------------------------------------- prepare
def _up(n, to=256):
    return (n + to - 1) // to * to


def _state_view(buf, nx, ny, prec, populations=False, nz=None):
    """The residual snapshot inside a grid's device memory (include/lbt1.h): two parities,
    the flags, then one more copy of the fields."""
    c, pitch = VALUE_BYTES[prec], _up(nx, 64)
    rows = ny * (nz or 1)
    fields = 4 if nz else 3
    state = _up((9 if populations else fields) * pitch * rows * c)
    off = 2 * state + _up(pitch * rows)
    if populations:
        plane = _up(pitch * ny * c) // c
        v = buf[off:off + 3 * plane * c].view(TORCH[prec]).view(3, plane)[:, :pitch * ny]
        return v.view(3, ny, pitch)[:, :, :nx]
    v = buf[off:off + fields * pitch * rows * c].view(TORCH[prec])
    return v.view(*((nz,) if nz else ()), ny, fields, pitch)[..., :nx]


def _grid(case, force, per):
    from paper_1912_09327_amd.grid import Grid
    more = {}
    if case["kind"] == "populations":
        more = dict(populations=True, tau=case["tau"])
    if case["kind"] == "drop":
        more = dict(multiphase=DROP_G)
    return Grid(case["nx"], case["ny"], prec=case["prec"], periodic=per, force=force,
                wall=case.get("wall", "halfway" if case["kind"] == "drop" else "paper"), **more)


def prepare(case, seed):
    if case["kind"] == "batch":
        from paper_1912_09327_amd.batch import Batch
        from paper_1912_09327_amd.grid import Grid
        grids = []
        for side, lid in zip(*_batch_inputs(case, seed)):
            flags, jx = _cavity_inputs(side, side, lid)
            grids.append(Grid(side, side, prec=case["prec"], periodic=0))
            grids[-1].set_geometry(flags, np.ones_like(jx), jx, np.zeros_like(jx))
        b = Batch(sum(g.nbytes for g in grids) + (1 << 20), len(grids))
        slots = [b.admit(g, 1 << 40) for g in grids]
        return dict(case=case, batch=b, slots=slots, grids=grids,
                    views=[_state_view(g._buf, g.nx, g.ny, case["prec"]) for g in grids])
    flags, rho, j, per, force = _inputs(case, seed)
    if case["kind"] == "request":
        return dict(case=case, host=(flags, rho, *j), per=per, force=force)
    if case["kind"].endswith("3d"):
        from paper_1912_09327_amd.grid3d import Grid3D
        g = Grid3D(case["nx"], case["ny"], case["nz"], q=case["q"], prec=case["prec"], wall=case.get("wall", "paper"),
                   periodic=per)
        view = _state_view(g._buf, g.nx, g.ny, case["prec"], nz=g.nz)
    else:
        g = _grid(case, force, per)
        view = _state_view(g._buf, g.nx, g.ny, case["prec"], populations=case["kind"] == "populations")
    g.set_geometry(flags, rho, *j)
    return dict(case=case, grid=g, view=view)


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        state["batch"].run(case["steps"])
        return state["views"] + [np.array([state["batch"].slot_info(s)[2] for s in state["slots"]])]
    if case["kind"] == "request":
        with _grid(case, state["force"], state["per"]) as g:
            g.set_geometry(*state["host"])
            g.step(case["steps"])
            return g.read_moments()
    g = state["grid"]
    g.step(case["steps"])
    check = g.reduce()
    if case["kind"].endswith("3d"):
        return state["view"], check["nonfinite"], check["fluid"]
    return state["view"], check


# -------------------------------------------------------------------------------- work
def work(case):
    """State in and out once, the snapshot in and out, the flags in; FP operations of the
    update as the kernels' expressions count them (emission, arrivals, sums)."""
    kind, steps = case["kind"], case["steps"]
    c = VALUE_BYTES[case["prec"]]
    if kind == "batch":
        n = sum(s * s for s in _batch_inputs(case, 0)[0])
        return {"bytes": n * (12 * c + 1), "flops": 43 * n * steps}
    n = case["nx"] * case["ny"]
    if kind == "request":
        return {"bytes": n * (6 * 8 + 1), "flops": 43 * n * steps}
    if kind.endswith("3d"):
        n *= case["nz"]
        return {"bytes": n * (16 * c + (kind == "box3d")), "flops": n * steps * (120 if case["q"] == 19 else 160)}
    walled = kind in ("cavity", "channel") or case.get("channel") or not case.get("periodic", True)
    fields, flops = {"populations": (9, 70), "drop": (3, 85)}.get(kind, (3, 43))
    return {"bytes": n * ((2 * fields + 6) * c + walled), "flops": flops * n * steps}


# ------------------------------------------------------------------------------- exact
def _lattice(q):
    """Velocities (x, y, z) and weights."""
    if q == 9:
        e = [(x, y, 0) for x in (-1, 0, 1) for y in (-1, 0, 1)]
        w = [4 / 9, 1 / 9, 1 / 36]
    else:
        e = [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1) if q == 27 or abs(x) + abs(y) + abs(z) < 3]
        w = [1 / 3, 1 / 18, 1 / 36] if q == 19 else [8 / 27, 2 / 27, 1 / 54, 1 / 216]
    return [(v, w[sum(map(abs, v))]) for v in e]


class _Exact:
    """The method in 64 bits with plain torch: equilibria of every node, shifted and summed."""

    def __init__(self, q, flags, per, force, wall, tau=None, sc=None):
        self.lat, self.force, self.wall, self.tau, self.sc = _lattice(q), force, wall, tau, sc
        self.inv = {v: k for k, (v, _) in enumerate(self.lat)}
        self.walled = flags is not None
        if not self.walled:
            return
        f = torch.as_tensor(flags, device="cuda")
        self.fluid, self.fixed = f == FLUID, f == FIXED
        solid = f == SOLID
        dims = solid.dim()
        self.from_wall = []
        for (v, _) in self.lat:
            m = self._shift(solid, v)
            for a in range(dims):
                if v[a] and not per >> a & 1:
                    m.select(dims - 1 - a, 0 if v[a] > 0 else -1).fill_(True)
            self.from_wall.append(m)

    @staticmethod
    def _shift(a, v):
        """a at the upwind node x - v."""
        d = a.dim()
        return torch.roll(a, [v[k] for k in range(d)], [d - 1 - k for k in range(d)]) if any(v) else a.clone()

    def _equilibria(self, rho, J):
        u = [c / rho for c in J]
        base = 1.0 - 1.5 * sum(c * c for c in u)
        for v, w in self.lat:
            if not any(v):
                yield w * rho * base
                continue
            eu = sum(c * s for c, s in zip(u, v) if s)
            yield w * rho * (base + 3.0 * eu + 4.5 * eu * eu)

    def _forces(self, rho):
        if self.sc is None:
            return self.force
        psi = self.sc[1] * (1.0 - torch.exp(-rho / self.sc[1]))
        out = list(self.force)
        for v, w in self.lat:
            if any(v):
                back = self._shift(psi, tuple(-c for c in v))
                for a in range(len(out)):
                    if v[a]:
                        out[a] = out[a] - self.sc[0] * w * v[a] * psi * back
        return out

    def _arrivals(self, sent, rho):
        """What reaches every node, direction by direction; `sent` yields what leaves."""
        need_all = self.walled and self.wall == "halfway"
        sent = list(sent) if need_all else sent
        for k, s in enumerate(sent):
            v, w = self.lat[k]
            a = self._shift(s, v)
            if self.walled and any(v):
                back = sent[self.inv[tuple(-c for c in v)]] if need_all else w * rho
                a = torch.where(self.from_wall[k], back, a)
            yield k, a

    def _moments(self, arrivals, rho, dims):
        r, m = torch.zeros_like(rho), [torch.zeros_like(rho) for _ in range(dims)]
        for k, a in arrivals:
            r += a
            for c, s in zip(m, self.lat[k][0]):
                if s:
                    c += s * a
        return r, m

    def march(self, rho, j, n):
        dims = len(j)
        if self.tau is not None:
            return self._march_populations(rho, j, n)
        for _ in range(n):
            F = self._forces(rho)
            r, m = self._moments(self._arrivals(self._equilibria(rho, [c + f for c, f in zip(j, F)]), rho), rho, dims)
            if self.walled:
                r = torch.where(self.fluid, r, rho)
                m = [torch.where(self.fluid, a, b) for a, b in zip(m, j)]
            rho, j = r, m
        return rho, j

    def _march_populations(self, rho, j, n):
        dims, rho0, j0 = len(j), rho, j
        F = [self.tau * f for f in self.force]
        pops = list(self._equilibria(rho, j))
        for _ in range(n):
            post = [p + (e - p) / self.tau for p, e in zip(pops, self._equilibria(rho, [c + f for c, f in zip(j, F)]))]
            if self.walled:
                held = list(self._equilibria(rho0, [c + f for c, f in zip(j0, F)]))
                post = [torch.where(self.fixed, h, p) for h, p in zip(held, post)]
            pops = [a for _, a in self._arrivals(post, rho)]
            rho, j = self._moments(enumerate(pops), rho, dims)
            if self.walled:
                rho = torch.where(self.fluid, rho, rho0)
                j = [torch.where(self.fluid, a, b) for a, b in zip(j, j0)]
        return rho, j


def _exact_grid(case, flags, rho, j, per, force):
    """(rho, j) before and after the pass's steps."""
    kind = case["kind"]
    sim = _Exact(case.get("q", 9), flags, per, force, case.get("wall", "halfway" if kind == "drop" else "paper"),
                 tau=case.get("tau"), sc=DROP_G if kind == "drop" else None)
    first = torch.as_tensor(rho, device="cuda"), [torch.as_tensor(c, device="cuda") for c in j]
    return first, sim.march(*first, case["steps"])


def exact(case, seed):
    if case["kind"] == "batch":
        out, res = [], []
        for side, lid in zip(*_batch_inputs(case, seed)):
            flags, jx = _cavity_inputs(side, side, lid)
            (r0, j0), (r, j) = _exact_grid(case, flags, np.ones_like(jx), [jx, np.zeros_like(jx)], 0, (0.0, 0.0))
            out.append(torch.stack([r - 1.0, *j], 1))
            res.append(_residual(r0, j0, r, j, torch.as_tensor(flags == FLUID, device="cuda")))
        return out + [np.array(res)]
    flags, rho, j, per, force = _inputs(case, seed)
    (r0, j0), (r, j) = _exact_grid(case, flags, rho, j, per, force)
    if case["kind"] == "request":
        return tuple(a.cpu().numpy() for a in (r, *j))
    axis = 0 if case["kind"] == "populations" else r.dim() - 1
    state = torch.stack([r - 1.0, *j], axis)
    fluid = torch.ones_like(r, dtype=torch.bool) if flags is None else torch.as_tensor(flags == FLUID, device="cuda")
    if case["kind"].endswith("3d"):
        return state, 0.0, int(fluid.sum())
    # the net momentum of a symmetric flow is zero but for rounding: no value there
    mom = [None if case["kind"] in ("channel", "drop") else float(c[fluid].sum()) for c in j]
    check = dict(mass=float(r[fluid].sum()), mom_x=mom[0], mom_y=mom[1], residual=_residual(r0, j0, r, j, fluid),
                 nonfinite=0.0, fluid=int(fluid.sum()))
    return state, check


def _residual(r0, j0, r, j, fluid):
    return max(float((a / r - b / r0).abs()[fluid].max()) for a, b in zip(j, j0))
