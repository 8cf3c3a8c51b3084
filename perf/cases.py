"""Performance cases of the isoAdvector framework: the work its users have it do, over the range of
sizes, cell types and options in use.

A case is one pass through the public entry points of ``paper_1804_01130_amd`` on a mesh, a plan and
fields that a flow solver holds already:

  step      one advection step (``Plan.step``)
  outer     one step of an outer iteration: averaged fields and the interpolated isoface velocity
  coupled   a wave tank's time step: advection with the statistics a solver logs, the relaxation
            zones' blend, then the ghost-fluid face data for the pressure equation
  run       several steps of one mesh in one call (``Plan.run``)
  ensemble  several steps of independent tanks advanced together (``Batch.advect``)
  gradient  a checkpointed trajectory and the gradient of a misfit (``autograd.advect``, backward)
  adjoint   a traced step and its vector-Jacobian product

Meshes: ``slab`` (one cell thick, periodic in x, y vertical), ``box`` (hexahedra graded towards the
still-water level, z vertical), ``prisms`` and ``tets`` (the box's cells cut), ``merged`` (pairs and
quadruples of the box's cells joined into polyhedra of 10 and 16 faces).  The surface is a column
beside random waves, the flow a stream plus a vortex array with a vector potential, integrated along
face edges so that it is free of divergence; amplitudes, wavelengths and phases come from the seed.
"""
from __future__ import annotations

import math
from collections import OrderedDict

import numpy as np
import torch

import paper_1804_01130_amd as iso
from paper_1804_01130_amd import autograd

WALL, EMPTY, CYCLIC = 0, 1, 3
RHO_HEAVY, RHO_LIGHT, GRAVITY = 1000.0, 1.2, 9.81


# ------------------------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest meshes: a 2D study, where launches and latency are all there is
        {"name": "slab_64x32", "op": "step", "mesh": "slab", "nx": 64, "ny": 32, "nz": 1},
        # an ordinary 2D wave tank
        {"name": "slab_1024x256", "op": "step", "mesh": "slab", "nx": 1024, "ny": 256, "nz": 1},
        # an outer iteration of a coupled solver on a small, ragged 3D box
        {"name": "outer_box_75x37x41", "op": "outer", "mesh": "box", "nx": 75, "ny": 37, "nz": 41},
        # a 3D wave tank coupled to a pressure solver, ragged sizes
        {"name": "coupled_box_151x75x85", "op": "coupled", "mesh": "box", "nx": 151, "ny": 75, "nz": 85},
        # the large 3D box: a violent surface, the headline workload
        {"name": "box_256x128x128", "op": "step", "mesh": "box", "nx": 256, "ny": 128, "nz": 128},
        # a 2D run in one call
        {"name": "run_slab_384x96", "op": "run", "mesh": "slab", "nx": 384, "ny": 96, "nz": 1, "steps": 10},
        # a parameter study: 64 tanks of 128..1024 x 64..256 cells with fields that change every step
        {"name": "ensemble_64", "op": "ensemble", "mesh": "slab", "members": 64, "layout": 1, "steps": 5},
        # unstructured meshes: tetrahedra, and polyhedra of a mesh with split faces
        {"name": "tets_48x24x24", "op": "step", "mesh": "tets", "nx": 48, "ny": 24, "nz": 24},
        {"name": "merged_64x32x32", "op": "step", "mesh": "merged", "nx": 64, "ny": 32, "nz": 32},
        # data assimilation: the gradient of a short 2D trajectory, and one 3D adjoint step
        {"name": "gradient_slab_256x128", "op": "gradient", "mesh": "slab", "nx": 256, "ny": 128, "nz": 1, "steps": 5},
        {"name": "adjoint_box_128x64x64", "op": "adjoint", "mesh": "box", "nx": 128, "ny": 64, "nz": 64},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["step"] * 6 + ["outer", "coupled", "run", "ensemble", "gradient", "adjoint"])
    if op == "ensemble":
        return {"op": op, "mesh": "slab", "members": size(3, 48), "layout": rng.randrange(1 << 16), "steps": rng.randint(2, 5)}
    if op in ("run", "gradient"):
        return {"op": op, "mesh": "slab", "nx": size(48, 512), "ny": size(24, 128), "nz": 1,
                "steps": rng.randint(3, 12) if op == "run" else rng.randint(2, 5)}
    if op in ("coupled", "outer"):
        return {"op": op, "mesh": "box", "nx": size(32, 200), "ny": size(20, 96), "nz": size(20, 96)}
    if op == "adjoint":
        return {"op": op, "mesh": "box", "nx": size(32, 128), "ny": size(20, 64), "nz": size(20, 64)}
    mesh = rng.choice(["slab", "slab", "box", "box", "box", "prisms", "tets", "merged"])
    if mesh == "slab":
        return {"op": op, "mesh": mesh, "nx": size(48, 1500), "ny": size(24, 300), "nz": 1}
    if mesh == "box":
        return {"op": op, "mesh": mesh, "nx": size(32, 250), "ny": size(20, 128), "nz": size(20, 128)}
    if mesh == "prisms":
        return {"op": op, "mesh": mesh, "nx": size(16, 64), "ny": size(12, 32), "nz": size(12, 32)}
    if mesh == "tets":
        return {"op": op, "mesh": mesh, "nx": size(12, 48), "ny": size(10, 24), "nz": size(10, 24)}
    return {"op": op, "mesh": mesh, "nx": size(16, 80), "ny": size(12, 40), "nz": size(12, 32)}


def _members(case):
    """Sizes of an ensemble's tanks."""
    rng = np.random.default_rng(case["layout"])
    return [(32 * int(rng.integers(4, 33)), 16 * int(rng.integers(4, 17))) for _ in range(case["members"])]


# ------------------------------------------------------------------------------------------ meshes
def _nodes(case):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["mesh"] == "slab":
        return np.linspace(0.0, nx / ny, nx + 1), np.linspace(0.0, 1.0, ny + 1), np.array([0.0, 1.0 / ny])
    t = np.linspace(-1.0, 1.0, nz + 1)  # cell heights 4:1 towards z = 1/2
    zs = 0.5 + 0.5 * np.sign(t) * np.expm1(np.log(4.0) * np.abs(t)) / 3.0
    return np.linspace(0.0, 2.0, nx + 1), np.linspace(0.0, 1.0, ny + 1), zs


class Grid:
    """A mesh in face-based form as host arrays: interior faces in upper-triangular order, then the
    patches xmin, xmax (cyclic), ymin, ymax, zmin, zmax; faces counter-clockwise from outside."""

    def __init__(self, case):
        self.xs, self.ys, self.zs = _nodes(case)
        nx, ny, nz = (len(v) - 1 for v in (self.xs, self.ys, self.zs))
        self.shape = (nz, ny, nx)
        Z, Y, X = np.meshgrid(self.zs, self.ys, self.xs, indexing="ij")
        self.points = np.stack([X.ravel(), Y.ravel(), Z.ravel()], 1)
        k, j, i = (v.ravel() for v in np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij"))
        P = lambda di, dj, dk: ((i + di) + (nx + 1) * ((j + dj) + (ny + 1) * (k + dk))).astype(np.int64)
        self.corner = np.stack([P(a, b, c) for c in (0, 1) for b in (0, 1) for a in (0, 1)], 1)  # x fastest
        self.side_kinds = [CYCLIC, CYCLIC, WALL, WALL] + ([EMPTY] * 2 if case["mesh"] == "slab" else [WALL] * 2)
        dv = [np.diff(v) for v in (self.xs, self.ys, self.zs)]
        vol = (dv[2][:, None, None] * dv[1][None, :, None] * dv[0][None, None, :]).ravel()
        kind = case["mesh"]
        if kind in ("prisms", "tets"):
            # local corner numbers: x + 2 y + 4 z; the splits match across faces and periodic sides
            if kind == "prisms":
                cells = [[(0, 3, 1), (4, 5, 7), (0, 1, 5, 4), (1, 3, 7, 5), (3, 0, 4, 7)],
                         [(0, 2, 3), (4, 7, 6), (0, 3, 7, 4), (3, 2, 6, 7), (2, 0, 4, 6)]]
            else:
                cells = []
                for a, b in ((1, 2), (2, 1), (1, 4), (4, 1), (2, 4), (4, 2)):  # paths 0 -> a -> a+b -> 7
                    t = (0, a, a + b, 7)
                    faces = [(t[1], t[2], t[3]), (t[0], t[3], t[2]), (t[0], t[1], t[3]), (t[0], t[2], t[1])]
                    even = (a, b) in ((1, 2), (2, 4), (4, 1))
                    cells.append(faces if even else [f[::-1] for f in faces])
            self._from_cells(cells)
            self.members, self.vol = len(cells), np.repeat(vol / len(cells), len(cells))
        else:
            self._hexahedra(i, j, k, nx, ny, nz)
            self.vol, self.members = vol, 1
            if kind == "merged":
                self._merge(i, j, k, nx, ny, vol)
        self.n_cells, self.n_faces, self.n_points = len(self.vol), len(self.owner), len(self.points)

    def _hexahedra(self, i, j, k, nx, ny, nz):
        c = np.arange(nx * ny * nz)
        loops = {"x+": (1, 3, 7, 5), "x-": (2, 0, 4, 6), "y+": (3, 2, 6, 7), "y-": (0, 1, 5, 4), "z+": (4, 5, 7, 6),
                 "z-": (0, 2, 3, 1)}
        inner = np.stack([i < nx - 1, j < ny - 1, k < nz - 1], 1)
        quads = np.stack([self.corner[:, loops[s]] for s in ("x+", "y+", "z+")], 1)
        own = np.repeat(c, 3).reshape(-1, 3)
        nbr = np.stack([c + 1, c + nx, c + nx * ny], 1)
        self.neighbour = nbr[inner].astype(np.int32)
        owner, quad = [own[inner]], [quads[inner]]
        self.patch_size = []
        for s, at in (("x-", i == 0), ("x+", i == nx - 1), ("y-", j == 0), ("y+", j == ny - 1), ("z-", k == 0), ("z+", k == nz - 1)):
            owner.append(c[at])
            quad.append(self.corner[at][:, loops[s]])
            self.patch_size.append(int(at.sum()))
        self.owner = np.concatenate(owner).astype(np.int32)
        self.quads = np.concatenate(quad).astype(np.int32)

    def _from_cells(self, cells):
        """Faces of the cut cells: a face met twice is interior, the others go to the block's sides."""
        n = len(self.corner)
        own, pts = [], []
        for q, faces in enumerate(cells):
            for f in faces:
                own.append(np.arange(n) * len(cells) + q)
                pts.append(self.corner[:, f if len(f) == 4 else f + (f[-1],)])
        own, pts = np.concatenate(own), np.concatenate(pts)
        key = np.sort(pts, 1)
        tri = pts[:, 2] == pts[:, 3]
        key[tri] = np.sort(np.concatenate([pts[tri][:, :3], np.full((int(tri.sum()), 1), -1)], 1), 1)
        order = np.lexsort((own, key[:, 3], key[:, 2], key[:, 1], key[:, 0]))
        own, pts, key = own[order], pts[order], key[order]
        same = np.all(key[1:] == key[:-1], 1)
        first = np.nonzero(same)[0]
        lone = np.ones(len(own), bool)
        lone[first] = lone[first + 1] = False
        by = np.lexsort((own[first + 1], own[first]))
        owner, quad = [own[first][by]], [pts[first][by]]
        self.neighbour = own[first + 1][by].astype(np.int32)
        lone = np.nonzero(lone)[0]
        cen = self.points[pts[lone]].mean(1)
        self.patch_size = []
        for axis, nodes in enumerate((self.xs, self.ys, self.zs)):
            flat = np.all(np.abs(self.points[pts[lone]][:, :, axis] - cen[:, None, axis]) < 1e-12, 1)
            for side in (0, -1):
                at = lone[flat & (np.abs(cen[:, axis] - nodes[side]) < 1e-12)]
                x = np.round(self.points[pts[at]][:, :3].mean(1), 9)  # the same order on opposite sides
                at = at[np.lexsort(tuple(x[:, d] for d in range(3) if d != axis))]
                owner.append(own[at])
                quad.append(pts[at])
                self.patch_size.append(len(at))
        self.owner = np.concatenate(owner).astype(np.int32)
        self.quads = np.concatenate(quad).astype(np.int32)

    def _merge(self, i, j, k, nx, ny, vol):
        """Joins cells: 2x2 in x and y where x is in an even pair of pairs, else pairs along x."""
        bx, odd = i // 2, (i // 4) % 2
        label = bx + (nx + 1) * (np.where(odd == 0, 2 * (j // 2), j) + (ny + 1) * k)
        _, cell = np.unique(label, return_inverse=True)
        ni = len(self.neighbour)
        a, b = cell[self.owner[:ni]], cell[self.neighbour]
        keep = a != b
        quad = self.quads[:ni][keep]
        a, b = a[keep], b[keep]
        quad = np.where((a > b)[:, None], quad[:, ::-1], quad)
        a, b = np.minimum(a, b), np.maximum(a, b)
        order = np.lexsort((b, a))
        self.owner = np.concatenate([a[order], cell[self.owner[ni:]]]).astype(np.int32)
        self.neighbour = b[order].astype(np.int32)
        self.quads = np.concatenate([quad[order], self.quads[ni:]])
        self.vol = np.bincount(cell, vol)
        self.cell = cell

    def create(self):
        tri = self.quads[:, 2] == self.quads[:, 3]
        ptr = np.concatenate([[0], np.cumsum(np.where(tri, 3, 4))])
        pts = self.quads.ravel()[np.stack([tri * 0 == 0] * 3 + [~tri], 1).ravel()] if tri.any() else self.quads.ravel()
        size = np.array(self.patch_size)
        start = len(self.neighbour) + np.concatenate([[0], np.cumsum(size)[:-1]])
        shift = np.zeros((6, 3))
        shift[0, 0] = self.xs[-1] - self.xs[0]
        shift[1, 0] = -shift[0, 0]
        return iso.Mesh(self.points, ptr, pts, self.owner, self.neighbour, self.n_cells, start, size,
                        np.array(self.side_kinds), np.array([1, 0, -1, -1, -1, -1]), shift, np.zeros(6))


def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


class Held:
    """What depends on a mesh alone: its host arrays on the device, and the framework's handle."""

    def __init__(self, case):
        d = _device()
        g = self.grid = Grid(case)
        self.vol = torch.tensor(g.vol, device=d)
        self.owner = torch.tensor(g.owner.astype(np.int64), device=d)
        self.neighbour = torch.tensor(g.neighbour.astype(np.int64), device=d)
        self.quads = torch.tensor(g.quads.astype(np.int64), device=d)
        self.points = torch.tensor(g.points, device=d)
        size = g.patch_size
        n0 = len(g.neighbour)
        self.partner = self.owner[n0 + size[0]:n0 + size[0] + size[1]]  # the cells across the xmin faces
        self.n_flux = n0 + size[0]  # the faces that carry a flux come first: interior, then xmin
        self._mesh = None

    @property
    def mesh(self):
        if self._mesh is None:
            self._mesh = self.grid.create()
        return self._mesh


_held: OrderedDict = OrderedDict()


def _hold(key, make):
    """The last few meshes: a program creates its mesh once and steps it many times."""
    if key not in _held:
        _held[key] = make()
        while len(_held) > 24:
            _held.popitem(last=False)
    _held.move_to_end(key)
    return _held[key]


def _held_mesh(case):
    return _hold((case["mesh"], case["nx"], case["ny"], case["nz"]), lambda: Held(case))


# ------------------------------------------------------------------------------------------ fields
class Flow:
    """A column, waves and vortices drawn from the seed; psi is the vertical vector potential."""

    def __init__(self, case, rng):
        xs, ys, _ = _nodes(case)
        self.slab = case["mesh"] == "slab"
        L = float(xs[-1])
        most = max(2, min(8, case["nx"] // 8))
        self.kx = 2.0 * np.pi / L * int(rng.integers(max(1, most // 2), most + 1))
        self.ky = np.pi * int(rng.integers(1, max(2, min(6, case["ny"] // 8)) + 1))
        self.kz = 0.0 if self.slab else 2.0 * np.pi * float(rng.uniform(0.5, 2.0))
        self.amp, self.u0 = float(rng.uniform(0.6, 1.2)), float(rng.uniform(0.3, 0.6))
        self.phase = rng.uniform(0.0, 2.0 * np.pi, 6)
        self.waves = [(2.0 * np.pi / L * int(rng.integers(1, 5)), np.pi * int(rng.integers(0, 4)), float(rng.uniform(0.008, 0.025)))
                      for _ in range(2)]
        self.level = float(rng.uniform(0.44, 0.52))
        self.column = (float(rng.uniform(0.12, 0.2)) * L, self.level + float(rng.uniform(0.08, 0.15)))
        self.om = float(rng.uniform(2.0, 6.0))

    def psi(self, x, y, z, t=0.0):
        return self.u0 * y + self.amp / self.kx * torch.sin(self.kx * x + self.phase[0] - self.om * t) * torch.sin(self.ky * y) * torch.cos(self.kz * z + self.phase[1])

    def velocity(self, x, y, z, t=0.0):
        a, cz = self.kx * x + self.phase[0] - self.om * t, torch.cos(self.kz * z + self.phase[1])
        return (self.u0 + self.amp * self.ky / self.kx * torch.sin(a) * torch.cos(self.ky * y) * cz,
                -self.amp * torch.cos(a) * torch.sin(self.ky * y) * cz)

    def surface(self, x, y):
        s = self.level + 0.0 * x
        for n, (kx, ky, amp) in enumerate(self.waves):
            s = s + amp * torch.cos(kx * x + self.phase[2 + n]) * (1.0 if self.slab else torch.cos(ky * y + self.phase[4 + n]))
        if self.slab:
            return s
        # a collapsing column: a wavy top beside a front that falls steeply
        top = self.column[1] + 0.02 * x + 0.01 * torch.cos(5.0 * x + 3.0 * y + self.phase[1])
        front = self.column[0] + 0.05 * torch.cos(4.0 * y + self.phase[2])
        return torch.maximum(s, top - 4.0 * torch.clamp(x - front, min=0.0))


def _below(flow, x, y, lo, hi):
    """The share of [lo, hi] under the surface, averaged over the sample points (last axis)."""
    return ((flow.surface(x, y) - lo) / (hi - lo)).clamp(0.0, 1.0).mean(-1)


def _alpha(case, h, flow):
    g, d = h.grid, _device()
    T = lambda v: torch.tensor(v, device=d)
    lo = h.points[T(g.corner[:, 0])]
    ext = h.points[T(g.corner[:, 7])] - lo
    gauss = T(0.5 + 0.5 * np.array([-math.sqrt(0.6), 0.0, math.sqrt(0.6)]))
    w = T(np.array([5.0, 8.0, 5.0]) / 18.0)
    if case["mesh"] == "slab":
        x = lo[:, :1] + ext[:, :1] * gauss
        return (((flow.surface(x, None) - lo[:, 1:2]) / ext[:, 1:2]).clamp(0.0, 1.0) * w).sum(1)
    if case["mesh"] in ("box", "merged"):
        # a cell's share under the surface, taken as a plane through it: fronts steeper than a cell stay smooth
        mid, x, y = lo + 0.5 * ext, ext[:, 0] * 0.5, ext[:, 1] * 0.5
        at = lambda dx, dy: flow.surface(mid[:, 0] + dx, mid[:, 1] + dy)
        rise = (at(x, 0.0) - at(-x, 0.0)).abs() + (at(0.0, y) - at(0.0, -y)).abs()
        frac = (0.5 + (at(0.0, 0.0) - mid[:, 2]) / (ext[:, 2] + rise)).clamp(0.0, 1.0)
        if case["mesh"] == "box":
            return frac
        v = ext[:, 0] * ext[:, 1] * ext[:, 2]
        out = T(np.bincount(g.cell, (frac * v).cpu().numpy(), minlength=g.n_cells))
        return (out / h.vol).clamp(0.0, 1.0)
    r = np.random.default_rng(7)  # the same sample points in every cell
    u = r.random((64, 3))
    if case["mesh"] == "prisms":
        u[:, :2] = np.sort(u[:, :2], 1)
        pts = [u[:, [1, 0]], u[:, [0, 1]]]  # below and above the diagonal
        out = []
        for q in pts:
            x = lo[:, :1] + ext[:, :1] * T(q[:, 0])
            y = lo[:, 1:2] + ext[:, 1:2] * T(q[:, 1])
            out.append(_below(flow, x, y, lo[:, 2:], lo[:, 2:] + ext[:, 2:]))
        return torch.stack(out, 1).reshape(-1)
    u = np.sort(u, 1)[:, ::-1]
    out = []
    for a, b in ((1, 2), (2, 1), (1, 4), (4, 1), (2, 4), (4, 2)):
        axes = [int(math.log2(v)) for v in (a, b, 7 - a - b)]
        q = np.empty_like(u)
        q[:, axes[0]], q[:, axes[1]], q[:, axes[2]] = u[:, 0], u[:, 1], u[:, 2]
        x, y, z = (lo[:, m:m + 1] + ext[:, m:m + 1] * T(np.ascontiguousarray(q[:, m])) for m in range(3))
        soft = 0.1 * ext[:, 2:]
        out.append(((flow.surface(x, y) - z) / soft + 0.5).clamp(0.0, 1.0).mean(-1))
    return torch.stack(out, 1).reshape(-1)


def _flux(h, flow, t=0.0):
    """phi = circulation of the vector potential around each face (midpoint rule on each edge)."""
    phi = torch.zeros(h.grid.n_faces, dtype=torch.float64, device=h.points.device)
    q = h.quads[:h.n_flux]
    for a in range(4):
        p, r = h.points[q[:, a]], h.points[q[:, (a + 1) % 4]]
        m = 0.5 * (p + r)
        phi[:h.n_flux] += flow.psi(m[:, 0], m[:, 1], m[:, 2], t) * (r[:, 2] - p[:, 2])
    return phi


def _centres(case, h):
    g = h.grid
    c = h.points[torch.tensor(g.corner, device=h.points.device)].mean(1)
    if case["mesh"] == "merged":
        c = c.cpu().numpy()
        n = np.bincount(g.cell)
        return torch.tensor(np.stack([np.bincount(g.cell, c[:, m]) / n for m in range(3)], 1), device=h.points.device)
    return c.repeat_interleave(g.members, 0)


def _velocity(c, flow, t=0.0):
    u, v = flow.velocity(c[:, 0], c[:, 1], c[:, 2], t)
    return torch.cat([u, v, torch.zeros_like(u)])


def _time_step(h, phi, courant=0.5):
    f = phi[:h.n_flux].abs()
    s = torch.zeros_like(h.vol).index_add_(0, h.owner[:h.n_flux], f)
    s.index_add_(0, torch.cat([h.neighbour, h.partner]), f)
    return float("%.10g" % float(courant / (0.5 * s / h.vol).max()))  # the sums' last bits depend on their order


def _inputs(case, seed):
    """Everything a pass reads, from the seed alone."""
    rng = np.random.default_rng([int(seed), 20])
    h = _held_mesh(case)
    flow = Flow(case, rng)
    c = _centres(case, h)
    s = {"held": h, "flow": flow, "alpha": _alpha(case, h, flow), "phi": _flux(h, flow), "U": _velocity(c, flow)}
    s["dt"] = _time_step(h, s["phi"])
    if case["op"] == "outer":
        s["phi1"], s["U1"] = _flux(h, flow, s["dt"]), _velocity(c, flow, s["dt"])
    elif case["op"] == "coupled":
        rho = torch.where(s["alpha"] > 0.5, RHO_HEAVY, RHO_LIGHT)
        noise = torch.tensor(rng.standard_normal(h.grid.n_cells), device=c.device)
        s["p_d"] = 1.0e5 + GRAVITY * (flow.level * rho + 0.02 * RHO_HEAVY * noise)
        s["target"] = ((flow.level - c[:, 2]) / (c[:, 2].max() - c[:, 2].min()) * h.grid.shape[0] + 0.5).clamp(0.0, 1.0)
    elif case["op"] == "gradient":
        times = [(n + 0.5) * s["dt"] for n in range(case["steps"])]
        s["phis"] = torch.stack([_flux(h, flow, t) for t in times])
        s["Us"] = torch.stack([_velocity(c, flow, t) for t in times])
        s["target"] = (s["alpha"] + 0.05 * torch.tensor(rng.standard_normal(h.grid.n_cells), device=c.device)).clamp(0.0, 1.0)
    elif case["op"] == "adjoint":
        s["seed_bar"] = torch.tensor(rng.standard_normal(h.grid.n_cells), device=c.device)
    return s


ZONES = [((0.3, 0.0, 0.0), (-1.0, 0.0, 0.0), 0.3), ((1.7, 0.0, 0.0), (1.0, 0.0, 0.0), 0.3)]


def prepare(case, seed):
    if case["op"] == "ensemble":
        return _prepare_ensemble(case, seed)
    s = _inputs(case, seed)
    h, op = s.pop("held"), case["op"]
    mesh = h.mesh
    s["op"], s["mesh"], s["steps"] = op, mesh, case.get("steps", 1)
    s["plan"] = iso.Plan(mesh, iso.default_options(us_mode=1) if op == "outer" else None)
    s["out"] = torch.empty_like(s["alpha"])
    if op == "coupled":
        s["plan"].set_relaxation(ZONES)
        s["faces"] = {k: torch.empty_like(s["phi"]) for k in iso.Plan.GFM_KEYS}
    elif op == "adjoint":
        n, f = mesh.n_cells, mesh.n_faces
        new = lambda m, t=torch.float64: torch.empty(m, dtype=t, device=s["alpha"].device)
        s["trace"] = {"vert_alpha": new(8 * n), "kind": new(n, torch.int32), "iso": new(n), "dV": new(f), "alpha_raw": new(n)}
        s["bars"] = (new(n), new(f))
    return s


class Tanks:
    """An ensemble's meshes and the concatenated arrays its fields are evaluated on."""

    def __init__(self, case):
        self.cases = [{"mesh": "slab", "nx": nx, "ny": ny, "nz": 1} for nx, ny in _members(case)]
        self.held = [Held(c) for c in self.cases]
        self.centres = [_centres(c, h) for c, h in zip(self.cases, self.held)]
        self.meshes = [h.mesh for h in self.held]


def _prepare_ensemble(case, seed):
    tanks = _hold(("ensemble", case["members"], case["layout"]), lambda: Tanks(case))
    rng = np.random.default_rng([int(seed), 20])
    batch = iso.Batch(tanks.meshes)
    N, F, S, d = batch.n_cells, batch.n_faces, case["steps"], _device()
    s = {"op": "ensemble", "batch": batch, "steps": S, "F": F, "N": N}
    s["alpha"] = torch.empty(N, dtype=torch.float64, device=d)
    s["phi"] = torch.empty(S, F, dtype=torch.float64, device=d)
    s["U"] = torch.empty(S, 3, N, dtype=torch.float64, device=d)
    s["dt"] = []
    for m, (c, h) in enumerate(zip(tanks.cases, tanks.held)):
        flow = Flow(c, rng)
        a, b = batch.cell_off[m], batch.cell_off[m + 1]
        f0, f1 = batch.face_off[m], batch.face_off[m + 1]
        s["alpha"][a:b] = _alpha(c, h, flow)
        dt = _time_step(h, _flux(h, flow), float(rng.uniform(0.3, 0.5)))
        for n in range(S):
            s["phi"][n, f0:f1] = _flux(h, flow, (n + 0.5) * dt)
            s["U"][n, :, a:b] = _velocity(tanks.centres[m], flow, (n + 0.5) * dt).view(3, -1)
        s["dt"].append(dt)
    s["dt"] = np.array(s["dt"])
    s["out"] = torch.empty_like(s["alpha"])
    return s


# ------------------------------------------------------------------------------------------- passes
def run(s):
    op = s["op"]
    if op == "step":
        return s["plan"].step(s["alpha"], s["phi"], s["U"], s["dt"], out=s["out"])[0]
    if op == "outer":
        return s["plan"].step(s["alpha"], s["phi"], s["U"], s["dt"], out=s["out"], phi1=s["phi1"], U1=s["U1"])[0]
    if op == "coupled":
        new, st = s["plan"].step(s["alpha"], s["phi"], s["U"], s["dt"], out=s["out"], stats=True)
        s["plan"].relax_blend(new, s["target"])
        faces = s["plan"].gfm_faces(new, s["p_d"], RHO_HEAVY, RHO_LIGHT, (0.0, 0.0, -GRAVITY), out=s["faces"])
        return {"alpha": new, "n_surface": st["n_surface"], "vol_after": st["vol_after"], **faces}
    if op == "run":
        s["out"].copy_(s["alpha"])
        return s["plan"].run(s["out"], s["phi"], s["U"], s["dt"], s["steps"])
    if op == "ensemble":
        s["out"].copy_(s["alpha"])
        return s["batch"].advect(s["out"], s["phi"], s["U"], s["dt"], s["steps"], phi_stride=s["F"], U_stride=3 * s["N"])
    if op == "gradient":
        alpha, phis = s["alpha"].detach().requires_grad_(), s["phis"].detach().requires_grad_()
        out = autograd.advect(alpha, phis, s["plan"], s["Us"], s["dt"])
        misfit = 0.5 * (out - s["target"]).square().sum()
        return (out.detach(), *torch.autograd.grad(misfit, (alpha, phis)))
    new, _ = s["plan"].step(s["alpha"], s["phi"], s["U"], s["dt"], out=s["out"], trace=s["trace"])
    return (new, *s["plan"].adjoint(s["alpha"], s["phi"], s["U"], s["dt"], s["seed_bar"], trace=s["trace"],
                                    alpha_bar=s["bars"][0], phi_bar=s["bars"][1]))


def _counts(case):
    """(cells, flux faces, interface cells) of a case's mesh: the last an estimate."""
    if case["op"] == "ensemble":
        sizes = _members(case)
        n = sum(a * b for a, b in sizes)
        return n, 2 * n, sum(1.1 * a for a, _ in sizes)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n = nx * ny * nz
    if case["mesh"] == "slab":
        return n, 2 * n, 1.1 * nx
    per, faces = {"box": (1.0, 3.0), "prisms": (2.0, 2.5), "tets": (6.0, 2.0), "merged": (0.375, 7.0)}[case["mesh"]]
    return per * n, faces * per * n, 1.3 * per * nx * ny


def work(case):
    """Cells: alpha and the volume read, the new alpha written; flux faces: the flux and the pair of
    cells; interface cells: the eight neighbours around each vertex, the corners and 11 kflop."""
    n, f, s = _counts(case)
    bytes_, flops = 24.0 * n + 16.0 * f + 300.0 * s, 11e3 * s
    op = case["op"]
    if op == "outer":
        bytes_ += 8.0 * f
    elif op == "coupled":  # face data: the pair of cells read and five values written, two cell arrays
        bytes_ += 48.0 * f + 16.0 * n + 0.3 * 36.0 * n
    elif op in ("run", "ensemble"):
        bytes_, flops = bytes_ * case["steps"] + 16.0 * n, flops * case["steps"]
    elif op == "adjoint":  # the adjoint reads what the step does and writes both gradients
        bytes_, flops = 2.0 * bytes_ + 8.0 * (n + f), 4.0 * flops
    elif op == "gradient":  # the step twice (checkpoints) and its adjoint
        bytes_, flops = case["steps"] * (3.0 * bytes_ + 8.0 * (n + f)), 5.0 * flops * case["steps"]
    return {"bytes": bytes_, "flops": flops}


# ------------------------------------------------------------------------------- the method in torch
# One step on a block of rectangular hexahedra, literally: vertex values by inverse distance, the
# isovalue by bisection of the sub-volume between sorted vertex values, the isoface fanned about its
# perimeter centroid, the time integral of each face's wet fraction, the flux-form update and the
# redistribution.
_AXES = ((0, 1, 2), (1, 2, 0), (2, 0, 1))  # a face's normal axis and the two in its plane


def _vertex_alpha(g, alpha):
    """Vertex values [nz+1, ny+1, nx+1] of cell values, inverse distance weights, periodic in x."""
    d = alpha.device
    a = alpha.view(g.shape)
    half = [torch.tensor(0.5 * np.diff(v), device=d) for v in (g.zs, g.ys, g.xs)]
    w = 1.0 / torch.sqrt(half[0][:, None, None] ** 2 + half[1][None, :, None] ** 2 + half[2][None, None, :] ** 2)
    wrap = lambda v: torch.cat([v[:, :, -1:], v, v[:, :, :1]], 2)
    pad = lambda v: torch.nn.functional.pad(wrap(v), (0, 0, 1, 1, 1, 1))
    num, den = pad(w * a), pad(w)
    nz, ny, nx = g.shape
    total = lambda v: sum(v[k:k + nz + 1, j:j + ny + 1, i:i + nx + 1] for k in (0, 1) for j in (0, 1) for i in (0, 1))
    return total(num) / total(den)


def _face_segments(c, iso_v, tie):
    """c [n, 2, 2]: values at the corners (p, q) of a unit square.  Twice the wet area, and up to two
    isoface segments ((entry p, q), (exit p, q), present), each closing the wet part from exit to entry."""
    loop = [c[:, 0, 0], c[:, 1, 0], c[:, 1, 1], c[:, 0, 1]]
    at = [(0.0, 0.0), (1.0, 0.0), (1.0, 1.0), (0.0, 1.0)]
    wet = [(v >= iso_v) if tie else (v > iso_v) for v in loop]
    cut = []
    for i in range(4):
        j = (i + 1) % 4
        d = loop[j] - loop[i]
        t = torch.where(d == 0.0, torch.zeros_like(d), (iso_v - loop[i]) / torch.where(d == 0.0, torch.ones_like(d), d))
        cut.append((at[i][0] + t * (at[j][0] - at[i][0]), at[i][1] + t * (at[j][1] - at[i][1])))
    zero = torch.zeros_like(iso_v)
    area, le, segs = zero, (zero, zero), []
    exits = [wet[i] & ~wet[(i + 1) % 4] for i in range(4)]
    entries = [~wet[i] & wet[(i + 1) % 4] for i in range(4)]
    sel = lambda m, x, y: tuple(torch.where(m, u, v) for u, v in zip(x, y))
    for i in range(4):
        le = sel(exits[i], cut[i], le)
    for i in range(4):
        segs.append((cut[i], le, entries[i]))
        area = area + torch.where(entries[i], le[0] * cut[i][1] - le[1] * cut[i][0], zero)
        le = sel(exits[i], cut[i], le)
        j = (i + 1) % 4
        a = sel(wet[i], (zero + at[i][0], zero + at[i][1]), cut[i])
        b = sel(wet[j], (zero + at[j][0], zero + at[j][1]), cut[i])
        area = area + torch.where(wet[i] | wet[j], a[0] * b[1] - a[1] * b[0], zero)
    return area, segs


def _isoface(v, ext, iso_v, tie=False):
    """Wet share of the cell, and the isoface's edges as points [n, 3] in cell coordinates."""
    total, edges = torch.zeros_like(iso_v), []
    for n, p, q in _AXES:
        for r in (0, 1):
            c = v.select(1 + n, r)
            if p > q:
                c = c.transpose(1, 2)
            area, segs = _face_segments(c, iso_v, tie)
            if r:
                total = total + area
            for s0, s1, on in segs:
                a, b = torch.zeros_like(ext), torch.zeros_like(ext)
                for x, s in ((a, s0), (b, s1)):
                    x[:, n], x[:, p], x[:, q] = float(r), s[0], s[1]
                # seen from outside, the faces at the low end run the other way round
                edges.append((a, b, on) if r else (b, a, on))
    oL, o, B = torch.zeros_like(iso_v), torch.zeros_like(ext), torch.zeros_like(ext)
    for a, b, on in edges:
        l = torch.where(on, ((b - a) * ext).norm(dim=1), torch.zeros_like(iso_v))
        oL, o = oL + l, o + 0.5 * l[:, None] * (a + b)
        B = B + torch.where(on[:, None], torch.linalg.cross(a, b), torch.zeros_like(a))
    o = torch.where(oL[:, None] > 0.0, o / oL.clamp(min=1e-300)[:, None], torch.zeros_like(o))
    return (total + (o * B).sum(1)) / 6.0, o, B, edges


def _reconstruct(v, ext, target):
    """Isoface centre (cell coordinates) and unit normal [n, 3] of cells with corner values v [n, x, y, z]."""
    s = v.reshape(len(v), 8).sort(1).values
    il = torch.zeros(len(v), dtype=torch.int64, device=v.device)
    ih = il + 7
    for _ in range(3):  # the interval of sorted vertex values
        m = (il + ih) // 2
        wet = _isoface(v, ext, s.gather(1, m[:, None])[:, 0])[0] > target
        go = ih - il > 1
        il, ih = torch.where(go & wet, m, il), torch.where(go & ~wet, m, ih)
    lo, hi = s.gather(1, il[:, None])[:, 0], s.gather(1, ih[:, None])[:, 0]
    jump = _isoface(v, ext, hi, True)[0] > target  # the sub-volume jumps across the target there
    lo = torch.where(jump, hi, lo)
    for _ in range(64):
        m = 0.5 * (lo + hi)
        wet = _isoface(v, ext, m)[0] > target
        lo, hi = torch.where(wet, m, lo), torch.where(wet, hi, m)
    _, o, B, edges = _isoface(v, ext, 0.5 * (lo + hi))
    scale = torch.stack([ext[:, 1] * ext[:, 2], ext[:, 0] * ext[:, 2], ext[:, 0] * ext[:, 1]], 1)
    n = B * scale
    n = n / n.norm(dim=1, keepdim=True)
    acc, ws = torch.zeros_like(o), torch.zeros_like(target)
    for a, b, on in edges:
        w = torch.where(on, (torch.linalg.cross(a - o, b - o) * scale * n).sum(1), torch.zeros_like(ws))
        acc, ws = acc + w[:, None] * (o + a + b), ws + w
    return acc / (3.0 * ws[:, None]), n


def _swept(d, un, dt):
    """Integral over [0, dt] of the share of a rectangle with corner distances d [n, 2, 2] that the
    plane moving at un has passed."""
    ga, gb = (d[:, 1, 0] - d[:, 0, 0]).abs(), (d[:, 0, 1] - d[:, 0, 0]).abs()
    e0 = d.reshape(len(d), 4).min(1).values
    m, M = torch.minimum(ga, gb), torch.maximum(ga, gb)
    ends = [e0, e0 + m, e0 + M, e0 + m + M]
    safe = torch.where(un == 0.0, torch.ones_like(un), un)
    cuts = torch.stack([torch.zeros_like(un)] + [(e / safe).clamp(0.0, dt) for e in ends] + [torch.full_like(un, dt)], 1).sort(1).values

    def share(z):
        z = z - e0
        q = lambda t: t * t / (2.0 * m * M).clamp(min=1e-300)
        r = torch.where(z < m, q(z), torch.where(z < M, (z - 0.5 * m) / M.clamp(min=1e-300), 1.0 - q(m + M - z)))
        return torch.where(z < 0.0, torch.zeros_like(z), torch.where(z >= m + M, torch.ones_like(z), r))

    total = torch.zeros_like(un)
    for k in range(5):  # Gauss-Legendre on each quadratic piece
        a, b = cuts[:, k], cuts[:, k + 1]
        for x in (-0.5773502691896257, 0.5773502691896257):
            total = total + 0.5 * (b - a) * share(un * (0.5 * (a + b) + 0.5 * (b - a) * x))
    return torch.where(un == 0.0, dt * share(torch.zeros_like(un)), total)


def _exact_step(h, alpha, phi, U, dt, sweeps=3, tol=1e-12):
    g, nf = h.grid, h.n_flux
    nz, ny, nx = g.shape
    own, nbr, ph = h.owner[:nf], torch.cat([h.neighbour, h.partner]), phi[:nf]
    up = torch.where(ph > 0.0, own, nbr)
    dV = alpha[up] * ph * dt
    surf = torch.nonzero((alpha > 1e-8) & (alpha < 1.0 - 1e-8))[:, 0]
    va = _vertex_alpha(g, alpha)
    k, j, i = surf // (nx * ny), (surf // nx) % ny, surf % nx
    v = torch.stack([va[k + c, j + b, i + a] for a in (0, 1) for b in (0, 1) for c in (0, 1)], 1).view(-1, 2, 2, 2)
    full = v.reshape(-1, 8)
    keep = full.max(1).values - full.min(1).values > 1e-12
    surf, v, k, j, i = surf[keep], v[keep], k[keep], j[keep], i[keep]
    corner = torch.tensor(g.corner, device=alpha.device)[surf]
    ext = h.points[corner[:, 7]] - h.points[corner[:, 0]]
    x, n = _reconstruct(v, ext, alpha[surf])
    un = (U.view(3, -1)[:, surf].T * n).sum(1)
    # faces of each cell: the interior face ids by owner and direction, the xmin patch for the wrap
    c = torch.arange(nx * ny * nz, device=alpha.device)
    inner = torch.stack([c % nx < nx - 1, (c // nx) % ny < ny - 1, c // (nx * ny) < nz - 1], 1)
    face = torch.full(inner.shape, -1, device=alpha.device)
    face[inner] = torch.arange(len(h.neighbour), device=alpha.device)
    xmin = len(h.neighbour) + torch.arange(ny * nz, device=alpha.device)
    row = surf // nx
    for axis, (p, q) in enumerate(((1, 2), (0, 2), (0, 1))):
        for r in (0, 1):
            step = (1, nx, nx * ny)[axis]
            if axis == 0:
                last, first = i == nx - 1, i == 0
                f = torch.where(last, xmin[row], face[surf, 0]) if r else torch.where(first, xmin[row], face[(surf - 1).clamp(min=0), 0])
                sign = torch.where(last if r else first, -1.0 if r else 1.0, 1.0 if r else -1.0).to(alpha.dtype)
            else:
                inside = (j > 0) if axis == 1 else (k > 0)
                f = face[surf, axis] if r else torch.where(inside, face[(surf - step).clamp(min=0), axis], -1)
                sign = torch.full_like(un, 1.0 if r else -1.0)
            at = torch.nonzero((f >= 0) & (sign * ph[f.clamp(min=0)] > 0.0))[:, 0]
            hn = ext[at] * n[at]
            base = hn[:, axis] * (r - x[at, axis])
            d = torch.stack([torch.stack([base + hn[:, p] * (a - x[at, p]) + hn[:, q] * (b - x[at, q]) for b in (0, 1)], 1) for a in (0, 1)], 1)
            dV[f[at]] = ph[f[at]] * _swept(d, un[at], dt)
    new = alpha + 0.0
    apply = lambda a, f: a + (torch.zeros_like(a).index_add_(0, nbr, f).index_add_(0, own, -f)) / h.vol
    chop = lambda a: torch.where((a < 0.0) & (a >= -tol), torch.zeros_like(a), torch.where((a > 1.0) & (a <= 1.0 + tol), torch.ones_like(a), a))
    new = chop(apply(new, dV))
    side = torch.sign(ph)
    for _ in range(sweeps):
        over, under = new > 1.0 + tol, new < -tol
        out = dV * side
        cap = torch.where(over[up], ph.abs() * dt - out, torch.where(under[up], out, torch.zeros_like(out))).clamp(min=0.0)
        need = torch.where(over, (new - 1.0) * h.vol, torch.where(under, -new * h.vol, torch.zeros_like(new)))
        room = torch.zeros_like(new).index_add_(0, up, cap)
        ratio = torch.where(room > 0.0, (need / room.clamp(min=1e-300)).clamp(max=1.0), torch.zeros_like(room))
        change = cap * ratio[up] * side * torch.where(over[up], 1.0, -1.0)
        dV, new = dV + change, chop(apply(new, change))
    return new.clamp(0.0, 1.0)


def _exact_faces(s, h, alpha):
    """The ghost-fluid face data of the new volume fractions."""
    n = h.grid.n_faces
    c = _centres({"mesh": "box"}, h)
    own, nbr = h.owner[:h.n_flux], torch.cat([h.neighbour, h.partner])
    xo, xn = c[own], c[nbr].clone()
    xn[len(h.neighbour):, 0] -= float(h.grid.xs[-1] - h.grid.xs[0])
    ao, an, po, pn = alpha[own], alpha[nbr], s["p_d"][own], s["p_d"][nbr]
    cut = (ao > 0.5) != (an > 0.5)
    lam = torch.where(cut, (ao - 0.5) / torch.where(cut, ao - an, torch.ones_like(ao)), -torch.ones_like(ao))
    z = xo[:, 2] + lam * (xn[:, 2] - xo[:, 2])
    jump = torch.where(cut, -(RHO_HEAVY - RHO_LIGHT) * GRAVITY * z, torch.zeros_like(z))
    wet = ao > 0.5
    l = torch.where(wet, lam, 1.0 - lam)
    bh, bl = 1.0 / RHO_HEAVY, 1.0 / RHO_LIGHT
    bw = torch.where(cut, l * bl + (1.0 - l) * bh, torch.zeros_like(l))
    d = torch.where(cut, bw, torch.ones_like(bw))
    pw, pd = torch.where(wet, po, pn), torch.where(wet, pn, po)
    at_dry = bl / d * pd + (1.0 - bl / d) * pw - bl / d * jump  # the heavy fluid's value at the dry cell
    at_wet = bh / d * pw + (1.0 - bh / d) * pd + bh / d * jump
    full = {k: torch.zeros(n, dtype=torch.float64, device=alpha.device) for k in ("lambda", "jump", "beta_w", "ghost_own", "ghost_nbr")}
    full["lambda"] -= 1.0
    full["ghost_own"] += s["p_d"][h.owner]
    full["ghost_nbr"] += s["p_d"][h.owner]
    full["lambda"][:h.n_flux], full["jump"][:h.n_flux], full["beta_w"][:h.n_flux] = lam, jump, bw
    full["ghost_own"][:h.n_flux] = torch.where(cut, torch.where(wet, at_wet, at_dry), po)
    full["ghost_nbr"][:h.n_flux] = torch.where(cut, torch.where(wet, at_dry, at_wet), pn)
    return full


def exact(case, seed):
    """The step, the run and the coupled step on blocks of hexahedra; the interpolated velocity of an
    outer iteration, other cell types, ensembles (64 meshes) and gradients have no value here."""
    if case["op"] not in ("step", "run", "coupled") or case["mesh"] not in ("slab", "box"):
        return None
    s = _inputs(case, seed)
    h, alpha = s["held"], s["alpha"]
    n_surface = int(((alpha > 1e-8) & (alpha < 1.0 - 1e-8)).sum())
    for _ in range(case.get("steps", 1)):
        alpha = _exact_step(h, alpha, s["phi"], s["U"], s["dt"])
    if case["op"] != "coupled":
        return alpha
    vol_after = float((alpha * h.vol).sum())
    x = _centres(case, h)[:, 0]
    for origin, direction, length in ZONES:
        chi = (x - origin[0]) * direction[0] / length
        w = 1.0 - torch.expm1(chi.clamp(0.0, 1.0) ** 3.5) / (math.e - 1.0)
        alpha = torch.where((chi >= 0.0) & (chi <= 1.0), w * alpha + (1.0 - w) * s["target"], alpha)
    return {"alpha": alpha, "n_surface": n_surface, "vol_after": vol_after, **_exact_faces(s, h, alpha)}
