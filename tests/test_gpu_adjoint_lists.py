"""The adjoint through bounding lists of every length and through every division of its sweeps between
launches: a mesh of up to 2^17 cells (all sweeps, forwards and back, in one launch) and one above (the first
sweep on the whole grid), lists of thousands of cells in every sweep, several calls on one workspace.

The fields hold values of 1 to 1.3 and of 0 to -0.3 at four times the workloads' time step: cells out of bounds
everywhere and in every sweep (asserted), no interface cell, and no value near a chop's threshold."""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import gpu_plan, say, to_dev

pytestmark = pytest.mark.gpu

MESHES = {"slab": lambda: W.airy_slab(256, 128, 64, 0.08, 0.5, 1, "airy_256x128"),
          "box": lambda: W.violent_3d(nx=48, ny=32, nz=32, steps=1),
          "large box": lambda: W.violent_3d(nx=72, ny=48, nz=48, steps=1),
          "merged": lambda: W.poly_violent("merged", nx=32, ny=32, nz=32, steps=1)}
MULT = 4.0


def _field(n):
    rng = np.random.default_rng(3)
    full = rng.random(n) < 0.5
    return np.where(full, 1.0 + 0.3 * rng.random(n), -0.3 * rng.random(n))


def _copies(m, k):
    """k copies of mesh m side by side as one mesh, and the faces of each copy in it."""
    ni, nf, size = m.n_internal, m.n_faces, np.diff(m.face_ptr)
    fmap = np.zeros((k, nf), dtype=np.int64)
    fmap[:, :ni] = np.arange(k)[:, None] * ni + np.arange(ni)
    patches, at = [], k * ni
    for p in m.patches:
        fmap[:, p.start:p.start + p.size] = at + np.arange(k)[:, None] * p.size + np.arange(p.size)
        patches.append(W.Patch(p.name, p.kind, at, k * p.size, p.partner, p.translation, p.alpha_in))
        at += k * p.size
    assert at == k * nf
    back = np.argsort(fmap.ravel())  # new face -> (copy, face)
    copy, face = back // nf, back % nf
    pts = np.concatenate([m.face_pts[m.face_ptr[f]:m.face_ptr[f + 1]] + i * m.n_points for i, f in zip(copy, face)])
    ptr = np.concatenate([[0], np.cumsum(size[face])]).astype(m.face_ptr.dtype)
    own = (np.asarray(m.owner)[face] + copy * m.n_cells).astype(np.int32)
    nb = (np.asarray(m.neighbour)[face[:k * ni]] + copy[:k * ni] * m.n_cells).astype(np.int32)
    mesh = W.Mesh(np.tile(m.points, (k, 1)), ptr, pts.astype(m.face_pts.dtype), own, nb, k * m.n_cells, patches)
    return mesh, fmap


def _adjoint(plan, a, phi, U, dt, bar):
    import torch
    ab, pb = plan.adjoint(to_dev(a), to_dev(phi), to_dev(U), dt, to_dev(bar))
    torch.cuda.synchronize()
    return ab.cpu().numpy(), pb.cpu().numpy()


def _offenders(w, a, phi, U, sweeps):
    gm, plan = gpu_plan(w.mesh, n_bound_iter=sweeps, clip=0)
    x, st = plan.step(to_dev(a), to_dev(phi), to_dev(U), MULT * w.dt, stats=True)
    x = x.cpu().numpy()
    assert st["n_surface"] == 0
    return int(((x > 1 + 1e-12) | (x < -1e-12)).sum())


@pytest.mark.parametrize("n_iter", [1, 2, 3, 7])
@pytest.mark.parametrize("mesh", ["slab", "box", "large box"])
def test_dot_product_against_oracle_tangent(oracle_lib, mesh, n_iter):
    """<alpha_bar, da> + <phi_bar, dphi> = <alpha_new_bar, tangent> to 1e-9 of the sum of the magnitudes, the bar
    of the other dot-product test."""
    w = MESHES[mesh]()
    n = w.mesh.n_cells
    a = _field(n)
    phi, U = w.phi_U(0)
    left = [_offenders(w, a, phi, U, s) for s in range(n_iter)]
    say(f"[gpu] adjoint, {mesh}, {n} cells, {n_iter} sweeps; out of bounds before each {left}")
    assert min(left) > 2048
    rng = np.random.default_rng(4)
    bar = rng.standard_normal(n)
    gm, plan = gpu_plan(w.mesh, n_bound_iter=n_iter)
    ga, gp = _adjoint(plan, a, phi, U, MULT * w.dt, bar)
    om = oracle_lib.OracleMesh(w.mesh)
    for _ in range(4):
        da = rng.standard_normal(n)
        dp = rng.standard_normal(w.mesh.n_faces) * np.abs(phi).max()
        _, t = om.step_tlm(a, phi, U, MULT * w.dt, da, dp, oracle_lib.default_opts(n_bound_iter=n_iter))
        lhs, rhs = ga @ da + gp @ dp, bar @ t
        assert abs(lhs - rhs) <= 1e-9 * (np.abs(ga * da).sum() + np.abs(gp * dp).sum()), (lhs, rhs)
    again = _adjoint(plan, a, phi, U, MULT * w.dt, bar)
    assert np.array_equal(ga, again[0]) and np.array_equal(gp, again[1])


@pytest.mark.parametrize("n_iter", [1, 3, 5])
@pytest.mark.parametrize("mesh", ["slab", "box", "merged"])
def test_copies_in_one_mesh(mesh, n_iter):
    """Copies of a mesh in one of more than 2^17 cells: each copy's adjoint is the mesh's own, bit for bit, from
    long lists and, in the next call, from the workload's short ones."""
    w = MESHES[mesh]()
    m, n = w.mesh, w.mesh.n_cells
    k = (1 << 17) // n + 1
    union, fmap = _copies(m, k)
    say(f"[gpu] adjoint, {mesh}: {k} copies of {n} cells, {n_iter} sweeps")
    phi, U = w.phi_U(0)
    uphi = np.zeros(k * m.n_faces)
    uphi[fmap] = phi
    uU = np.tile(U.reshape(3, 1, n), (1, k, 1)).ravel()
    bar = np.random.default_rng(4).standard_normal(n)
    _, plan = gpu_plan(m, n_bound_iter=n_iter)
    _, uplan = gpu_plan(union, n_bound_iter=n_iter)
    for a, dt in ((_field(n), MULT * w.dt), (w.alpha0, w.dt), (_field(n), MULT * w.dt)):
        ga, gp = _adjoint(plan, a, phi, U, dt, bar)
        ua, up = _adjoint(uplan, np.tile(a, k), uphi, uU, dt, np.tile(bar, k))
        assert np.abs(ga).max() > 0 and np.abs(gp).max() > 0
        assert np.array_equal(ua.reshape(k, n), np.broadcast_to(ga, (k, n)))
        assert np.array_equal(up[fmap], np.broadcast_to(gp, (k, m.n_faces)))
