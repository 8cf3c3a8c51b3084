"""The interface kernel of rectangular hexahedra (csrc/box.hip) against the oracle and against the general
kernel, on blocks turned and mirrored onto every axis, at sizes that leave part of a wave.

Tolerances are those of one step from identical inputs: kinds exact, vertex values to 16 units in the
last place, isoface geometry 1e-11, face volumes 1e-13 of the largest flux volume, alpha 1e-13.  Random
fields put saddles, jumps and ties in; there the isovalue may sit on either side of a jump by rounding, so
they are compared in alpha over three steps at the trajectory bar 1e-10.
"""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import gpu_plan, gpu_traced_step, gpu_trajectory, oracle_trajectory, say

pytestmark = pytest.mark.gpu

# where the block's x, y, z axes go, and their directions
TURNS = {"as built": ((0, 1, 2), (1, 1, 1)), "x to y to z": ((1, 2, 0), (1, 1, 1)), "x to -z": ((2, 1, 0), (-1, 1, 1)),
         "mirrored y": ((0, 1, 2), (1, -1, 1)), "all down": ((2, 0, 1), (-1, -1, -1))}


def _turned(w, perm, sign):
    m = w.mesh
    R = np.zeros((3, 3))
    for i in range(3):
        R[perm[i], i] = sign[i]
    pts = m.face_pts.reshape(-1, 4)
    if np.linalg.det(R) < 0:  # a mirror turns every face around
        pts = pts[:, ::-1]
    patches = [W.Patch(p.name, p.kind, p.start, p.size, p.partner, tuple(R @ np.array(p.translation)), p.alpha_in)
               for p in m.patches]
    mesh = W.Mesh(np.ascontiguousarray(m.points @ R.T), m.face_ptr, np.ascontiguousarray(pts.ravel()), m.owner, m.neighbour,
                  m.n_cells, patches, m.shape, m.xs, m.ys, m.zs)
    phi, U = w.phi_U(0)
    U = np.ascontiguousarray((R @ U.reshape(3, -1)).ravel())
    return W.Workload(w.name, mesh, w.alpha0, w.dt, w.n_steps, lambda n: (phi, U), steady=True)


def _one_step(O, w, us_mode=0):
    gm, plan = gpu_plan(w.mesh, us_mode=us_mode)
    phi, U = w.phi_U(0)
    new, st, g = gpu_traced_step(plan, gm, w.alpha0, phi, U, w.dt)
    om = O.OracleMesh(w.mesh)
    ref, ost, o = om.step(w.alpha0, phi, U, w.dt, O.default_opts(us_mode=us_mode), trace=True)
    return (new, st, g, gm), (ref, ost, o, om), phi, U


@pytest.mark.parametrize("us_mode", [0, 1])
@pytest.mark.parametrize("turn", list(TURNS))
@pytest.mark.parametrize("size", [(12, 8, 8), (17, 5, 6), (3, 9, 4)])
def test_turned_blocks(oracle_lib, size, turn, us_mode):
    w = _turned(W.violent_3d(nx=size[0], ny=size[1], nz=size[2], steps=3), *TURNS[turn])
    say(f"[gpu] box kernel: {size} {turn} us_mode={us_mode}")
    (new, st, g, gm), (ref, ost, o, om), phi, U = _one_step(oracle_lib, w, us_mode)
    _, V = om.geometry()
    rec = np.nonzero(o["kind"] == 1)[0]
    assert len(rec) > 0 and np.array_equal(g["kind"], o["kind"]) and st["n_surface"] == ost["n_surface"]
    surf = np.nonzero(o["kind"] > 0)[0]
    assert np.abs(g["vert_alpha"][surf] - o["a_pts"][gm.cell_points()[surf]]).max() <= 16 * np.finfo(float).eps
    h = np.cbrt(V[rec]).max()
    assert np.abs(g["rec"][rec, :3] - o["rec"][rec, :3]).max() <= 1e-11 * h
    assert np.abs(g["rec"][rec, 3:6] - o["rec"][rec, 3:6]).max() <= 1e-11
    assert np.abs(g["rec"][rec, 6] - o["rec"][rec, 6]).max() <= 1e-11 * max(1.0, np.abs(U).max())
    on = ~np.isnan(g["dV"])
    assert np.abs(g["dV"][on] - o["dV"][on]).max() <= 1e-13 * np.abs(phi).max() * w.dt
    assert np.abs(new - ref).max() <= 1e-13


@pytest.mark.parametrize("turn", ["x to y to z", "all down"])
@pytest.mark.parametrize("size", [(7, 5, 4), (33, 2, 2)])
def test_random_fields(oracle_lib, size, turn):
    """Every cell an interface cell with any wet pattern (saddles and jumps among them); 140 and 132
    cells, four waves of 32 and a part of one."""
    w = _turned(W.violent_3d(nx=size[0], ny=size[1], nz=size[2], steps=3), *TURNS[turn])
    w.alpha0 = np.random.default_rng(5).uniform(0.02, 0.98, w.mesh.n_cells)
    gm, plan = gpu_plan(w.mesh)
    got = gpu_trajectory(plan, w, 3)
    ref = oracle_trajectory(oracle_lib.OracleMesh(w.mesh), w, 3)
    say(f"[gpu] box kernel, random field {size} {turn}: max |gpu - oracle| = {np.abs(got - ref).max():.3e}")
    assert np.abs(got - ref).max() <= 1e-10


@pytest.mark.parametrize("case", ["box", "slab", "slab thin in x"])
def test_against_the_general_kernel(case):
    """The same block with one corner point moved by a unit in the last place is no longer made of
    rectangular hexahedra and takes the general kernel: the same step to 1e-13."""
    if case == "box":
        w = W.violent_3d(nx=20, ny=9, nz=10, steps=3)
    else:
        w = W.airy_slab(32, 16, 32, 0.08, 0.5, 3, "slab")
        if case != "slab":
            phi, U = w.phi_U(0)
            w = _turned(W.Workload(w.name, w.mesh, w.alpha0, w.dt, 3, lambda n: (phi, U), steady=True), (1, 2, 0), (1, 1, 1))
    phi, U = w.phi_U(0)
    gm, plan = gpu_plan(w.mesh)
    a, st, tr = gpu_traced_step(plan, gm, w.alpha0, phi, U, w.dt)
    P = w.mesh.points.copy()
    far = P.argmax(0)[np.argmax(P.max(0))]
    axis = int(np.argmax(P[far]))
    P[far, axis] = np.nextafter(P[far, axis], 10.0)
    m = w.mesh
    other = W.Mesh(P, m.face_ptr, m.face_pts, m.owner, m.neighbour, m.n_cells, m.patches, m.shape, m.xs, m.ys, m.zs)
    gm2, plan2 = gpu_plan(other)
    b, st2, tr2 = gpu_traced_step(plan2, gm2, w.alpha0, phi, U, w.dt)
    say(f"[gpu] box against general kernel, {case}: max |difference| = {np.abs(a - b).max():.3e}, "
        f"rounds {st['max_root_iter']} and {st2['max_root_iter']}")
    assert np.array_equal(tr["kind"], tr2["kind"]) and st["n_surface"] == st2["n_surface"]
    assert not np.array_equal(tr["rec"], tr2["rec"], equal_nan=True)  # (two kernels, two roundings)
    assert np.abs(a - b).max() <= 1e-13
