"""Values that are not finite beside interface cells of rectangular hexahedra: the box kernel does with them
what the general kernel does.  A cell with such a vertex value has no isoface and moves the bulk flux; a
speed that is no number sweeps the faces whole, an infinite one sweeps them whole or not at all.

The general kernel's side is the same block with its far corner moved by a unit in the last place; both
agree to 1e-13 in alpha, as on finite inputs (tests/test_gpu_box.py), and exactly in kind and in where
alpha is not finite."""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import gpu_plan, gpu_traced_step, say

pytestmark = pytest.mark.gpu

MESHES = {"box": lambda: W.violent_3d(nx=12, ny=8, nz=8, steps=1),
          "slab": lambda: W.airy_slab(32, 16, 32, 0.08, 0.5, 1, "airy_32x16")}


def _both(w, alpha, phi, U, **opts):
    """(alpha, trace) of one step by the box kernel and by the general one."""
    m, P = w.mesh, w.mesh.points.copy()
    far = P.argmax(0)[np.argmax(P.max(0))]
    axis = int(np.argmax(P[far]))
    P[far, axis] = np.nextafter(P[far, axis], 10.0)
    other = W.Mesh(P, m.face_ptr, m.face_pts, m.owner, m.neighbour, m.n_cells, m.patches, m.shape, m.xs, m.ys, m.zs)
    out = []
    for mesh in (m, other):
        gm, plan = gpu_plan(mesh, n_bound_iter=0, clip=0, **opts)
        new, _, tr = gpu_traced_step(plan, gm, alpha, phi, U, w.dt)
        out.append((new, tr, gm))
    return out


def _agree(a, b):
    assert np.array_equal(np.isnan(a), np.isnan(b))
    on = np.isfinite(a)
    assert np.array_equal(on, np.isfinite(b)) and np.array_equal(a[~on], b[~on], equal_nan=True)
    assert np.abs(a[on] - b[on]).max() <= 1e-13


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("mesh", list(MESHES))
def test_vertex_values(mesh, bad):
    w = MESHES[mesh]()
    phi, U = w.phi_U(0)
    cut = np.nonzero((w.alpha0 > 1e-8) & (w.alpha0 < 1 - 1e-8))[0]
    c = cut[len(cut) // 2]
    alpha = w.alpha0.copy()
    alpha[c] = bad
    say(f"[gpu] {mesh}: alpha of interface cell {c} is {bad}")
    (a, ta, gm), (b, tb, _) = _both(w, alpha, phi, U)
    pts = gm.cell_points()
    beside = np.array([i for i in cut if i != c and np.isin(pts[i], pts[c]).any()])
    assert len(beside) >= 2 and (ta["kind"][beside] == 2).all()
    # (an infinite value below zero on one vertex alone, in 3D the bad cell's neighbours over a corner, is a dry
    # end like any other to the general kernel's cut points: those cells are not compared)
    if mesh == "slab" or bad != -np.inf:
        assert np.array_equal(ta["kind"], tb["kind"])
        _agree(a, b)


# (interpolated velocities: an infinite one times a weight that rounds to zero in one kernel only is no
# number there and infinite in the other)
@pytest.mark.parametrize("us_mode,bad", [(0, np.nan), (0, np.inf), (0, -np.inf), (1, np.nan)])
@pytest.mark.parametrize("mesh", list(MESHES))
def test_speeds(mesh, us_mode, bad):
    w = MESHES[mesh]()
    phi, U = w.phi_U(0)
    cut = np.nonzero((w.alpha0 > 1e-8) & (w.alpha0 < 1 - 1e-8))[0]
    c = cut[len(cut) // 2]
    U = U.reshape(3, -1).copy()
    up = 2 if mesh == "box" else 1  # the vertical: across the surface
    U[:, c] = 0.0
    U[up, c] = bad
    if np.isnan(bad):
        U[:, c] = bad
    say(f"[gpu] {mesh} us_mode={us_mode}: velocity of interface cell {c} is {U[:, c]}")
    (a, ta, _), (b, tb, _) = _both(w, w.alpha0, phi, np.ascontiguousarray(U.ravel()), us_mode=us_mode)
    assert ta["kind"][c] == 1 and not np.isfinite(ta["rec"][c, 6])
    assert np.array_equal(ta["kind"], tb["kind"])
    _agree(a, b)
