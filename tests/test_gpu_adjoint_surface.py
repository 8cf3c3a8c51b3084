"""The reverse pass through the isoface (k_adj_surface) on random fields: every cell an interface cell, with
saddle faces (two isoface edges), three wet vertices, planar and bent faces, triangles among them; against
the oracle's gradient at the bar of the one-step adjoint tests, 1e-9 of the gradient's largest entry.

No slab is among them: the vertices of a cell one layer thick are equal in pairs, up to the last bits, and
where the isovalue sits at a jump of such a pair those bits decide which side the gradient is taken on."""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import gpu_plan, say
from tests.test_gpu_adjoint import _adjoint

pytestmark = pytest.mark.gpu

MESHES = {"graded box": lambda: W.violent_3d(nx=7, ny=5, nz=4, steps=1),
          "bent box": lambda: W.perturbed_box(nx=5, ny=4, nz=5, steps=1),
          "tets": lambda: W.poly_violent("tet", nx=3, ny=2, nz=3, steps=1),
          "bent prisms": lambda: W.poly_violent("prism", nx=4, ny=3, nz=2, steps=1, perturb=0.15)}


@pytest.mark.parametrize("seed", [1, 2])
@pytest.mark.parametrize("mesh", list(MESHES))
def test_random_fields(oracle_lib, mesh, seed):
    w = MESHES[mesh]()
    rng = np.random.default_rng(seed)
    a = rng.uniform(0.05, 0.95, w.mesh.n_cells)
    abar_new = rng.standard_normal(w.mesh.n_cells)
    phi, U = w.phi_U(0)
    dt = 0.2 * w.dt
    say(f"[gpu] adjoint of a random field: {mesh}, seed {seed}, {w.mesh.n_cells} cells")
    w.dt = dt
    gm, plan = gpu_plan(w.mesh)
    ga, gp = _adjoint(plan, w, a, phi, U, abar_new)
    oa, op = oracle_lib.OracleMesh(w.mesh).gradient(a, phi, U, dt, abar_new)
    assert np.abs(ga - oa).max() <= 1e-9 * np.abs(oa).max()
    assert np.abs(gp - op).max() <= 1e-9 * np.abs(op).max()
