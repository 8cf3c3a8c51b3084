"""The update kernel where its straight-line path mends exceptions: values that are not finite next to faces
without a flux, and work-groups larger than the many-sided cells' kernel takes.

A face without a flux moves exactly nothing, whatever lies on either side of it, so those comparisons are
exact; launch shapes give the same bits.
"""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import dev, gpu_plan, gpu_trajectory, say, to_dev

pytestmark = pytest.mark.gpu

MESHES = {"hex": lambda: W.violent_3d(nx=12, ny=8, nz=8, steps=2), "slab": lambda: W.airy_slab(40, 9, 20, 0.07, 0.5, 2, "airy_40x9"),
          "tet": lambda: W.poly_violent("tet", nx=6, ny=4, nz=4, steps=2),
          "merged": lambda: W.poly_violent("merged", nx=8, ny=4, nz=4, steps=2)}


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("mesh", list(MESHES))
def test_values_not_finite_stay_behind_faces_without_flux(mesh, bad):
    w = MESHES[mesh]()
    import torch
    gm, plan = gpu_plan(w.mesh, n_bound_iter=0, clip=0)
    phi, U = w.phi_U(0)
    owner, nb = np.asarray(w.mesh.owner), np.asarray(w.mesh.neighbour)
    n = w.mesh.n_cells
    a = (np.arange(n) % 2).astype(float)  # full and empty cells only
    c = n // 2 + 1
    phi = phi.copy()
    phi[owner == c] = 0.0
    phi[:len(nb)][nb == c] = 0.0
    for q in w.mesh.patches:  # both halves of a cyclic face carry its flux
        if q.partner >= 0:
            p = w.mesh.patches[q.partner]
            far = owner[p.start:p.start + p.size] == c
            phi[q.start:q.start + q.size][far] = 0.0
    say(f"[gpu] {mesh}: alpha of cell {c} is {bad}")
    dV = torch.zeros((gm.n_faces,), device=dev(), dtype=torch.float64)  # (empty patches' faces are not written)

    def step():
        out = plan.step(to_dev(a), to_dev(phi), to_dev(U), w.dt, trace={"dV": dV})
        return (out[0] if isinstance(out, tuple) else out).cpu().numpy()

    ref = step()
    a[c] = bad
    new = step()
    others = np.arange(n) != c
    assert np.array_equal(new[others], ref[others]) and (np.isnan(new[c]) if np.isnan(bad) else new[c] == bad)
    assert not dV.cpu().numpy()[phi == 0.0].any()


@pytest.mark.parametrize("block_cells", [64, 100, 300, 1024])
def test_block_sizes_of_many_sided_cells(block_cells):
    w = W.poly_violent("merged", nx=16, ny=8, nz=8, steps=3)
    gm, plan = gpu_plan(w.mesh)
    ref = gpu_trajectory(plan, w, 3)
    gm, plan = gpu_plan(w.mesh, block_cells=block_cells)
    assert np.array_equal(gpu_trajectory(plan, w, 3), ref)
