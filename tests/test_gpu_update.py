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


@pytest.mark.parametrize("n_bound_iter", [0, 1, 2, 3, 7])
@pytest.mark.parametrize("size", [(48, 32, 32), (72, 48, 48)])
def test_sweeps_in_one_work_group_and_on_the_grid(size, n_bound_iter):
    """A mesh whose sweeps run in one work-group (49152 cells) or after the first (165888), alone and as a
    member of an ensemble, whose sweeps run on the grid: the same bits, from fields that leave cells out
    of bounds in every sweep, over more touched cells than the work-group has threads."""
    import torch
    from paper_1804_01130_amd import Batch, Mesh, Plan, default_options
    w = W.violent_3d(nx=size[0], ny=size[1], nz=size[2], steps=3)
    m = Mesh.from_arrays(w.mesh)
    opts = default_options(n_bound_iter=n_bound_iter)
    rng = np.random.default_rng(5)
    a0 = [w.alpha0, rng.uniform(0.0, 1.0, w.mesh.n_cells), np.where(rng.random(w.mesh.n_cells) < 0.02, rng.random(w.mesh.n_cells), w.alpha0)]
    phi, U = w.phi_U(0)
    say(f"[gpu] sweeps: {size} n_bound_iter={n_bound_iter}")
    plan, alone, active = Plan(m, opts), [], []
    for a in a0:
        a, b = to_dev(a), torch.empty(m.n_cells, dtype=torch.float64, device=dev())
        for _ in range(3):
            _, st = plan.step(a, to_dev(phi), to_dev(U), w.dt, out=b, stats=True)
            a, b = b, a
        active.append(st["n_bound_active"])
        alone.append(a)
    assert max(active) > 300
    batch = Batch([m] * 3, opts)
    x = to_dev(batch.concat_cells(a0))
    batch.advect(x, torch.cat([to_dev(phi)] * 3), to_dev(batch.concat_U([U] * 3)), np.full(3, w.dt), 3)
    torch.cuda.synchronize()
    assert torch.equal(x, torch.cat(alone))
