"""Bounding sweeps over lists of every length: short ones walked by one work-group, long ones shared by all of
a launch's, and runs that pass from one to the other.  Random fields at ten times the workloads' time step
leave thousands of cells out of bounds, sweep after sweep (asserted).

Who walks a list changes no result: the same bits as a member of an ensemble of more than 2^17 cells, whose
sweeps are launches of their own on the whole grid, and from the plan's next call on the same input.  On fields of full and empty cells, where
no interface kernel takes part, the oracle's alpha to 1e-12: sums of at most 16 terms of at most 10 (the
Courant number), rounded a few times per sweep."""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import dev, gpu_plan, say, to_dev

pytestmark = pytest.mark.gpu

MESHES = {"slab": lambda: W.airy_slab(512, 256, 64, 0.08, 0.5, 1, "airy_512x256"),
          "box": lambda: W.violent_3d(nx=48, ny=32, nz=32, steps=1),
          "large box": lambda: W.violent_3d(nx=72, ny=48, nz=48, steps=1),
          "tets": lambda: W.poly_violent("tet", nx=16, ny=12, nz=12, steps=1),
          "merged": lambda: W.poly_violent("merged", nx=32, ny=32, nz=32, steps=1)}


def _field(w):
    return np.random.default_rng(7).uniform(0.0, 1.0, w.mesh.n_cells)


def _step(plan, w, a, mult, avg=False):
    phi, U = w.phi_U(0)
    extra = dict(phi1=to_dev(0.9 * phi), U1=to_dev(0.9 * U)) if avg else {}
    out, st = plan.step(to_dev(a), to_dev(phi), to_dev(U), mult * w.dt, stats=True, **extra)
    return out.cpu().numpy(), st


def _offenders(w, a, mult, sweeps, avg=False):
    """Cells out of bounds after `sweeps` sweeps."""
    gm, plan = gpu_plan(w.mesh, n_bound_iter=sweeps, clip=0)
    x, _ = _step(plan, w, a, mult, avg)
    return int(((x > 1 + 1e-12) | (x < -1e-12)).sum())


def _grid(w, a, mult, sweeps, avg=False):
    """The same step as the first and last member of an ensemble whose sweeps run on the grid."""
    import torch
    from paper_1804_01130_amd import Batch, Mesh, default_options
    m, k = Mesh.from_arrays(w.mesh), (1 << 17) // w.mesh.n_cells + 1
    phi, U = w.phi_U(0)
    if avg:
        phi, U = 0.5 * (phi + 0.9 * phi), 0.5 * (U + 0.9 * U)
    batch = Batch([m] * k, default_options(n_bound_iter=sweeps))
    x = to_dev(batch.concat_cells([a] * k))
    batch.advect(x, torch.cat([to_dev(phi)] * k), to_dev(batch.concat_U([U] * k)), np.full(k, mult * w.dt), 1)
    x = x.cpu().numpy()
    assert np.array_equal(x[:m.n_cells], x[-m.n_cells:])
    return x[:m.n_cells]


ALONE = 512  # touched cells that one work-group walks alone


@pytest.mark.parametrize("avg", [False, True])
@pytest.mark.parametrize("mesh", list(MESHES))
def test_long_lists(oracle_lib, mesh, avg):
    w, mult = MESHES[mesh](), 10.0
    a = _field(w)
    left = [_offenders(w, a, mult, s, avg) for s in range(3)]
    say(f"[gpu] {mesh}, avg={avg}: {w.mesh.n_cells} cells, out of bounds after 0, 1, 2 sweeps {left}")
    assert min(left[:2]) > 2 * ALONE and left[2] > ALONE  # (a listed cell is touched itself)
    om = oracle_lib.OracleMesh(w.mesh)
    for n_iter in (1, 2, 3, 7):
        gm, plan = gpu_plan(w.mesh, n_bound_iter=n_iter)
        new, st = _step(plan, w, a, mult, avg)
        again, st2 = _step(plan, w, a, mult, avg)
        assert np.array_equal(new, again) and st == st2 and st["n_bound_active"] == left[0]
        assert np.array_equal(new, _grid(w, a, mult, n_iter, avg))
        calm, _ = _step(plan, w, w.alpha0, 0.2, avg)
        assert np.array_equal(calm, _grid(w, w.alpha0, 0.2, n_iter, avg))
        if not avg and mesh != "large box":
            phi, U = w.phi_U(0)
            full = np.round(a)
            new, st = _step(plan, w, full, mult)
            ref, ost = om.step(full, phi, U, mult * w.dt, oracle_lib.default_opts(n_bound_iter=n_iter))
            assert st["n_bound_active"] == ost["n_bound_active"] > ALONE and st["n_surface"] == 0
            assert np.abs(new - ref).max() <= 1e-12


def test_lists_that_become_short():
    """Long in the first sweeps, a part of a work-group in the later ones."""
    w, mult = MESHES["box"](), 6.0
    a = _field(w)
    left = [_offenders(w, a, mult, s) for s in range(4)]
    say(f"[gpu] out of bounds after 0 .. 3 sweeps {left}")
    assert left[1] > 2 * ALONE and 0 < 7 * left[3] <= ALONE
    for n_iter in (4, 5, 12):
        gm, plan = gpu_plan(w.mesh, n_bound_iter=n_iter)
        for _ in range(2):
            assert np.array_equal(_step(plan, w, a, mult)[0], _grid(w, a, mult, n_iter))


def test_graphs_from_long_lists_to_short_ones():
    """A captured run whose lists go from one length to the other, against single steps."""
    import torch
    w = MESHES["box"]()
    n = w.mesh.n_cells
    gm, plan = gpu_plan(w.mesh, n_bound_iter=4)
    phi, U = (to_dev(x) for x in w.phi_U(0))
    say(f"[gpu] runs of {n} cells")
    for a0, mult in ((_field(w), 10.0), (np.round(_field(w)), 3.0), (w.alpha0, 0.5), (_field(w), 10.0)):
        a, b = to_dev(a0), torch.empty(n, dtype=torch.float64, device=dev())
        for _ in range(6):
            plan.step(a, phi, U, mult * w.dt, out=b)
            a, b = b, a
        x = to_dev(a0)
        plan.run(x, phi, U, mult * w.dt, 6)
        torch.cuda.synchronize()
        assert torch.equal(x, a)
