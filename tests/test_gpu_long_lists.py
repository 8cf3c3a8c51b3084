"""Fields out of bounds in half of all cells, sweep after sweep: what the bounding costs then, and what several
plans do that share such lists between work-groups at the same time.

The times are held against a step of the same mesh as an ensemble of one member, whose sweeps are launches on the
whole grid, best of five each.  Bounds of 3 for the step and 12 for the adjoint (a traced step, sweeps forwards and
back): a work-group that walks such lists alone takes some 10 and 50 times the ensemble's step, sharing them
some 1.1 and 3 times."""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import gpu_plan, say, to_dev

pytestmark = pytest.mark.gpu


def _field(n):
    rng = np.random.default_rng(3)
    full = rng.random(n) < 0.5
    return np.where(full, 1.0 + 0.3 * rng.random(n), -0.3 * rng.random(n))


def _best(go):
    import torch
    go()
    times = []
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record()
        for _ in range(4):
            go()
        e1.record()
        torch.cuda.synchronize()
        times.append(e0.elapsed_time(e1) / 4)
    return min(times)


def test_cost_of_long_lists():
    import torch
    from paper_1804_01130_amd import Batch, Mesh, default_options
    w = W.violent_3d(nx=128, ny=64, nz=64, steps=1)
    n = w.mesh.n_cells
    a0, (phi, U) = _field(n), w.phi_U(0)
    a, dphi, dU = to_dev(a0), to_dev(phi), to_dev(U)
    _, plan = gpu_plan(w.mesh)
    out = torch.empty_like(a)
    plan.step(a, dphi, dU, w.dt, out=out)
    batch = Batch([Mesh.from_arrays(w.mesh)], default_options())
    x, bU = to_dev(a0), to_dev(batch.concat_U([U]))

    def member():
        x.copy_(a)
        batch.advect(x, dphi, bU, np.full(1, w.dt), 1)

    member()
    assert torch.equal(out, x)
    bar = to_dev(np.random.default_rng(4).standard_normal(n))
    grid = _best(member)
    step = _best(lambda: plan.step(a, dphi, dU, w.dt, out=out))
    adjoint = _best(lambda: plan.adjoint(a, dphi, dU, w.dt, bar))
    say(f"[gpu] {n} cells, half of them out of bounds: ensemble {grid * 1e3:.0f} us, step {step * 1e3:.0f}, "
        f"adjoint {adjoint * 1e3:.0f}")
    assert step < 3.0 * grid and adjoint < 12.0 * grid


def test_plans_on_several_streams():
    """Steps and adjoints of four plans at once, each on a stream of its own, against the same one by one."""
    import torch
    w = W.violent_3d(nx=64, ny=32, nz=32, steps=1)
    n = w.mesh.n_cells
    phi, U = w.phi_U(0)
    dphi, dU, bar = to_dev(phi), to_dev(U), to_dev(np.random.default_rng(4).standard_normal(n))
    fields = [to_dev(np.roll(_field(n), 97 * i)) for i in range(4)]
    plans = [gpu_plan(w.mesh, n_bound_iter=5) for _ in range(4)]
    go = lambda p, a: (p.step(a, dphi, dU, 4.0 * w.dt)[0], *p.adjoint(a, dphi, dU, 4.0 * w.dt, bar))
    ref = [go(plans[0][1], a) for a in fields]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    say(f"[gpu] four streams, {n} cells")
    for _ in range(10):
        got = []
        for (gm, p), a, s in zip(plans, fields, streams):
            with torch.cuda.stream(s):
                got.append(go(p, a))
        torch.cuda.synchronize()
        for r, g in zip(ref, got):
            assert all(torch.equal(x, y) for x, y in zip(r, g))
