"""Ensembles of rectangular hexahedra beside other cells without general polyhedra: two interface kernels side
by side, each taking its own cells.  The same bits as each member alone, on every replay of the captured steps
with other work in between, and launched step by step."""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import say
from tests.test_gpu_batch import STEPS, _build, _run

pytestmark = pytest.mark.gpu

SETS = {"tets": lambda: [W.poly_violent("tet", nx=8, ny=4, nz=4, steps=STEPS), W.airy_slab(64, 32, 32, 0.05, 0.35, STEPS, "m1"),
                         W.violent_3d(nx=16, ny=8, nz=8, steps=STEPS)],
        "bent": lambda: [W.airy_slab(96, 48, 24, 0.07, 0.45, STEPS, "m0"), W.perturbed_box(nx=10, ny=6, nz=6, steps=STEPS)]}


@pytest.mark.parametrize("us_mode", [0, 1])
@pytest.mark.parametrize("kind", list(SETS))
def test_members_alone(kind, us_mode):
    import torch
    E = _build(SETS[kind](), us_mode=us_mode)
    ref = np.concatenate(E["alone"])
    say(f"[gpu] {kind}, us_mode={us_mode}: {E['batch'].n_cells} cells")
    for k in range(4):
        assert np.array_equal(_run(E).cpu().numpy(), ref), k
        (torch.rand(1 << 20, device="cuda:0", dtype=torch.float64) ** 2).sum().item()


def test_step_by_step():
    """260 steps, beyond the captured length, against two captured runs of 130."""
    import torch
    E = _build(SETS["tets"]())
    phi, U, dts = E["phi"][0].contiguous(), E["U"][0].contiguous(), 0.05 * E["dts"]
    a, b = E["alpha0"].clone(), E["alpha0"].clone()
    say("[gpu] 260 steps")
    E["batch"].advect(a, phi, U, dts, 260)
    for _ in range(2):
        E["batch"].advect(b, phi, U, dts, 130)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.isfinite(a).all()
