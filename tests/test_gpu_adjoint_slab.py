"""The adjoint on slabs one layer thick, whose vertex values tie in pairs up to their last bits: gradients of
evolved states at the components around the surface, against the oracle's at the bar of the one-step adjoint
tests, 1e-9 of the gradient's largest entry."""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import gpu_plan, say
from tests.test_gpu_adjoint import _adjoint, _state_after

pytestmark = pytest.mark.gpu

SLABS = {"airy": lambda: W.airy_slab(64, 32, 32, 0.08, 0.5, 8, "airy_64x32"),
         "cosine": lambda: W.cosine_uniform(nx=64, ny=32, steps=8, co=0.5)}


@pytest.mark.parametrize("step", [0, 1, 3, 6])
@pytest.mark.parametrize("slab", list(SLABS))
def test_evolved_states(oracle_lib, slab, step):
    w = SLABS[slab]()
    a = _state_after(oracle_lib, w, step)
    phi, U = w.phi_U(step)
    rng = np.random.default_rng(step)
    bar = rng.standard_normal(w.mesh.n_cells)
    gm, plan = gpu_plan(w.mesh)
    ga, gp = _adjoint(plan, w, a, phi, U, bar)
    cut = np.nonzero((a > 1e-8) & (a < 1 - 1e-8))[0]
    cells = rng.choice(cut, min(len(cut), 150), replace=False)
    near = np.nonzero(np.isin(w.mesh.owner, cut))[0]
    faces = rng.choice(near, min(len(near), 150), replace=False)
    say(f"[gpu] {slab} slab after {step} steps: {len(cut)} interface cells")
    assert len(cut) > 50
    oa, op = oracle_lib.OracleMesh(w.mesh).gradient(a, phi, U, w.dt, bar, cells=cells, faces=faces)
    assert np.abs(ga[cells] - oa).max() <= 1e-9 * np.abs(ga).max()
    assert np.abs(gp[faces] - op).max() <= 1e-9 * np.abs(gp).max()
