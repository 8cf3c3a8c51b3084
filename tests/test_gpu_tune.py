"""The autotuner leaves alone the launch shapes that no kernel of the ensemble reads."""
import numpy as np
import pytest

import wavegen as W
from tests.gpuutil import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["rectangular hexahedra", "with tetrahedra"])
def test_shapes_not_read_stay(kind):
    import torch
    from paper_1804_01130_amd import Batch, Mesh, default_options
    ws = [W.airy_slab(64, 32, 32, 0.05, 0.35, 1, "m0"), W.violent_3d(nx=16, ny=8, nz=8, steps=1)]
    if kind == "with tetrahedra":
        ws.append(W.poly_violent("tet", nx=8, ny=4, nz=4, steps=1))
    batch = Batch([Mesh.from_arrays(w.mesh) for w in ws], default_options())
    phi = torch.cat([to_dev(w.phi_U(0)[0]) for w in ws])
    U = to_dev(batch.concat_U([w.phi_U(0)[1] for w in ws]))
    a = to_dev(batch.concat_cells([w.alpha0 for w in ws]))
    dts = np.array([w.dt for w in ws])
    batch.set_config(surface_waves=4, bound_blocks=77)  # (neither is a candidate)
    for _ in range(3):
        cfg, ms = batch.tune(a, phi, U, dts, n_trial=2)
        say(f"[gpu] tuned {kind}: {cfg} {ms:.4f} ms")
        assert cfg["bound_blocks"] == 77  # below 2^17 cells one launch runs the sweeps
        assert cfg["surface_waves"] == 4 or kind == "with tetrahedra"
        assert cfg["surface_blocks"] in (0, 512, 1024, 2048, 4096) and cfg["block_cells"] in (128, 256, 512)
