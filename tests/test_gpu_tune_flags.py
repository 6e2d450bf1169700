"""Tuning a mesh in caller-owned memory on an MI355X times single stage
launches on its state: they must not leave a mark, also where the mesh's own CFL
step would be unphysical (the program steps with a dt of its own)."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2607_19277_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("physics", ["euler", "srhd"])
def test_tuning_does_not_flag_a_mesh_whose_cfl_step_is_unphysical(physics):
    import torch
    from paper_2607_19277_amd import agile as A
    blocks = W.refine_blocks(W.uniform_blocks((2, 2, 2)), [3])
    w = (W.smooth_random if physics == "euler" else W.srhd_smooth_random)(blocks, (2, 2, 2), 2)
    dt = A.Mesh.from_workload(w).dt()
    w.cfl *= 1000.0
    need = A.plan(w.blocks, physics=w.physics, riemann=w.riemann, base_blocks=w.base, lo=w.lo, hi=w.hi,
                  max_level=w.max_level)["device_bytes"]
    pool = torch.zeros(need, dtype=torch.uint8, device="cuda")
    a, b = A.Mesh.from_workload(w, pool=pool), A.Mesh.from_workload(w)
    for _ in range(2):
        a.tune()
        assert a.dt() == b.dt()      # checks the flag
        assert np.array_equal(a.readback(), b.readback())
        for m in (a, b):
            m.step(dt)
        assert (a.time(), a.last_dt()) == (b.time(), b.last_dt())
    a.close()
    b.close()
