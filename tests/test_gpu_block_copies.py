"""Device states copied into and out of the block pool on an MI355X: the same
bytes as through host memory for every block size and variable count, for
pointers at 16-byte and at 8-byte alignment, in a permuted block order."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2607_19277_amd import workloads as W

pytestmark = pytest.mark.gpu

L2 = lambda: W.refine_blocks(W.uniform_blocks((2, 2, 2)), [3])
CASES = {
    "one_16": lambda: W.smooth_random(W.uniform_blocks((1, 1, 1)), (1, 1, 1), 1),
    "two_level_16": lambda: W.permute(W.smooth_random(L2(), (2, 2, 2), 2)),
    "two_level_32": lambda: W.smooth_random(L2(), (2, 2, 2), 2, bn=32),
    "one_64": lambda: W.smooth_random(W.uniform_blocks((1, 1, 1)), (1, 1, 1), 1, bn=64),
    "mhd_16": lambda: W.permute(W.mhd_smooth_random(L2(), (2, 2, 2), 2)),
}


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("case", list(CASES))
def test_device_copies_equal_host_copies(case, shift):
    import torch
    from paper_2607_19277_amd import agile as A
    w = CASES[case]()

    def shifted(n):   # n doubles at 16-byte alignment, or 8 bytes past it
        t = torch.empty(n + 2, dtype=torch.float64, device="cuda")
        assert t.data_ptr() % 16 == 0
        return t[shift:shift + n]

    src = shifted(w.U.size).view(w.U.shape)
    src.copy_(torch.from_numpy(np.ascontiguousarray(w.U)))
    h, d = A.Mesh.from_workload(w), A.Mesh.from_workload(w, U=src)
    for m in (h, d):
        assert np.array_equal(m.readback(), w.U)
        assert np.array_equal(m.readback(shifted(w.U.size).view(w.U.shape)).cpu().numpy(), w.U)
    assert h.dt() == d.dt()
    if w.bn[0] == 16:
        g = h.read_ghosts()
        assert np.array_equal(d.read_ghosts(shifted(g.size).view(g.shape)).cpu().numpy(), g)
    h.close()
    d.close()
