"""A step captured by the caller on an MI355X and replayed between the
program's own calls: ghosts, error estimate and regrid see the state after
each replay, as with eager steps."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2607_19277_amd import workloads as W

pytestmark = pytest.mark.gpu

L2 = lambda: W.refine_blocks(W.uniform_blocks((2, 2, 2)), [3])
CASES = {
    "euler": lambda: W.smooth_random(L2(), (2, 2, 2), 2),
    "srhd": lambda: W.srhd_smooth_random(L2(), (2, 2, 2), 2),
    "mhd": lambda: W.mhd_smooth_random(L2(), (2, 2, 2), 2),
}


@pytest.mark.parametrize("case", list(CASES))
def test_ghosts_follow_the_replays_of_a_captured_step(case):
    import torch
    from paper_2607_19277_amd import agile as A
    w = CASES[case]()
    s = torch.cuda.Stream()
    g, e = A.Mesh.from_workload(w, stream=s), A.Mesh.from_workload(w)
    for m in (g, e):
        m.step_cfl(1)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        g.step_cfl(1)
    junk = torch.zeros(1 << 16, device="cuda")
    for _ in range(4):
        with torch.cuda.stream(s):
            graph.replay()
        e.step_cfl(1)
        junk.add_(1.0)
        torch.cuda.synchronize()
        assert np.array_equal(g.readback(), e.readback())
        assert np.array_equal(g.read_ghosts(), e.read_ghosts())
        assert np.array_equal(g.error(), e.error())
    with torch.cuda.stream(s):
        graph.replay()
    e.step_cfl(1)
    torch.cuda.synchronize()
    for m in (g, e):
        m.regrid(-1.0, -2.0, 2)   # every block refined
    assert np.array_equal(g.readback(), e.readback())
    g.close()
    e.close()
