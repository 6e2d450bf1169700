"""Replays of captured steps on an MI355X, one and several steps to a graph:
the same bits, times and last dt as eager launches, over calls of different
lengths with the program's own work and readbacks between them, and after a
regrid."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2607_19277_amd import workloads as W

pytestmark = pytest.mark.gpu

L2 = lambda: W.refine_blocks(W.uniform_blocks((2, 2, 2)), [3])
CASES = {
    "uniform": lambda: W.smooth_random(W.uniform_blocks((2, 2, 2)), (2, 2, 2), 1),
    "two_level": lambda: W.smooth_random(L2(), (2, 2, 2), 2),
    "mhd": lambda: W.mhd_smooth_random(L2(), (2, 2, 2), 2),
}


@pytest.mark.parametrize("case", list(CASES))
def test_graphs_of_several_steps_equal_eager_steps(case):
    import torch
    from paper_2607_19277_amd import agile as A
    w = CASES[case]()
    s = torch.cuda.Stream()
    g, e = A.Mesh.from_workload(w, stream=s), A.Mesh.from_workload(w)
    g.set_option(A.OPT_GRAPH, 1)
    junk = torch.zeros(1 << 16, device="cuda")

    def same(n):
        for m in (g, e):
            m.step_cfl(n)
        junk.add_(1.0)
        torch.cuda.synchronize()
        assert np.array_equal(g.readback(), e.readback())
        assert (g.last_dt(), g.time(), g.dt()) == (e.last_dt(), e.time(), e.dt())

    for n in (1, 30, 1, 8, 19, 7, 16):
        same(n)
    for m in (g, e):
        m.step(0.5 * m.dt())
    same(9)
    if case == "two_level":
        for m in (g, e):
            m.regrid(1e9, -1.0, 2)   # the same blocks again
        same(8)
        same(41)
    g.close()
    e.close()


CHAINS = {
    "one_block": lambda: W.smooth_random(W.uniform_blocks((1, 1, 1)), (1, 1, 1), 1),
    "full_wave": lambda: W.smooth_random(W.uniform_blocks((4, 4, 4)), (4, 4, 4), 1),
    "one_more": lambda: W.smooth_random(W.uniform_blocks((13, 5, 1)), (13, 5, 1), 1),
    "two_level": lambda: W.smooth_random(L2(), (2, 2, 2), 2),
    "srhd": lambda: W.srhd_smooth_random(W.uniform_blocks((2, 2, 2)), (2, 2, 2), 1),
}


@pytest.mark.parametrize("rk", [2, 3])
@pytest.mark.parametrize("case", list(CHAINS))
def test_steps_of_one_call_equal_single_steps(case, rk):
    import torch
    from paper_2607_19277_amd import agile as A
    w = CHAINS[case]()
    w.rk, w.hi = rk, tuple(float(c) for c in w.base)   # cubic cells
    a, b = A.Mesh.from_workload(w), A.Mesh.from_workload(w)
    for n in (1, 2, 5, 4):
        a.step_cfl(n)
        for _ in range(n):
            b.step_cfl(1)
        torch.cuda.synchronize()
        assert (a.last_dt(), a.time(), a.dt()) == (b.last_dt(), b.time(), b.dt())
        assert np.array_equal(a.readback(), b.readback())
        for m in (a, b):
            m.step(0.5 * m.dt())
        assert (a.last_dt(), a.time(), a.dt()) == (b.last_dt(), b.time(), b.dt())
    a.close()
    b.close()
