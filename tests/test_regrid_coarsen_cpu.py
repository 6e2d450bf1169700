"""The library's refine / coarsen decision where whole regions coarsen, so that
octets are withdrawn in chains for the 2:1 balance: equal to the oracle's on
three- and four-level meshes, with the blocks in any order."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import regrid as RG
from paper_2607_19277_amd import agile as A
from paper_2607_19277_amd import workloads as W


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("base,levels", [((2, 2, 2), 4), ((4, 2, 1), 3), ((1, 1, 1), 4), ((3, 3, 2), 3)])
def test_coarsening_of_regions_matches_the_oracle(base, levels, seed):
    rng = np.random.default_rng(40 + seed)
    blocks = W.uniform_blocks(base)
    for _ in range(levels - 1):
        blocks = np.array(RG.decide(blocks, rng.random(len(blocks)), base, levels, 0.5, -1.0)[0], dtype=np.int32)
    blocks = blocks[rng.permutation(len(blocks))]
    # an estimate that falls off from a point: everything far from it coarsens
    scale = 2.0 ** (blocks[:, 0] - 1)
    x = (blocks[:, 1:] + 0.5) / (scale[:, None] * np.array(base))
    err = np.exp(-3.0 * np.abs(x - rng.random(3)).sum(axis=1)) + 0.02 * rng.random(len(blocks))
    refine, coarsen = np.quantile(err, [0.95, 0.7 if seed % 2 else 0.98])
    ref, R, P = RG.decide(blocks, err, base, levels, refine, coarsen)
    new, st = A.regrid_decide(blocks, err, refine, coarsen, levels, base_blocks=base, max_level=levels,
                              hi=tuple(float(b) for b in base))
    assert [tuple(r) for r in new.tolist()] == ref
    assert (st["refined"], st["coarsened"]) == (len(R), len(P))
