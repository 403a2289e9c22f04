"""K-means on both sides of the block count and of the crowding from which points
are assigned through the grid of cells: the blocks equal those of the definition."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import preprocess as P
from test_gpu_preprocess import _lloyd_fixed_point

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("n,bc", [(3001, 1023), (3001, 1024), (5003, 1500)])
@pytest.mark.parametrize("part", [0.0, 0.25, 0.6])
def test_blocks_equal_lloyd(n, bc, d, part):
    """A part of the points in a clump of a 50th of the extent; two equal starting
    points leave a cluster empty, so that it is re-seeded.  Metric weights are powers
    of two, so the scaled coordinates are exact."""
    from paper_2410_04477_amd import api
    g = W.rng(61 + d)
    s = g.random((n, d))
    k = int(part * n)
    s[:k] = 0.4 + 0.02 * g.random((k, d))
    w = [1.0, 1.0, 4.0][:d]
    init = W.kmeans_init(n, bc, 3)
    s[init[7]] = s[init[3]]
    bperm = W.block_permutation(bc, 3)
    dev = lambda a: torch.tensor(a, device="cuda")
    for iters in (0, 1, 9):
        perm, bp, it = api.blocks(dev(s), bc, dev(init), dev(bperm), w, max_iter=iters)
        perm_r, bp_r = P.order_blocks(_lloyd_fixed_point(s, np.array(w), init, iters), bperm)
        assert it <= iters
        np.testing.assert_array_equal(bp.cpu().numpy(), bp_r)
        np.testing.assert_array_equal(perm.cpu().numpy(), perm_r)
