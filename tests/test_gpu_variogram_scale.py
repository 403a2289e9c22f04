"""Variogram bins do not depend on the unit of length: coordinates and cut-off scaled by
the same power of two fall in the same bins, down to squares near the smallest
normal numbers."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import learned as OLR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("power", [0, -440, -480, -490, -500, 400])
@pytest.mark.parametrize("shared", [False, True])
def test_bins_at_any_unit(power, shared):
    from paper_2410_04477_amd import api
    g = W.rng(21)
    k, nsets, f = 500, 3, 2.0 ** power
    locs, y = g.random((k, 2)), g.standard_normal((nsets, k))
    loc = locs * f if shared else np.broadcast_to(locs * f, (nsets, k, 2)).copy()
    dev = lambda a, dt=torch.float64: torch.tensor(a, dtype=dt, device="cuda")
    _, gam = api.variogram(dev(loc), dev(y), dev(np.zeros(nsets), torch.int32), 32, 0.5 * f, 1, shared_design=shared)
    for b in range(nsets):
        ref, _ = OLR.variogram(locs, y[b], 32)
        np.testing.assert_allclose(gam[b].cpu().numpy(), ref, rtol=1e-12, atol=0)
