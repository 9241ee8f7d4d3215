"""A caller's grid 8 bytes past a 16-byte boundary: pairs of adjacent edges are then read from both kinds
of address on every axis, and the samples are those of the aligned grid."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nbins", [50, 51])
@pytest.mark.parametrize("dim", [2, 3, 5, 8, 10])
def test_grid_at_an_odd_address(dim, nbins, precision):
    import paper_2302_05730_amd as mc
    opt = mc.mcubes_default_options(nbins=nbins)
    opt.precision = getattr(mc, f"MCUBES_{precision.upper()}")
    rng = np.random.default_rng(dim)
    params = list(rng.uniform(1.0, 3.0, dim)) + list(rng.uniform(0.3, 0.7, dim))
    plan = mc.mcubes_plan_create(workloads.GAUSSIAN, params, dim, 100_000, 5, opt)
    grid = torch.linspace(0.0, 1.0, nbins + 1, dtype=torch.float64, device="cuda") ** 1.2
    grid = grid.repeat(dim)
    sums = []
    for offset in (0, 1):
        room = torch.empty(grid.numel() + 1, dtype=torch.float64, device="cuda")
        assert room.data_ptr() % 16 == 0
        at = room[offset:offset + grid.numel()]
        at.copy_(grid)
        buf = mc.Buffers(plan)
        mc.mcubes_vsample(plan, 3, at, buf.bins, buf.partials)
        torch.cuda.synchronize()
        sums.append((buf.partials.clone(), buf.bins.clone()))
    assert torch.equal(sums[0][0], sums[1][0])
    assert torch.allclose(sums[0][1], sums[1][1], rtol=1e-12, atol=0.0)
