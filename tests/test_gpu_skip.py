"""`skip` at and beyond the iterations that are run, up to the largest int32: nothing is combined, so
the estimate is 0 with an infinite error, whatever the number of iterations."""
import math

import pytest
import torch

import paper_2302_05730_amd as mc
import workloads

pytestmark = pytest.mark.gpu

INT32_MAX = 2**31 - 1
SKIPS = [3, 4, INT32_MAX - 512, INT32_MAX - 511, INT32_MAX - 63, INT32_MAX]
PARAMS = [5.0, 7.0, 3.0, 0.4, 0.5, 0.6]


def _uncombined(r, iterations):
    assert r["estimate"] == 0.0 and r["error"] == math.inf and r["chi2_dof"] == 0.0
    assert r["dof"] == 0 and r["iterations"] == iterations and not r["converged"]


@pytest.mark.parametrize("skip", SKIPS)
def test_skip_beyond_the_iterations(skip):
    opt = mc.mcubes_default_options(nbins=50, skip=skip)
    for entry in (mc.mcubes_integrate, mc.mcubes_integrate_noalloc):
        r = entry(workloads.PRODUCT_PEAK, PARAMS, 3, 5000, 3, 0.0, 11, opt)
        _uncombined(r, 3)
    batch = mc.Batch([(workloads.PRODUCT_PEAK, 3, 5000, PARAMS)] * 2, 11, opt)
    for r in batch.integrate(3, 0.0)[1]:
        _uncombined(r, 3)


@pytest.mark.parametrize("skip", SKIPS)
def test_skip_in_the_step_calls(skip):
    plan = mc.mcubes_plan_create(workloads.PRODUCT_PEAK, PARAMS, 3, 5000, 11,
                                 mc.mcubes_default_options(nbins=50, skip=skip))
    buf = mc.Buffers(plan)
    mc.mcubes_init_grid(plan, buf.grid[0])
    for t in range(3):
        mc.mcubes_iteration(plan, t, buf.grid[t & 1], buf.grid[(t + 1) & 1], buf.bins, buf.partials,
                            buf.est, buf.state, 0.0)
    fused = buf.state.clone()
    mc.mcubes_combine(plan, 2, buf.est, buf.state, 0.0)
    torch.cuda.synchronize()
    assert torch.equal(fused[:7], buf.state[:7])
    assert fused[0] == 0.0 and fused[1] == math.inf and fused[4] == 3.0 and fused[5] == 0.0
