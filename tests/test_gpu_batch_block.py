"""The batched form's default workgroup size: the kernels whose registers allow three waves per SIMD take
768 threads, the others 512; and the iteration it samples is the single form's."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is the one the library then uses)

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("family,dim,block", [
    (workloads.GAUSSIAN, 9, 768), (workloads.PRODUCT_PEAK, 10, 768), (workloads.DISCONTINUOUS, 10, 768),
    (workloads.DISCONTINUOUS, 8, (768, 512)), (workloads.GAUSSIAN, 8, 512), (workloads.OSCILLATORY, 2, 512)])
def test_default_block_and_its_iteration(family, dim, block, precision):
    import paper_2302_05730_amd as mc
    opt = mc.mcubes_default_options(nbins=50)
    opt.precision = getattr(mc, f"MCUBES_{precision.upper()}")
    rng = np.random.default_rng(dim)
    params = list(rng.uniform(1.0, 3.0, dim)) + list(rng.uniform(0.3, 0.7, dim))
    ncalls = [30_000, 300_001]
    batch = mc.Batch([(family, dim, n, params) for n in ncalls], 5, opt)
    if isinstance(block, tuple):  # the FP32 kernel holds fewer registers
        block = block[precision == "fp32"]
    assert {c["block_size"] for c in batch.classes()} == {block}
    grid = np.linspace(0.0, 1.0, 51) ** 1.1
    grid[-1] = 1.0
    grids = [np.tile(grid, (dim, 1)) for _ in ncalls]
    est, refined = batch.step(2, grids)
    for i, n in enumerate(ncalls):
        opt.stream_id = i
        plan = mc.mcubes_plan_create(family, params, dim, n, 5, opt)
        I, var, _, new = mc.mcubes_iterate(plan, grids[i], 2)
        assert abs(est[i][0] - I) <= 1e-12 * abs(I) and abs(est[i][1] - var) <= 1e-11 * abs(var)
        assert np.abs(refined[i] - new).max() <= 1e-12
