"""GPU kernels at the edges of their tiles and ranges, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2302_05730_amd as m
    m.lib()
    return m


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _f32(a):
    return np.asarray(a, dtype=np.float32).astype(np.float64)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257])
def test_bf16_sampling_at_bin_edges_of_the_identity_flow(mc, n):
    """z at the edges k/16 of the identity flow's sixteen equal bins and at both
    ends of (0, 1): whichever neighbouring bin takes an edge, x = z and q = 1,
    to the rounding of sixteen FP32 widths (16 x 2^-24) per mapped coordinate
    and layer, at most three layers deep."""
    import torch
    fl = mc.Flow(workloads.flow_init(5))
    edges = np.concatenate([np.arange(1, 16) / 16.0, [2.0 ** -33, 2.0 ** -24, 1.0 - 2.0 ** -24, 0.5 - 2.0 ** -25]])
    rng = np.random.default_rng(n)
    z = _f32(rng.choice(edges, (n, 6)))
    d_x = torch.empty(n * 6, dtype=torch.float64, device="cuda")
    d_lq = torch.empty(n, dtype=torch.float64, device="cuda")
    fl.sample(_dev(z), n, d_x, d_lq, precision=mc.MCUBES_BF16)
    assert np.abs(d_x.cpu().numpy().reshape(n, 6) - z).max() <= 3 * 16 * 2.0 ** -24
    assert np.abs(d_lq.cpu().numpy()).max() <= 12 * 16 * 2.0 ** -24


@pytest.mark.parametrize("n", [1, 63, 65, 300])
def test_bf16_sampling_of_a_partial_wave_matches_oracle(mc, n):
    """A steep flow at sample counts around one wave, within the bounds that any
    sample of the BF16 path has (ten times the 99% ones: 2e-3 in x, 2e-2 in log q)."""
    import torch
    theta = _f32(workloads.flow_random(11, out_scale=0.8))
    fl = mc.Flow(theta)
    z = _f32(np.random.default_rng(n).uniform(0.0, 1.0, (n, 6)))
    d_x = torch.empty(n * 6, dtype=torch.float64, device="cuda")
    d_lq = torch.empty(n, dtype=torch.float64, device="cuda")
    fl.sample(_dev(z), n, d_x, d_lq, precision=mc.MCUBES_BF16)
    ref = [oracle.flow_sample(theta, p, bf16=True) for p in z]
    assert np.abs(d_x.cpu().numpy().reshape(n, 6) - np.array([r[0] for r in ref])).max() <= 2e-3
    assert np.abs(d_lq.cpu().numpy() - np.array([r[1] for r in ref])).max() <= 2e-2
