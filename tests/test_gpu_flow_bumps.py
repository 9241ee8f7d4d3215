"""The one-blob encoding inside the BF16 gradient: with one sample the gradient of W1 is bump times
delta and that of b1 the delta, both products of BF16 values that FP32 holds exactly, so their quotient
is the bump as the kernel rounded it."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

HID, BLOBS = 64, 32


def _bf16(v):
    """v (64 bits) rounded to BF16, and how far (relative) v is from the nearest place where that turns."""
    m, e = np.frexp(v)
    scaled = m * 256.0  # in [128, 256): BF16 has 8 bits
    return np.ldexp(np.round(scaled) / 256.0, e), np.abs(scaled - np.floor(scaled) - 0.5) / scaled


def test_bumps_of_the_weight_gradient_are_rounded_from_fp32():
    """Each bump is exp(-t^2/2) to FP32 accuracy before it is rounded.  t = 32 (u - c) is exact where
    |u - c| <= u (a difference of multiples of u's unit no larger than u) and rounded once otherwise, x =
    t^2/2 is rounded once, and the exponential is good to a unit: (x + 2) 2^-24 of the bump, or (3 x + 2)
    2^-24.  Bumps within that of a rounding boundary may go either way; no other."""
    import torch

    import paper_2302_05730_amd as mc
    theta = np.asarray(workloads.flow_random(21, out_scale=0.5), np.float32).astype(np.float64)
    flow = mc.Flow(theta)
    calls = 16000
    x = np.random.default_rng(8).random((calls, 6)).astype(np.float32).astype(np.float64)
    d_x = torch.tensor(x, device="cuda")
    one = torch.ones(1, dtype=torch.float64, device="cuda")
    grad = torch.empty(mc.MCUBES_FLOW_PARAMS, dtype=torch.float64, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    bumps = torch.empty(calls, 3 * BLOBS, dtype=torch.float64, device="cuda")
    rows = 3 * BLOBS * HID
    for i in range(calls):
        flow.loss_grad(d_x[i], one, 1, grad, loss, precision=mc.MCUBES_BF16)
        delta = grad[rows:rows + HID]
        o = delta.abs().argmax()
        bumps[i] = grad[:rows].view(-1, HID)[:, o] / delta[o]
    got = bumps.cpu().numpy().reshape(calls, 3, BLOBS)
    t = (x[:, :3, None] - (np.arange(BLOBS) + 0.5) / BLOBS) * BLOBS
    half = 0.5 * t * t
    want, margin = _bf16(np.exp(-half))
    roundings = np.where(np.abs(t) <= 32.0 * x[:, :3, None], 1, 3)
    sure = (half < 20.0) & (margin > (roundings * half + 2) * 2.0**-24)
    assert sure.sum() > 0.99 * (half < 20.0).sum()
    wrong = sure & (got != want)
    assert not wrong.any(), (int(wrong.sum()), t[wrong][:5], got[wrong][:5], want[wrong][:5])
