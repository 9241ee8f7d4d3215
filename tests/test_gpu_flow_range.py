"""The FP32 flow against 64 bits where operands and range are the hardest: products whose operands
fill all their bits, and spline outputs that span the exponent range of FP32."""
import math

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

HID, RAW, BINS, IN = 64, 33, 16, 96
OFF = {}
_at = 0
for _name, _count in (("W1", IN * HID), ("b1", HID), ("W2", HID * HID), ("b2", HID),
                      ("W3", HID * 3 * RAW), ("b3", 3 * RAW)):
    OFF[_name] = slice(_at, _at + _count)
    _at += _count
LAYER = _at
BUMP = 10                     # the one bump of coordinate 0 with a weight: exactly 1 at its centre
CENTRE = (BUMP + 0.5) / 32.0


@pytest.fixture(scope="module")
def mc():
    import paper_2302_05730_amd as m
    return m


def _run(mc, theta, x, direction):
    import torch
    d = torch.tensor(x, dtype=torch.float64, device="cuda")
    out, lq = torch.empty_like(d), torch.empty(len(x), dtype=torch.float64, device="cuda")
    getattr(mc.Flow(theta), direction)(d, len(x), out, lq)
    torch.cuda.synchronize()
    return out.cpu().numpy(), lq.cpu().numpy()


def _log_density(raw, x):
    """log of the spline density of raw (33 values, 64 bits) at x."""
    W = np.exp(raw[:BINS] - raw[:BINS].max())
    W /= W.sum()
    E = np.exp(raw[BINS:] - raw[BINS:].max())
    Z = (0.5 * (E[1:] + E[:-1]) * W).sum()
    X = np.concatenate([[0.0], np.cumsum(W)])
    k = min(int(np.searchsorted(X[1:], x, side="right")), BINS - 1)
    a = (x - X[k]) / W[k]
    return math.log((E[k] + a * (E[k + 1] - E[k])) / Z)


def _operands(kind, rng):
    """64 FP32 values in [1, 1 + 2^-7).  "split": the second of their three BF16 parts, in [2^-9, 2^-8),
    has all its bits and the third is near -2^-17, the most there is."""
    if kind == "random":
        return (1.0 + rng.random(HID) * 2.0**-7).astype(np.float32)
    mid = (128 + rng.integers(0, 128, HID)) / 128 * 2.0**-9
    return (1.0 + mid - 2.0**-17 + rng.integers(1, 9, HID) * 2.0**-23).astype(np.float32)


@pytest.mark.parametrize("direction", ["density", "sample"])
@pytest.mark.parametrize("kind", ["split", "random"])
@pytest.mark.parametrize("seed", range(3))
def test_products_of_operands_with_all_their_bits(mc, seed, kind, direction):
    """64 products h w, each a sum by itself.  Their sum, less 64 and times 2^14, is the difference of
    two halves of the spline heights.  The parts left out of a product are at most 2 x 2^-8 x 2^-17 =
    2^-24 of it, and its one addition at full size is off by less than a unit of FP32 there, 2^-23: 3 x
    2^-24 per product.  (Leaving out hi lo, or mid mid, would be 2^-17 or 2^-16.)"""
    rng = np.random.default_rng(seed)
    h, w = _operands(kind, rng), _operands(kind, rng)
    A = 2.0**14
    total = A * (h.astype(np.float64) * w - 1.0).sum()
    theta = np.zeros(4 * LAYER)
    first = theta[:LAYER]
    first[OFF["W1"]].reshape(IN, HID)[BUMP] = h
    first[OFF["W2"]].reshape(HID, HID)[np.arange(HID), np.arange(HID)] = w
    first[OFF["b2"]] = -1.0
    W3, b3 = first[OFF["W3"]].reshape(HID, 3, RAW), first[OFF["b3"]].reshape(3, RAW)
    W3[:, :, BINS + 9:] = A
    b3[:, BINS + 9:] = np.float32(-total)
    delta = total + float(np.float32(-total))
    assert abs(delta) < 1e-2
    raw = np.zeros(RAW)
    raw[BINS + 9:] = delta
    x = np.full((67, 6), CENTRE)
    x[:, 3:] = np.linspace(0.05, 0.45, 67)[:, None]
    out, lq = _run(mc, theta, x, direction)
    at = x if direction == "density" else out
    ref = np.array([sum(_log_density(raw, p[j]) for j in (3, 4, 5)) for p in at])
    slope = 3 * 7.5 / 16  # d log q / d delta, to first order
    third = 24 * 2.0**13 * 2.0**-23  # the third product's 24 additions, its sum below 2^13
    assert np.abs(lq - ref).max() <= (HID * 3 * 2.0**-24 * A + third) * slope + 2e-5


@pytest.mark.parametrize("depth", [80.0, 87.0, 88.0, 95.0, 100.0])
def test_heights_far_below_the_highest(mc, depth):
    """Heights e^-depth of the highest, down to 26 steps of the least subnormal number 2^-149: the
    log density in their bins is finite, off by no more than a rounding of the height and one of the
    density at that step (and 1e-5 for the rest)."""
    theta = np.zeros(4 * LAYER)
    b3 = theta[:LAYER][OFF["b3"]].reshape(3, RAW)
    b3[:, BINS + 9:] = -depth
    raw = np.zeros(RAW)
    raw[BINS + 9:] = -depth
    x = np.full((65, 6), 0.3)
    x[:, 4] = np.linspace(0.64, 0.99, 65)
    _, lq = _run(mc, theta, x, "density")
    ref = np.array([sum(_log_density(raw, p[j]) for j in (3, 4, 5)) for p in x])
    assert np.isfinite(lq).all()
    assert np.abs(lq - ref).max() <= 2 * 0.5 * 2.0**-149 / math.exp(-depth) + 1e-5


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("direction", ["density", "sample"])
def test_values_outside_the_unit_cube(mc, direction, precision):
    """Coordinates beyond the cube map like its ends: to 1 from above (within sixteen roundings of the
    widths' sum), infinities like large numbers, and to 0 from below; a NaN coordinate leaves the
    other samples as they are."""
    import torch
    if direction == "density" and precision == "bf16":
        pytest.skip("the density direction is FP32")
    kw = {} if direction == "density" else {"precision": getattr(mc, f"MCUBES_{precision.upper()}")}
    rng = np.random.default_rng(5)
    theta = np.asarray(workloads.flow_random(13, out_scale=0.3), np.float32).astype(np.float64)
    flow = mc.Flow(theta)

    def run(x):
        d = torch.tensor(x, dtype=torch.float64, device="cuda")
        out, lq = torch.empty_like(d), torch.empty(len(x), dtype=torch.float64, device="cuda")
        getattr(flow, direction)(d, len(x), out, lq, **kw)
        torch.cuda.synchronize()
        return out.cpu().numpy(), lq.cpu().numpy()

    x = rng.uniform(0.0, 1.0, (130, 6))
    plain, lq_plain = run(x)
    odd = x.copy()
    odd[64:73] = np.array([1e4, 1e20, math.inf, -1e4, -1e20, -math.inf, 1.5, -0.5, math.nan])[:, None]
    out, lq = run(odd)
    rest = np.r_[0:64, 73:130]
    assert np.array_equal(out[rest], plain[rest]) and np.array_equal(lq[rest], lq_plain[rest])
    assert np.abs(out[64:67] - 1.0).max() <= 16 * 2.0**-23 and (out[67:70] == 0.0).all()
    assert np.isfinite(lq[64:70]).all()
    for group in (slice(64, 67), slice(67, 70)):
        assert (lq[group] == lq[group][0]).all() and (out[group] == out[group][0]).all()


@pytest.mark.parametrize("depth", [0.0, 60.0, 87.0, 100.0])
def test_sampling_above_the_cube_with_low_last_heights(mc, depth):
    """z beyond 1 ends at 1, however far the last bin's heights lie below the highest: the quotients in
    that bin neither overflow nor lose its end.  In the layer that maps z first (the fourth, coordinates
    0, 2 and 4); a later one meets 1 itself, whose bin may begin there."""
    theta = np.zeros(4 * LAYER)
    theta[3 * LAYER:][OFF["b3"]].reshape(3, RAW)[:, BINS + 9:] = -depth
    z = np.full((3, 6), 0.5)
    z[:, [0, 2, 4]] = np.array([2.0, 50.0, math.inf])[:, None]
    out, _ = _run(mc, theta, z, "sample")
    assert np.abs(out[:, [0, 2, 4]] - 1.0).max() <= 3 * 16 * 2.0**-23
