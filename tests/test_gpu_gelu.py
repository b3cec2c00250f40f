"""The GELU epilogue against float64 through an encoder block.

With zero out-projection and identity-like fc weights, an encoder block's output
is x + gelu(fc1 bias) of one picked unit per channel, and x is zero: the biases
sweep the activation's range.  64 units are read out at a time; the sweeps cover
the polynomial's fitted part on both sides, zero, its neighbourhood, the tail and
values whose polynomial overflows.
"""
import math

import numpy as np
import pytest
import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models as PM
from tests.hip_harness import Runner

pytestmark = pytest.mark.gpu

D, F, T = 64, 4096, 5

# Zero, near zero, around the ends of the fitted range and of the clamp, far out
EDGES = [0.0] + [s * v for v in (1e-30, 1e-12, 1e-6, 1e-4, 1e-3, 0.01, 0.05, 0.3, 6.49, 6.5, 6.51, 7.2, 8.0, 9.5, 12.0,
                                 15.99, 16.0, 16.01, 20.0, 40.0, 300.0, 1e4, 1e6, 1e10, 1e19, 1e30, 2.9e38)
                 for s in (1.0, -1.0)]


def _picked(bias64, batch):
    """The block's outputs [batch, T, D] when channel j reads a unit of bias bias64[j]."""
    layers = PM.vit(image=8, patch=4, dim=D, heads=1, mlp=F, depth=1)[:3]
    man = PM.raw_manifest(layers, (3, 8, 8))
    raw = [np.zeros(s, np.float32) for s, _ in man]
    i1 = [s for s, _ in man].index((F, D))
    pick = np.arange(D) * (F // D) + np.arange(D) % (F // D)   # every lane position of the epilogue
    raw[i1 + 1][pick] = bias64
    raw[i1 + 2][np.arange(D), pick] = 1.0
    r = Runner(layers, H.HAPI_BF16, raw, (3, 8, 8))
    x = torch.zeros((batch, 3, 8, 8), dtype=torch.bfloat16, device="cuda")
    got = r.extract_np(x, 3)
    assert got.shape == (batch, T, D)
    return got


def _large_tiles(batch):
    # 256 x 256 tiles of fc1, which take more than half the CUs
    return ((batch * T + 255) // 256) * (F // 256)


SWEEPS = {
    "edges": np.array((EDGES + [-0.5] * D)[:D]),
    "-7 .. -3.5": np.linspace(-7.0, -3.5, D),
    "-3.5 .. -1": np.linspace(-3.5, -1.0, D),
    "-1 .. 1": np.linspace(-1.0, 1.0, D),
    "1 .. 7": np.linspace(1.0, 7.0, D),
}


@pytest.mark.parametrize("sweep", SWEEPS)
@pytest.mark.parametrize("large", [False, True])
def test_gelu_epilogue_over_its_range(sweep, large):
    bias = SWEEPS[sweep].astype(np.float32)
    batch = 430 if large else 1
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert (2 * _large_tiles(batch) > cus) == large
    got = _picked(bias, batch).astype(np.float64)
    ref = np.array([float(v) * 0.5 * math.erfc(-float(v) / math.sqrt(2.0)) for v in bias])
    # One rounding to bf16, 2^-8 at most (the block adds zero to it), and the
    # activation's own error: in fp32 arithmetic with a correctly rounded exp2
    # 5.1e-8 for negative values and 6.2e-8 up to 1, past that a rounding to
    # fp32, which the first term holds.  An exp2 of one ulp adds 2^-24 of
    # |v| Phi(-|v|) <= 0.17.
    tol = 2.0 ** -8 * np.abs(ref) + 8e-8
    assert np.all(np.abs(got - ref) <= tol), (sweep, np.abs(got - ref).max())


@pytest.mark.parametrize("large", [False, True])
def test_gelu_of_infinities_and_nan(large):
    # v Phi(v) as products: -inf times 0 is NaN (as 0.5 v (1 + erf(v / sqrt 2))
    # gives), inf stays inf.  fc2 multiplies every other channel's zero weight with
    # the value, which makes NaN of an infinity too, so only the picked channel tells.
    batch = 430 if large else 1
    for v, want in ((-np.inf, np.isnan), (np.nan, np.isnan), (np.inf, np.isposinf)):
        bias = np.full(D, 0.5, np.float32)
        bias[7] = v
        got = _picked(bias, batch)
        assert np.all(want(got[:, :, 7])), v
