"""The GELU epilogue against float64 through an encoder block.

With zero out-projection and identity-like fc weights, an encoder block's output
is x + gelu(ln2(x) * 1 + fc1 bias), so the bias sweeps the activation's whole
range: the polynomial's fitted part, its tail, both signs and zero.
"""
import math

import numpy as np
import pytest
import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models as PM
from tests.hip_harness import Runner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 430])   # small tiles; 144 tiles of 256 x 256
def test_gelu_epilogue_over_its_range(batch):
    D, F, T = 64, 4096, 5
    layers = PM.vit(image=8, patch=4, dim=D, heads=1, mlp=F, depth=1)[:3]
    man = PM.raw_manifest(layers, (3, 8, 8))
    raw = [np.zeros(s, np.float32) for s, _ in man]
    # fc1: no weights, biases -12 .. 12 (and 0); fc2: unit j adds channel j of groups of F / D
    bias = np.linspace(-12.0, 12.0, F).astype(np.float32)
    bias[F // 2] = 0.0
    shapes = [s for s, _ in man]
    i1 = shapes.index((F, D))
    raw[i1 + 1] = bias
    w2 = np.zeros((D, F), np.float32)
    pick = np.arange(D) * (F // D) + 17 % (F // D)
    w2[np.arange(D), pick] = 1.0
    raw[i1 + 2] = w2
    r = Runner(layers, H.HAPI_BF16, raw, (3, 8, 8))
    x = torch.zeros((batch, 3, 8, 8), dtype=torch.bfloat16, device="cuda")
    got = r.extract_np(x, 3)
    b = bias[pick].astype(np.float64)
    ref = np.array([v * 0.5 * math.erfc(-v / math.sqrt(2.0)) for v in b])
    # two roundings to bf16 (the activation, the block's output), 2^-8 each at
    # most, and the activation's own error of at most 2.5e-7
    tol = 2 * 2.0 ** -8 * np.abs(ref) + 5e-7
    assert got.shape == (batch, T, D)
    assert np.all(np.abs(got - ref) <= tol), np.abs(got - ref).max()
