"""Attention over scores of every size up to the largest finite ones.

Tokens are rows of a Hadamard matrix, which layer-norm leaves as they are, and the
query and key projections are multiples of the identity, so the scores are a
multiple of 64 on the diagonal and 0 elsewhere, exactly; with the queries and keys
in the bias instead, all scores are equal.  The softmax is then one-hot, uniform
over the other tokens or uniform, whatever the scale.
"""
import numpy as np
import pytest
import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models as PM
from tests.hip_harness import Runner

pytestmark = pytest.mark.gpu

D, T = 64, 37    # one head; two key tiles, the second ragged

# query times key scale: scores of 64 times that, 1e3 to 2.6e38
SCALES = [16.0, 1e3, 1.7e7, 1e8, 1.3e8, 3.1e9, 4.4e10, 7.7e12, 9.1e17, 2.3e25, 4e36]


def _hadamard(n):
    h = np.ones((1, 1), np.float32)
    while h.shape[0] < n:
        h = np.block([[h, h], [h, -h]])
    return h


def _block(wq, wk, bq, bk, tokens):
    """An encoder block of 0.5-scaled identity values and no MLP, as raw weights."""
    layers = PM.vit(image=24, patch=4, dim=D, heads=1, mlp=64, depth=1)[:3]
    raw = [np.zeros(s, np.float32) for s, _ in PM.raw_manifest(layers, (3, 24, 24))]
    eye = np.eye(D, dtype=np.float32)
    raw[3][:] = tokens.reshape(raw[3].shape)                     # position embeddings
    raw[4][:] = 1.0                                              # ln1 gamma
    raw[6][:] = np.concatenate([wq * eye, wk * eye, 0.5 * eye])  # in-projection
    raw[7][:] = np.concatenate([np.full(D, bq), np.full(D, bk), np.zeros(D)]).astype(np.float32)
    raw[8][:] = eye                                              # out-projection
    return layers, raw


def _attend(wq, wk, bq, bk, tokens):
    layers, raw = _block(wq, wk, bq, bk, tokens)
    r = Runner(layers, H.HAPI_BF16, raw, (3, 24, 24))
    x = torch.zeros((2, 3, 24, 24), dtype=torch.bfloat16, device="cuda")
    return r.extract_np(x, 3)


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("kind", ["one-hot", "others", "equal", "equal, negative"])
def test_scores_of_any_size(kind, scale):
    a = float(np.sqrt(scale))
    tokens = _hadamard(D)[1:T + 1]
    print(f"case {kind}, scores of {64 * scale:g}", flush=True)
    if kind == "one-hot":      # the diagonal scores win by 64 scale / 8 >= 128
        got = _attend(a, a, 0.0, 0.0, tokens)
        att = 0.5 * tokens
    elif kind == "others":     # the diagonal scores are the lowest
        got = _attend(a, -a, 0.0, 0.0, tokens)
        att = 0.5 * (tokens.sum(0) - tokens) / (T - 1)
    else:
        got = _attend(0.0, 0.0, a, a if kind == "equal" else -a, tokens)
        att = np.broadcast_to(0.5 * tokens.mean(0), tokens.shape)
    # Two roundings to bf16, of 2^-8 relative at most each: the attention's output
    # and the block's.  Everything before them is exact (the layer-norm's epsilon
    # moves its +-1 by 5e-7, which rounds away).
    ref = tokens + att
    tol = 2.0 ** -8 * (np.abs(att) + np.abs(ref)) + 1e-6
    assert got.shape == (2, T, D)
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - ref) <= tol), np.abs(got - ref).max()
