"""The 256 x 256-tile convolution kernel against the small-tile kernels.

Layers with more tiles of 256 x 256 than half the CUs run on their own kernel.
A row of a large batch must equal, bit for bit, the same image extracted alone
in a batch of three, which the small-tile kernels (checked against the oracle
bit for bit and within tolerance) run: every kernel sums in the same order.
"""
import pytest
import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models as PM
import synth
from tests.hip_harness import Runner, images_for

pytestmark = pytest.mark.gpu

POOL1 = PM.maxpool(1, 1)


def _bneck(cin, w, stride=1):
    return dict(kind=H.HAPI_BOTTLENECK, cin=cin, width=w, cout=4 * w, stride=stride)


def _basic(cin, cout, stride=1):
    return dict(kind=H.HAPI_BASIC_BLOCK, cin=cin, cout=cout, stride=stride)


# name: (layers, input shape, batch, inflight); the last layer only takes the split
CASES = {
    # M = 36 x 31 x 31: 136 row tiles, the last ragged; nine taps with padding
    "3x3": ([POOL1, PM.conv(64, 256, 3, 1, 1), PM.conv(256, 64, 1)], (64, 31, 31), 36, 1),
    "3x3 of two partitions": ([POOL1, PM.conv(64, 256, 3, 1, 1), PM.conv(256, 64, 1)], (64, 31, 31), 72, 2),
    "3x3 stride 2": ([POOL1, PM.conv(128, 512, 3, 2, 1), PM.conv(512, 64, 1)], (128, 45, 45), 33, 1),
    # two k-tiles (the fewest), a ragged column tile (1088 = 4.25 tiles)
    "1x1 ragged columns": ([POOL1, PM.conv(128, 1088, 1), PM.conv(1088, 64, 1)], (128, 29, 29), 9, 1),
    "1x1 stride 2": ([POOL1, PM.conv(128, 256, 1, 2), PM.conv(256, 64, 1)], (128, 61, 61), 36, 1),
    # an odd number of k-tiles, and more tiles than CUs: several tiles per workgroup
    "1x1 many tiles": ([POOL1, PM.conv(192, 1024, 1), PM.conv(1024, 64, 1)], (192, 30, 30), 81, 1),
    "3x3 and pooling": ([POOL1, PM.conv(64, 256, 3, 1, 1), PM.maxpool(2, 2), PM.conv(256, 64, 1)], (64, 30, 34), 33, 1),
    "residual and fused shortcuts": ([POOL1, _bneck(256, 128, 2), _bneck(512, 128), _bneck(512, 256), PM.conv(1024, 64, 1)],
                                     (256, 57, 57), 33, 1),
    "basic blocks": ([POOL1, _basic(64, 256, 2), _basic(256, 256), PM.conv(256, 64, 1)], (64, 57, 57), 41, 1),
}


def _check(layers, in_shape, batch, inflight, raw, split):
    r = Runner(layers, H.HAPI_BF16, raw, in_shape)
    xd, _ = images_for(H.HAPI_BF16, synth.images(11, batch, *in_shape))
    big = r.extract(xd, split, inflight=inflight)
    for rows in ([0, 1, 2], [batch // 2 - 1, batch // 2, batch // 2 + 1], [batch - 3, batch - 2, batch - 1]):
        small = r.extract(xd[rows].contiguous(), split, inflight=1)
        assert torch.equal(big[rows].view(torch.int16), small.view(torch.int16)), rows


@pytest.mark.parametrize("name", CASES)
def test_large_tiles_equal_small_tiles(name):
    layers, in_shape, batch, inflight = CASES[name]
    raw = synth.params(11, PM.raw_manifest(layers, in_shape))
    print(f"case {name}", flush=True)
    _check(layers, in_shape, batch, inflight, raw, len(layers))


@pytest.mark.parametrize("batch,inflight", [(66, 1), (130, 2)])
def test_encoder_block_large_tiles(batch, inflight):
    # 4 x 4 patches of 40 x 40 images: 101 tokens; qkv, fc1 (GELU), the
    # projections with residual
    layers = PM.vit(image=40, patch=4, dim=768, heads=12, mlp=3072, depth=1)
    raw = synth.params(12, PM.raw_manifest(layers, (3, 40, 40)))
    print(f"case encoder block b{batch}", flush=True)
    _check(layers, (3, 40, 40), batch, inflight, raw, 3)
