"""The 256 x 256-tile convolution kernel against the small-tile kernels.

Layers whose rounds of 256 x 256 tiles are filled well enough run on their own kernel.
A row of a large batch must equal, bit for bit, the same image extracted alone
in a batch of three, which the small-tile kernels (checked against the oracle
bit for bit and within tolerance) run: every kernel sums in the same order.
Each case names the instances (loader, kernel size, epilogue) that its large
batch has to run on, so none compares a kernel with itself.
"""
import pytest
import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models as PM
import synth
from tests.hip_harness import Runner, assert_routes, images_for

pytestmark = pytest.mark.gpu

POOL1 = PM.maxpool(1, 1)


def _bneck(cin, w, stride=1):
    return dict(kind=H.HAPI_BOTTLENECK, cin=cin, width=w, cout=4 * w, stride=stride)


def _basic(cin, cout, stride=1):
    return dict(kind=H.HAPI_BASIC_BLOCK, cin=cin, cout=cout, stride=stride)


GEMM, NHWC, CAT = 1, 0, 5              # loaders
PLAIN, GELU, POOL, RES = 0, 1, 2, 3    # epilogues

# name: (layers, input shape, batch, inflight, instances); the last layer only takes the split
CASES = {
    # M = 36 x 31 x 31: 136 row tiles, the last ragged; nine taps with padding
    "3x3": ([POOL1, PM.conv(64, 256, 3, 1, 1), PM.conv(256, 64, 1)], (64, 31, 31), 36, 1, [(NHWC, 3, PLAIN)]),
    "3x3 of two partitions": ([POOL1, PM.conv(64, 256, 3, 1, 1), PM.conv(256, 64, 1)], (64, 31, 31), 72, 2,
                              [(NHWC, 3, PLAIN)]),
    "3x3 stride 2": ([POOL1, PM.conv(128, 512, 3, 2, 1), PM.conv(512, 64, 1)], (128, 45, 45), 33, 1, [(NHWC, 3, PLAIN)]),
    # two k-tiles (the fewest), a ragged column tile (1088 = 4.25 tiles)
    "1x1 ragged columns": ([POOL1, PM.conv(128, 1088, 1), PM.conv(1088, 64, 1)], (128, 29, 29), 9, 1, [(GEMM, 1, PLAIN)]),
    "1x1 stride 2": ([POOL1, PM.conv(128, 256, 1, 2), PM.conv(256, 64, 1)], (128, 61, 61), 36, 1, [(NHWC, 1, PLAIN)]),
    # an odd number of k-tiles, and more tiles than CUs: several tiles per workgroup
    "1x1 many tiles": ([POOL1, PM.conv(192, 1024, 1), PM.conv(1024, 64, 1)], (192, 30, 30), 81, 1, [(GEMM, 1, PLAIN)]),
    # pooled to 15 x 17 windows, odd both ways, the last row tile ragged
    "3x3 and pooling": ([POOL1, PM.conv(64, 256, 3, 1, 1), PM.maxpool(2, 2), PM.conv(256, 64, 1)], (64, 30, 34), 33, 1,
                        [(NHWC, 3, POOL)]),
    "residual and fused shortcuts": ([POOL1, _bneck(256, 128, 2), _bneck(512, 256), _bneck(1024, 256), PM.conv(1024, 64, 1)],
                                     (256, 57, 57), 37, 1, [(CAT, 1, PLAIN), (GEMM, 1, RES)]),
    "basic blocks": ([POOL1, _basic(64, 256, 2), _basic(256, 256), PM.conv(256, 64, 1)], (64, 57, 57), 41, 1,
                     [(NHWC, 3, PLAIN), (CAT, 3, PLAIN), (NHWC, 3, RES)]),
}


def _check(layers, in_shape, batch, inflight, raw, split, instances):
    r = Runner(layers, H.HAPI_BF16, raw, in_shape)
    xd, _ = images_for(H.HAPI_BF16, synth.images(11, batch, *in_shape))
    assert_routes(lambda: r.extract(xd, split, inflight=inflight),
                  wanted=["conv_bf16_pp_kernel<%d, %d, %d>" % i for i in instances])
    assert_routes(lambda: r.extract(xd[:3].contiguous(), split, inflight=1), unwanted=["conv_bf16_pp_kernel"])
    big = r.extract(xd, split, inflight=inflight)
    for rows in ([0, 1, 2], [batch // 2 - 1, batch // 2, batch // 2 + 1], [batch - 3, batch - 2, batch - 1]):
        small = r.extract(xd[rows].contiguous(), split, inflight=1)
        assert torch.equal(big[rows].view(torch.int16), small.view(torch.int16)), rows


@pytest.mark.parametrize("name", CASES)
def test_large_tiles_equal_small_tiles(name):
    layers, in_shape, batch, inflight, instances = CASES[name]
    raw = synth.params(11, PM.raw_manifest(layers, in_shape))
    print(f"case {name}", flush=True)
    _check(layers, in_shape, batch, inflight, raw, len(layers), instances)


# qkv and fc1 (GELU) at 66 images or partitions of 65, the projections with residual
# (12 and 48 k-tiles, in place) from 108 on: 86 x 3 tiles of 128 x 256
@pytest.mark.parametrize("batch,inflight,instances", [
    (66, 1, [(GEMM, 1, PLAIN), (GEMM, 1, GELU)]),
    (130, 2, [(GEMM, 1, PLAIN), (GEMM, 1, GELU)]),
    (110, 1, [(GEMM, 1, PLAIN), (GEMM, 1, GELU), (GEMM, 1, RES)])])
def test_encoder_block_large_tiles(batch, inflight, instances):
    # 4 x 4 patches of 40 x 40 images: 101 tokens; a second block takes the split
    layers = PM.vit(image=40, patch=4, dim=768, heads=12, mlp=3072, depth=2)
    raw = synth.params(12, PM.raw_manifest(layers, (3, 40, 40)))
    print(f"case encoder block b{batch}", flush=True)
    _check(layers, (3, 40, 40), batch, inflight, raw, 4, instances)
