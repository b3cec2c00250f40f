"""Small-tile routes of the convolutions against the large-tile ones.

A few images run on 32 x 64, 64 x 64, 64 x 32 or 32 x 32 tiles, more on larger
ones; the kernels sum in one order, so rows of batches of different sizes must
agree bit for bit.  Batches are chosen on both sides of each rule for a 256-CU
device, and each case names the tiles of its smallest batch (which its largest
must not run on).
"""
import pytest
import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models as PM
import synth
from tests.hip_harness import Runner, assert_routes, images_for

pytestmark = pytest.mark.gpu

POOL1 = PM.maxpool(1, 1)

RING32 = "conv_bf16_ws2_kernel<32, 64, 1, 2, 6"   # six stages, handed back one barrier late

CASES = {
    # k-tiles 1 .. 9 of the 32 x 64 route's six-stage ring, then 64 x 64 and 128-wide tiles
    "1x1, two k-tiles": ([POOL1, PM.conv(128, 128, 1), PM.conv(128, 64, 1)], (128, 13, 13), (1, 3, 40, 130), [RING32]),
    "1x1, five k-tiles": ([POOL1, PM.conv(320, 128, 1), PM.conv(128, 64, 1)], (320, 13, 13), (1, 3, 40, 130), [RING32]),
    "1x1, six k-tiles": ([POOL1, PM.conv(384, 128, 1), PM.conv(128, 64, 1)], (384, 13, 13), (1, 3, 40, 130), [RING32]),
    "3x3, nine k-tiles": ([POOL1, PM.conv(64, 136, 3, 1, 1), POOL1], (64, 13, 13), (1, 3, 60, 160), [RING32]),
    # 264 tiles of 64 x 64 at the second batch: long reductions, fragments one k-step ahead
    "1x1, 48 k-tiles": ([POOL1, PM.conv(3072, 768, 1), PM.conv(768, 64, 1)], (3072, 13, 13), (1, 8, 30, 60), [RING32]),
    "3x3, 72 k-tiles": ([POOL1, PM.conv(512, 512, 3, 1, 1), PM.conv(512, 64, 1)], (512, 11, 11), (1, 17, 40, 140), [RING32]),
    # the split layer: NCHW from the epilogue, on 64 x 64 and 128 x 128 tiles
    "3x3 split": ([POOL1, PM.conv(64, 136, 3, 1, 1)], (64, 13, 13), (1, 3, 40, 160), ["conv_bf16_ws2_kernel<64, 64, 2, 2, 4"]),
    "residual block": ([POOL1, dict(kind=H.HAPI_BOTTLENECK, cin=256, width=64, cout=256, stride=2),
                        dict(kind=H.HAPI_BOTTLENECK, cin=256, width=64, cout=256, stride=1), PM.conv(256, 64, 1)],
                       (256, 27, 27), (1, 2, 33, 130), [RING32]),
    # pre-activated 1 x 1 (ragged K: 72, 104, 136 ...) and the 32-channel 3 x 3
    "dense block": ([POOL1, PM.dense_block(64, 4)], (64, 13, 13), (1, 3, 48, 100, 220),
                    ["conv_bf16_ws2_kernel<32, 32, 1, 1, 6"]),
    "dense block, ragged prefixes": ([POOL1, PM.dense_block(72, 3, growth=40)], (72, 11, 11), (1, 3, 48, 300),
                                     ["conv_bf16_ws2_kernel<64, 64, 2, 2, 4, 1, 1, 2, true>"]),
    "dense block, narrow growth": ([POOL1, PM.dense_block(128, 3, growth=24), PM.batchnorm(200, True)], (128, 9, 9),
                                   (1, 5, 90, 250), ["conv_bf16_ws2_kernel<32, 32, 1, 1, 6"]),
}


@pytest.mark.parametrize("name", CASES)
def test_batches_agree(name):
    layers, in_shape, batches, tiles = CASES[name]
    raw = synth.params(14, PM.raw_manifest(layers, in_shape))
    print(f"case {name}", flush=True)
    r = Runner(layers, H.HAPI_BF16, raw, in_shape)
    xd, _ = images_for(H.HAPI_BF16, synth.images(14, max(batches), *in_shape))
    assert_routes(lambda: r.extract(xd[:batches[0]].contiguous(), len(layers), inflight=1), wanted=tiles)
    assert_routes(lambda: r.extract(xd, len(layers), inflight=1, chunk=len(xd)), unwanted=tiles)
    outs = [r.extract(xd[:b].contiguous(), len(layers), inflight=1, chunk=b) for b in batches]
    for b, o in zip(batches, outs):
        n = min(batches[0], b)
        assert torch.equal(o[:n].view(torch.int16), outs[0][:n].view(torch.int16)), b
        k = min(b, batches[-2])
        assert torch.equal(o[:k].view(torch.int16), outs[-1][:k].view(torch.int16)), b
    two = r.extract(xd, len(layers), inflight=2, chunk=(max(batches) + 1) // 2)
    assert torch.equal(two.view(torch.int16), outs[-1].view(torch.int16))
