"""Which tiles the bf16 convolutions run on, on a 256-CU device.

Results do not depend on the tiles (test_gpu_large_tiles and test_gpu_small_tiles
compare them bit for bit); times do: a route taken at a size where another kernel is
faster is the fault these cases pin.  Sizes lie on both sides of each rule.
"""
import pytest
import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models as PM
import synth
from tests.hip_harness import Runner, assert_routes, images_for, kernel_grids

pytestmark = pytest.mark.gpu

POOL1 = PM.maxpool(1, 1)
PP = "conv_bf16_pp_kernel"
# 64 x 64 tiles stored as NHWC (the split layer's go to NCHW): 3 x 3 and 1 x 1
W64 = "conv_bf16_ws2_kernel<64, 64, 2, 2, 4, 0, 3, 2"
W64L = "conv_bf16_ws2_kernel<64, 64, 2, 2, 4, 1, 1, 2"
TALL = "conv_bf16_pws_kernel<256, 128"


def _conv(cin, cout, k, hw, batch, inflight=1):
    # the second convolution takes the split
    return [POOL1, PM.conv(cin, cout, k, 1, k // 2), PM.conv(cout, 64, 1)], (cin, hw, hw), batch, inflight, 3


def _expansion(width, hw, batch, inflight=1):
    block = dict(kind=H.HAPI_BOTTLENECK, cin=4 * width, width=width, cout=4 * width, stride=1)
    return [POOL1, block, PM.conv(4 * width, 64, 1)], (4 * width, hw, hw), batch, inflight, 3


# (what, kernels to see, kernels not to see)
CASES = {
    # 256 x 256 tiles: one round of 147, two rounds for 294 (three halves are faster),
    # two for 441 (four halves)
    "3x3 147 tiles": (_conv(128, 256, 3, 56, 12), [PP], []),
    "3x3 294 tiles": (_conv(128, 256, 3, 56, 24), [], [PP]),
    "3x3 441 tiles": (_conv(128, 256, 3, 56, 36), [PP], []),
    # a residual short reduction: rounds filled to 148, 196 of 256 and 296 of 512
    "expansion 148 tiles": (_expansion(256, 14, 48), [], [PP]),
    "expansion 196 tiles": (_expansion(256, 14, 64), [PP + "<1, 1, 3>"], []),
    "expansion 296 tiles": (_expansion(256, 14, 96), [], [PP + "<1, 1, 3>"]),
    # the two-k-tile residual expansion has a kernel of its own at every size
    "short expansion": (_expansion(128, 28, 64), ["conv_bf16_short_kernel"], [PP + "<1, 1, 3>"]),
    # 148 tiles of 128 x 128 on 256 CUs: 64 x 64 tiles only for short reductions
    "3x3 of 9 k-tiles": (_conv(64, 128, 3, 28, 24), [W64], []),
    "3x3 of 36 k-tiles": (_conv(256, 256, 3, 14, 48), ["conv_bf16_pws_kernel<128, 128"], [W64]),
    "1x1 of 12 k-tiles": (_conv(768, 768, 1, 14, 16), [W64L], []),
    "1x1 of 48 k-tiles": (_conv(3072, 768, 1, 14, 16), ["conv_bf16_pws_kernel<128, 128"], [W64L]),
    # 64 x 64 tiles of long reductions, one for each of the 256 CUs and up to a third of them more
    "1x1 of 48 k-tiles, 264 tiles": (_conv(3072, 768, 1, 13, 8), ["conv_bf16_ws2_step_kernel"], [W64L]),
    "1x1 of 48 k-tiles, 360 tiles": (_conv(3072, 768, 1, 13, 11), [W64L], ["conv_bf16_ws2_step_kernel"]),
    "3x3 of 72 k-tiles, 264 tiles": (_conv(512, 512, 3, 11, 17), ["conv_bf16_ws2_step_kernel"], [W64]),
    # 128-channel 3 x 3s: the persistent kernel where two rounds of 256-row tiles are filled to 3/4,
    # more rounds to 7/8
    "3x3 to 128, 294 tiles": (_conv(128, 128, 3, 56, 24), [], [TALL]),
    "3x3 to 128, 392 tiles": (_conv(128, 128, 3, 56, 32), [TALL], []),
    "3x3 to 128, 698 tiles": (_conv(128, 128, 3, 56, 57), [TALL], []),
    "3x3 to 128, 1029 tiles": (_conv(128, 128, 3, 56, 84), [], [TALL]),
    "3x3 to 128, two partitions of 319": (_conv(128, 128, 3, 28, 208, 2), [], [TALL]),
}


@pytest.mark.parametrize("name", CASES)
def test_route(name):
    (layers, in_shape, batch, inflight, split), wanted, unwanted = CASES[name]
    raw = synth.params(15, PM.raw_manifest(layers, in_shape))
    print(f"case {name}", flush=True)
    r = Runner(layers, H.HAPI_BF16, raw, in_shape)
    xd, _ = images_for(H.HAPI_BF16, synth.images(15, 1, *in_shape))
    xd = xd.expand(batch, *in_shape).contiguous()
    assert_routes(lambda: r.extract(xd, split, inflight=inflight, chunk=-(-batch // inflight)), wanted, unwanted)


@pytest.mark.parametrize("side,batch,workgroups", [
    (224, 8, 224),     # bands of two pooled rows: 28 an image
    (224, 16, 256),    # one for every CU
    (192, 21, 252),    # 13 bands an image would be 273 workgroups: 12, of four rows
    (256, 13, 247),    # 20 would be 260: 19
    (224, 40, 280),    # from about 19 images on, bands of four rows and more, a workgroup per CU
    (224, 130, 260),   # two bands an image
])
def test_stem_bands(side, batch, workgroups):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("counted for 256 CUs")
    layers = PM.resnet18()[:3]
    raw = synth.params(16, PM.raw_manifest(layers, (3, side, side)))
    print(f"case {batch} images of {side}", flush=True)
    r = Runner(layers, H.HAPI_BF16, raw, (3, side, side))
    xd = torch.zeros((batch, 3, side, side), dtype=torch.bfloat16, device="cuda")
    for _ in range(3):  # the tracer can drop records
        got = [n for k, n in kernel_grids(lambda: r.extract(xd, 3, inflight=1, chunk=batch)) if k == "stem_pool_kernel"]
        if got:
            break
    assert got == [workgroups]
