"""The fp32 convolution kernel's tile shapes and slice modes against each other.

A long reduction's slices run as separate workgroups and are added by a second
kernel, or one after another inside a workgroup, by the number of tiles.  Both
add them in slice order, so a row of a large batch must equal, bit for bit, the
same image extracted alone (which the oracle checks cover).
"""
import pytest
import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models as PM
import synth
from tests.hip_harness import Runner, assert_routes, images_for

pytestmark = pytest.mark.gpu

DMA64, DMA128 = "conv_f32_dma_kernel<64, 64, 5", "conv_f32_dma_kernel<128, 64, 4"
STAGED, SUM = "conv_f32_kernel<", "f32_split_reduce_kernel"

# (NCHW input, C, N, k, s, p, (H, W), batch, kernels of the batch): 64 x 64 tiles with slices in
# sequence from 768 tiles, 128 x 64 tiles from 1024 on a 256-CU device
CASES = [
    (False, 64, 192, 5, 1, 2, (27, 27), 24, [DMA64]),     # 6 slices, 822 tiles of 64 x 64, ragged M
    (False, 64, 192, 5, 1, 2, (27, 27), 92, [DMA128]),    # 1572 tiles of 128 x 64, ragged M
    (False, 96, 264, 3, 2, 1, (33, 33), 96, [DMA128]),    # 3 slices, stride 2, ragged N
    (False, 32, 72, 1, 1, 0, (23, 23), 130, [DMA128]),    # 1 x 1, one slice, two k-tiles
    (False, 16, 64, 1, 1, 0, (40, 40), 90, [DMA128]),     # one k-tile: fewer than the ring's stages
    (True, 3, 64, 11, 4, 2, (63, 63), 600, [DMA128]),     # element gather, 1055 tiles of 128 x 64
    (True, 5, 40, 3, 2, 1, (21, 21), 7, [DMA64]),         # element gather, three k-tiles, ragged both ways
    (True, 3, 64, 19, 3, 9, (25, 25), 3, [STAGED, SUM]),  # K = 1083: past the tap table, the register-staged kernel
    # 12,288 rows and more lie past the row that the DMA kernel marks absent taps with: the
    # register-staged kernel's other loaders, slices apart and summed by the second launch, or one slice
    (False, 64, 72, 3, 1, 1, (12289, 3), 2, [STAGED, SUM]),
    (False, 16, 64, 3, 2, 1, (12291, 5), 3, [STAGED]),
    (False, 512, 40, 1, 1, 0, (12300, 1), 2, [STAGED, SUM]),
]


@pytest.mark.parametrize("case", CASES)
def test_f32_tiles_equal_single_images(case):
    nchw, C, N, k, s, p, HW, batch, kernels = case
    layers = ([] if nchw else [PM.maxpool(1, 1)]) + [PM.conv(C, N, k, s, p, bias=True)]
    params = [synth.param(13, 1, (N, C, k, k), "he"), synth.param(13, 2, (N,), "bias")]
    print(f"case {case}", flush=True)
    r = Runner(layers, H.HAPI_F32, params, (C, *HW))
    xd, xv = images_for(H.HAPI_F32, synth.images(13, batch, C, *HW))
    assert_routes(lambda: r.extract(xd, len(layers), inflight=1, chunk=batch), wanted=kernels)
    big = r.extract(xd, len(layers), inflight=1, chunk=batch)
    for i in (0, batch // 2, batch - 1):
        one = r.extract(xd[i:i + 1].contiguous(), len(layers))
        assert torch.equal(big[i:i + 1].view(torch.int32), one.view(torch.int32)), i
    # and against 64 bits on the last image: K products in sums of K terms
    ref = torch.nn.functional.conv2d(torch.from_numpy(xv[-1:]).double(), torch.from_numpy(params[0]).double(),
                                     torch.from_numpy(params[1]).double(), stride=s, padding=p).clamp(min=0)
    mag = torch.nn.functional.conv2d(torch.from_numpy(xv[-1:]).double().abs(), torch.from_numpy(params[0]).double().abs(),
                                     torch.from_numpy(params[1]).double().abs(), stride=s, padding=p)
    err = (big[-1:].cpu().double() - ref).abs()
    assert bool((err <= (C * k * k + 2) * 2.0 ** -24 * mag).all())
