"""1x1 convolutions whose columns run through all images (hidet_conv2d_implicit_gemm without a configuration, from the number of
tiles on that the size-based choice asks for): one to five stages of K, whole and partial, images of a chunk and more, odd
numbers of pixels, tensors of odd alignment, against the CPU oracle within the derived bound."""
import numpy as np
import pytest
import torch

import oracle
from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TORCH_DTYPE, assert_elementwise, conv_scale, to_f64, to_gpu

# images, input channels, height, width, output channels, residual
SHAPES = [(1000, 8, 3, 3, 72, True), (2064, 32, 2, 4, 130, False), (140, 64, 7, 7, 200, True), (500, 72, 3, 5, 136, True),
          (90, 104, 14, 13, 96, False), (90, 128, 13, 13, 65, True), (55, 160, 17, 17, 128, False), (1180, 40, 7, 7, 64, True),
          (60, 256, 11, 11, 256, True)]


def tile(Nb, IC, H, W, OC, dtype=hb.HIDET_F16, k=1, s=1, pad=0):
    i = hb.hidet_config_info(hb.hidet_conv2d_untuned_config(dtype, (Nb, IC, H, W), (OC, IC, k, k), (s, s), (pad, pad)))
    return i["block_m"], i["block_n"], i["schedule"]


def test_the_choice_between_the_two_forms():
    for Nb, IC, H, W, OC, _ in SHAPES:
        assert tile(Nb, IC, H, W, OC) == (128, 128, 1), (Nb, IC, H, W, OC)
    assert tile(274, 512, 7, 7, 128) == (128, 128, 1)  # 120 tiles; 119 below
    assert tile(272, 512, 7, 7, 128) != (128, 128, 1)
    assert tile(514, 256, 8, 8, 80) == (128, 128, 1)  # aligned rows: 257 tiles; 256 below
    assert tile(512, 256, 8, 8, 80) != (128, 128, 1)
    assert tile(1170, 64, 7, 7, 64)[:2] == (128, 128) and tile(1168, 64, 7, 7, 64)[:2] != (128, 128)  # 512 and 511 tiles
    assert tile(4000, 256, 1, 7, 256)[:2] != (128, 128) or tile(4000, 256, 1, 7, 256)[2] != 1  # no row of a chunk


def test_the_form_that_is_taken():
    """The tile alone does not tell the forms apart: the batched GEMM takes the same one for some layers."""
    def form(Nb, IC, H, W, OC, dtype=hb.HIDET_F16):
        return hb.hidet_conv2d_untuned_form(dtype, (Nb, IC, H, W), (OC, IC, 1, 1))

    for Nb, IC, H, W, OC, _ in SHAPES:
        assert form(Nb, IC, H, W, OC) == hb.HIDET_CONV_IMAGES and form(Nb, IC, H, W, OC, hb.HIDET_F32) == hb.HIDET_CONV_BATCHED
    assert form(274, 512, 7, 7, 128) == hb.HIDET_CONV_IMAGES and form(272, 512, 7, 7, 128) == hb.HIDET_CONV_BATCHED
    assert form(514, 256, 8, 8, 80) == hb.HIDET_CONV_IMAGES and form(512, 256, 8, 8, 80) == hb.HIDET_CONV_BATCHED
    assert form(1170, 64, 7, 7, 64) == hb.HIDET_CONV_IMAGES and form(1168, 64, 7, 7, 64) == hb.HIDET_CONV_BATCHED
    # tiles enough, but one round of large ones or a few full small ones carry the batched GEMM faster
    assert form(64, 1024, 14, 14, 256) == hb.HIDET_CONV_BATCHED and form(125, 2048, 14, 14, 512) == hb.HIDET_CONV_BATCHED
    assert form(65, 192, 32, 32, 32) == hb.HIDET_CONV_BATCHED and form(64, 512, 7, 7, 2048) == hb.HIDET_CONV_IMAGES
    assert form(4000, 256, 1, 7, 256) == hb.HIDET_CONV_BATCHED and form(140, 60, 7, 7, 200) == hb.HIDET_CONV_BATCHED


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_pointwise_over_all_images(shape, dtype):
    Nb, IC, H, W, OC, residual = shape
    c = wl.conv_case(9700 + SHAPES.index(shape), Nb, IC, H, W, OC, 1, 1, 1, 0, dtype, residual=residual)
    size = Nb * OC * H * W
    w, bias, res = to_gpu(c["w"], dtype), to_gpu(c["bias"], dtype), to_gpu(c["residual"], dtype)
    epi = hb.make_epilogue(bias=bias, bias_axis=hb.HIDET_BIAS_PER_ROW, residual=res, relu=True)
    x64, w64 = wl.widen(c["x"], dtype), wl.widen(c["w"], dtype)
    b64, r64 = wl.widen(c["bias"], dtype), None if res is None else wl.widen(c["residual"], dtype)
    ref = oracle.conv2d(x64, w64, bias=b64, residual=r64, relu=True)
    for shift in (0, 1):  # x and y at 16-byte and at element alignment, the latter at the end of their allocations
        x = torch.empty(c["x"].size + shift, dtype=TORCH_DTYPE[dtype], device="cuda")[shift:].view(Nb, IC, H, W)
        x.copy_(to_gpu(c["x"], dtype))
        around = torch.full((size + 32 + shift,), 7.0, dtype=TORCH_DTYPE[dtype], device="cuda")
        y = around[16 + shift:16 + shift + size].view(Nb, OC, H, W)
        y.fill_(float("nan"))
        hb.hidet_conv2d_implicit_gemm(x, w, y, stride=(1, 1), pad=(0, 0), epilogue=epi)
        torch.cuda.synchronize()
        got = to_f64(y)
        assert_elementwise(got, ref, conv_scale(x64, w64, (1, 1), (0, 0), 1.0, b64, r64), dtype, IC, "pointwise %s %s" % (shape, dtype))
        assert np.all(to_f64(around[:16 + shift]) == 7.0) and np.all(to_f64(around[16 + shift + size:]) == 7.0)
