"""3x3 and 5x5 convolutions that run from a patch of the input in LDS (hidet_conv2d_implicit_gemm without a configuration): one to five
stages of 16 channels, both tile heights and their remainders, the shortest and the longest rows, few and many images, tensors of
odd alignment, against the CPU oracle within the derived bound; and the choice between them and the gather."""
import numpy as np
import pytest
import torch

import oracle
from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TORCH_DTYPE, assert_elementwise, conv_scale, to_f64, to_gpu

# images, input channels, height, width, output channels, residual, rows of the tile, taps of a filter row
SHAPES = [(190, 16, 6, 6, 40, True, 64, 3), (9, 32, 31, 31, 80, False, 64, 3), (3, 48, 60, 62, 33, True, 64, 3), (3, 16, 61, 61, 64, True, 64, 3),
          (37, 64, 14, 14, 130, False, 64, 3), (25, 80, 13, 15, 192, True, 64, 3), (70, 32, 14, 14, 200, True, 128, 3), (30, 48, 27, 29, 96, False, 128, 3),
          (260, 16, 7, 7, 129, False, 64, 3), (64, 16, 28, 28, 65, True, 128, 3),
          (60, 16, 14, 14, 66, True, 64, 5), (20, 32, 29, 29, 64, False, 64, 5), (33, 48, 17, 13, 100, True, 64, 5), (150, 80, 9, 11, 40, False, 64, 5),
          (20, 16, 14, 14, 64, True, 64, 5), (10, 32, 14, 14, 256, False, 64, 5)]


def rows(Nb, IC, H, W, OC, dtype=hb.HIDET_F16, k=3, s=1, pad=1):
    return hb.hidet_conv2d_patch_rows(dtype, (Nb, IC, H, W), (OC, IC, k, k), (s, s), (pad, pad))


def test_the_choice_between_patch_and_gather():
    for Nb, IC, H, W, OC, _, bm, k in SHAPES:
        assert rows(Nb, IC, H, W, OC, k=k, pad=k // 2) == bm, (Nb, IC, H, W, OC)
        assert rows(Nb, IC, H, W, OC, hb.HIDET_BF16, k, 1, k // 2) == bm and rows(Nb, IC, H, W, OC, hb.HIDET_F32, k, 1, k // 2) == 0
    assert rows(40, 64, 14, 14, 64) == 0 and rows(41, 64, 14, 14, 64) == 64  # 71 and 73 tiles of 128 columns
    assert rows(64, 64, 14, 14, 64, s=2) == 0 and rows(64, 64, 14, 14, 64, k=7, pad=3) == 0 and rows(64, 64, 14, 14, 64, pad=0) == 0
    assert rows(64, 60, 14, 14, 64) == 0 and rows(64, 64, 14, 14, 15) == 0  # whole stages, half a matrix-core tile of rows
    assert rows(8, 64, 62, 62, 64) == 64 and rows(8, 64, 62, 63, 64) == 0  # the border of a row in the patch
    assert rows(1000, 64, 5, 5, 64) == 0 and rows(1000, 64, 6, 6, 64) == 64  # more than two fifths of zeros
    assert rows(64, 96, 14, 14, 256) == 128 and rows(74, 96, 14, 14, 256) == 64  # 226 tiles of 128 rows; 262
    assert rows(110, 96, 14, 14, 256) == 128 and rows(146, 96, 14, 14, 256) == 64  # 388; 514
    assert rows(104, 256, 14, 14, 64, k=5, pad=2) == 64 and rows(51, 256, 14, 14, 64, k=5, pad=2) == 64  # 102 tiles: 44.8 us, patch 32.9
    assert rows(60, 272, 14, 14, 64, k=5, pad=2) == 64 and rows(75, 272, 14, 14, 64, k=5, pad=2) == 64  # 120: 47.4 and 33.5 us
    assert rows(12, 256, 14, 14, 256, k=5, pad=2) == 64 and rows(28, 512, 7, 7, 512, k=5, pad=2) == 64  # 42.8 and 31.5, 90.6 and 59.5 us
    assert rows(19, 16, 14, 14, 64, k=5, pad=2) == 0 and rows(20, 16, 14, 14, 64, k=5, pad=2) == 64  # 38 and 40 tiles
    assert rows(40, 64, 29, 29, 64, k=5, pad=2) == 64 and rows(40, 64, 29, 30, 64, k=5, pad=2) == 0


def test_the_gather_where_it_is_faster():
    """Rows of 8 and 16 pixels, of which no column of the gather is padding, and patches of a second round that is nearly empty."""
    assert rows(101, 256, 8, 8, 256, k=5, pad=2) == 0 and rows(64, 128, 16, 16, 128, k=5, pad=2) == 0
    assert rows(13, 512, 8, 8, 512) == 0 and rows(128, 128, 8, 8, 32) == 0
    assert rows(8, 1024, 15, 15, 1024, k=5, pad=2) == 0 and rows(48, 512, 8, 8, 512, k=5, pad=2) == 0  # 198 us, patch 223; 99 and 119
    assert rows(32, 512, 16, 16, 128, k=5, pad=2) == 64 and rows(40, 512, 8, 8, 512, k=5, pad=2) == 64  # 81 us, patch 58; 101 and 65
    assert rows(64, 512, 7, 7, 512) == 64 and rows(64, 256, 14, 14, 256) == 128 and rows(60, 256, 14, 14, 256, k=5, pad=2) == 64


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_patch_convolution(shape, dtype):
    Nb, IC, H, W, OC, residual, _, k = shape
    c = wl.conv_case(9800 + SHAPES.index(shape), Nb, IC, H, W, OC, k, k, 1, k // 2, dtype, residual=residual)
    size = Nb * OC * H * W
    w, bias, res = to_gpu(c["w"], dtype), to_gpu(c["bias"], dtype), to_gpu(c["residual"], dtype)
    epi = hb.make_epilogue(bias=bias, bias_axis=hb.HIDET_BIAS_PER_ROW, residual=res, relu=True)
    x64, w64 = wl.widen(c["x"], dtype), wl.widen(c["w"], dtype)
    b64, r64 = wl.widen(c["bias"], dtype), None if res is None else wl.widen(c["residual"], dtype)
    ref = oracle.conv2d(x64, w64, stride=(1, 1), pad=(k // 2, k // 2), bias=b64, residual=r64, relu=True)
    for shift in (0, 1):  # x and y at 16-byte and at element alignment, the latter at the end of their allocations
        x = torch.empty(c["x"].size + shift, dtype=TORCH_DTYPE[dtype], device="cuda")[shift:].view(Nb, IC, H, W)
        x.copy_(to_gpu(c["x"], dtype))
        around = torch.full((size + 32 + shift,), 7.0, dtype=TORCH_DTYPE[dtype], device="cuda")
        y = around[16 + shift:16 + shift + size].view(Nb, OC, H, W)
        y.fill_(float("nan"))
        hb.hidet_conv2d_implicit_gemm(x, w, y, stride=(1, 1), pad=(k // 2, k // 2), epilogue=epi)
        torch.cuda.synchronize()
        got = to_f64(y)
        assert_elementwise(got, ref, conv_scale(x64, w64, (1, 1), (k // 2, k // 2), 1.0, b64, r64), dtype, IC * k * k, "patch %s %s" % (shape, dtype))
        assert np.all(to_f64(around[:16 + shift]) == 7.0) and np.all(to_f64(around[16 + shift + size:]) == 7.0)
