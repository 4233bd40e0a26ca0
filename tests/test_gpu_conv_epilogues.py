"""The epilogues of the convolution forms that have their own (3x3 and 5x5 from a patch of the input, 1x1 over all images): every
combination of scale, bias, residual and ReLU, a residual that is the output itself, on rows of every alignment; and infinities
and NaN beside the borders of the input."""
import numpy as np
import pytest
import torch

import oracle
from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TORCH_DTYPE, assert_elementwise, conv_scale, to_f64, to_gpu

PATCHES = (hb.HIDET_CONV_PATCH_64, hb.HIDET_CONV_PATCH_128)
# images, input channels, height, width, output channels, filter, forms
SHAPES = [(64, 32, 14, 14, 80, 3, PATCHES), (70, 32, 14, 15, 200, 3, PATCHES), (60, 16, 14, 13, 66, 5, PATCHES),
          (300, 64, 7, 7, 136, 1, (hb.HIDET_CONV_IMAGES,)), (240, 200, 8, 8, 260, 1, (hb.HIDET_CONV_IMAGES,))]


def test_the_forms_under_test():
    for Nb, IC, H, W, OC, k, forms in SHAPES:
        assert hb.hidet_conv2d_untuned_form(hb.HIDET_F16, (Nb, IC, H, W), (OC, IC, k, k), pad=(k // 2,) * 2) in forms


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_epilogue(shape, dtype):
    Nb, IC, H, W, OC, k, _ = shape
    pad = (k // 2,) * 2
    c = wl.conv_case(9950 + Nb, Nb, IC, H, W, OC, k, k, 1, k // 2, dtype, residual=True)
    x, w, bias, res = (to_gpu(c[n], dtype) for n in ("x", "w", "bias", "residual"))
    x64, w64, b64, r64 = (wl.widen(c[n], dtype) for n in ("x", "w", "bias", "residual"))
    product = oracle.conv2d(x64, w64, pad=pad)
    for alpha, with_bias, residual, relu in [(1.0, 0, None, 0), (-0.75, 0, None, 1), (1.0, 1, None, 0), (1.0, 0, "other", 1),
                                             (0.5, 1, "other", 0), (1.0, 1, "in place", 1), (2.0, 0, "in place", 0)]:
        y = torch.full(res.shape, float("nan"), dtype=TORCH_DTYPE[dtype], device="cuda")
        if residual == "in place":
            y.copy_(res)
        epi = hb.make_epilogue(alpha=alpha, bias=bias if with_bias else None, bias_axis=hb.HIDET_BIAS_PER_ROW if with_bias else 0,
                               residual=None if residual is None else y if residual == "in place" else res, relu=bool(relu))
        hb.hidet_conv2d_implicit_gemm(x, w, y, pad=pad, epilogue=None if (alpha, with_bias, residual, relu) == (1.0, 0, None, 0) else epi)
        torch.cuda.synchronize()
        bb, rr = b64 if with_bias else None, r64 if residual else None
        ref = alpha * product + (0.0 if bb is None else bb[None, :, None, None]) + (0.0 if rr is None else rr)
        ref = np.maximum(ref, 0.0) if relu else ref
        assert_elementwise(to_f64(y), ref, conv_scale(x64, w64, (1, 1), pad, alpha, bb, rr), dtype, IC * k * k,
                           "%s alpha %g bias %d residual %s relu %d" % (shape, alpha, with_bias, residual, relu))


@pytest.mark.gpu
@pytest.mark.parametrize("k", [3, 5])
def test_infinities_and_nan_beside_the_borders_of_a_patch(k):
    """A value reaches exactly the outputs whose filter covers it: not the other end of the next row, not the next image."""
    Nb, IC, H, W, OC = 64, 32, 14, 14, 64
    pad = (k // 2,) * 2
    assert hb.hidet_conv2d_untuned_form(hb.HIDET_F16, (Nb, IC, H, W), (OC, IC, k, k), pad=pad) in PATCHES
    x = torch.ones((Nb, IC, H, W), dtype=torch.float16, device="cuda")
    marks = torch.zeros((Nb, 1, H, W), device="cuda")
    for img, ch, r, q, v in [(0, 0, 0, 0, float("inf")), (0, 31, 13, 13, float("nan")), (1, 8, 0, 13, float("inf")), (2, 7, 13, 0, float("nan")),
                             (5, 15, 6, 13, float("inf")), (6, 16, 7, 0, float("nan")), (63, 31, 13, 13, float("inf")), (63, 0, 0, 0, float("nan"))]:
        x[img, ch, r, q] = v
        marks[img, 0, r, q] = 1.0
    w = torch.full((OC, IC, k, k), 2.0 ** -6, dtype=torch.float16, device="cuda")
    y = torch.empty((Nb, OC, H, W), dtype=torch.float16, device="cuda")
    hb.hidet_conv2d_implicit_gemm(x, w, y, pad=pad)
    torch.cuda.synchronize()
    reached = torch.nn.functional.max_pool2d(marks.cpu(), k, stride=1, padding=k // 2).expand(Nb, OC, H, W) > 0
    count = torch.nn.functional.avg_pool2d(torch.ones((1, 1, H, W)), k, stride=1, padding=k // 2, divisor_override=1)
    got = y.cpu().float()
    assert torch.equal(~torch.isfinite(got), reached)
    assert torch.equal(got[~reached], (count * IC * 2.0 ** -6).expand(Nb, OC, H, W)[~reached])  # (exact in fp16)
