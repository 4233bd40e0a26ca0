"""Convolutions that have a form of their own beside the gather, after a tuning file has been loaded: an entry that cannot serve
the call leaves it as it is without one."""
import pytest
import torch

from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TORCH_DTYPE, run_conv_case, to_gpu, within_bound

pytestmark = pytest.mark.gpu

# images, input channels, height, width, output channels, filter: from a patch, over all images, as a batched GEMM
PATCH, IMAGES, BATCHED = (64, 32, 14, 14, 80, 3), (300, 64, 7, 7, 136, 1), (4, 128, 28, 28, 64, 1)


@pytest.fixture(autouse=True)
def nothing_remembered():
    hb.hidet_tune_clear()
    yield
    hb.hidet_tune_clear()


def case(shape, dtype="f16"):
    Nb, IC, H, W, OC, k = shape
    c = wl.conv_case(9900 + Nb, Nb, IC, H, W, OC, k, k, 1, k // 2, dtype, residual=True)
    c["relu"] = True
    return c


def key(c, dtype="f16"):
    Nb, IC, H, W = c["x"].shape
    OC, _, KH, KW = c["w"].shape
    return "conv:t%d:n%d:c%d:%dx%d:o%d:k%dx%d:s1x1:p%dx%d:e%d:m0" % ({"f16": 1, "bf16": 2}[dtype], Nb, IC, H, W, OC, KH, KW, KH // 2,
                                                                  KW // 2, 2 | 4 | 8)


@pytest.mark.parametrize("shape", [PATCH, IMAGES, BATCHED])
def test_entries_that_cannot_serve_the_call(shape, tmp_path):
    c = case(shape)
    err, plain, ref = run_conv_case(c)
    assert within_bound(err, ref, "f16")
    f32 = next(i for i in range(hb.hidet_config_count()) if hb.hidet_config_info(i)["is_f32"])
    for entry in ("%d 1 0" % f32, "%d 1 1" % f32):
        path = tmp_path / "tuned.txt"
        path.write_text("%s %s\n" % (key(c), entry))
        hb.hidet_tune_clear()
        hb.hidet_tune_load(str(path))
        _, got, _ = run_conv_case(c)
        assert (got == plain).all(), entry
    # the batched-GEMM form of a convolution that has none: the configuration is that of the gather
    if shape == PATCH:
        path.write_text("%s 7 1 1\n" % key(c))
        hb.hidet_tune_clear()
        hb.hidet_tune_load(str(path))
        _, got, _ = run_conv_case(c)
        _, gather, _ = run_conv_case(c, config=7)
        assert (got == gather).all()
