"""Convolutions that name no configuration, at the edges of the rule that chooses one (whole rounds of K-splitting
workgroups on a long K, few output channels), against the CPU oracle within the derived bound."""
import pytest

from paper_2210_09603_amd import workloads as wl

from helpers import run_conv_case, within_bound

pytestmark = pytest.mark.gpu

# images, input channels, height, width, output channels, filter, stride, padding
SHAPES = {
    "256 tiles of 16x16, K 513": (2, 57, 64, 16, 32, 3, 1, 1),
    "260 tiles of 16x16": (2, 64, 65, 16, 32, 3, 1, 1),
    "K 504, below the rule": (1, 56, 8, 8, 256, 3, 1, 1),
    "K 576, 64 rows": (1, 64, 64, 63, 64, 3, 1, 1),
    "K 576, 65 rows": (1, 64, 64, 64, 65, 3, 1, 1),
    "few rows, many columns": (1, 32, 160, 160, 48, 3, 1, 1),
    "K 2088": (1, 232, 32, 32, 128, 3, 1, 1),
    "large tiles in one round": (4, 128, 56, 57, 96, 3, 1, 1),
    "one output pixel": (1, 64, 3, 3, 40, 3, 1, 0),
    "strided": (3, 64, 31, 29, 72, 5, 2, 2),
}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_conv_of_unnamed_configuration(shape, dtype):
    Nb, IC, H, W, OC, k, s, pad = SHAPES[shape]
    c = wl.conv_case(9100 + list(SHAPES).index(shape), Nb, IC, H, W, OC, k, k, s, pad, dtype, residual=True)
    for packed in ([False, True] if IC % 64 == 0 else [False]):
        err, _, ref = run_conv_case(c, packed=packed)
        print("%s %s packed=%d err %.3e" % (shape, dtype, packed, err), flush=True)
        assert within_bound(err, ref, dtype)
