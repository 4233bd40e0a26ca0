"""Convolutions that name no configuration, at the edges of the rule that chooses one (whole rounds of K-splitting
workgroups on a long K, few output channels): the tile each edge is meant to reach, and its result against the CPU oracle
within the derived bound."""
import pytest

from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import run_conv_case, within_bound

pytestmark = pytest.mark.gpu

# images, input channels, height, width, output channels, filter, stride, padding: tile (rows, columns, K, matrix-core shape,
# schedule; 3 splits K over wave groups) from OIHW weights, and from repacked ones where the channels allow them
SHAPES = {
    "256 tiles of 16x16, K 513": ((2, 57, 64, 16, 32, 3, 1, 1), (16, 16, 512, 16, 3)),
    "260 tiles of 16x16 are 130 of 32x16": ((2, 64, 65, 16, 32, 3, 1, 1), (32, 16, 512, 16, 3), (32, 32, 64, 16, 2)),
    "K 504, below the rule": ((1, 56, 8, 8, 256, 3, 1, 1), (32, 32, 256, 16, 0)),
    "256 tiles of 32x32": ((1, 64, 64, 63, 64, 3, 1, 1), (32, 32, 256, 16, 3), (32, 32, 64, 16, 2)),
    "65 channels: 256 tiles of 64x32": ((1, 64, 64, 64, 65, 3, 1, 1), (64, 32, 256, 16, 3), (64, 32, 64, 16, 2)),
    "few channels, many columns": ((1, 32, 160, 160, 48, 3, 1, 1), (64, 64, 64, 32, 0)),
    "64 channels, K 504, many columns": ((1, 56, 160, 160, 64, 3, 1, 1), (64, 64, 64, 32, 0)),
    "65 channels, K 504, many columns": ((1, 56, 160, 160, 65, 3, 1, 1), (128, 64, 64, 32, 0)),
    "32 tiles across, K 2088": ((1, 232, 32, 32, 128, 3, 1, 1), (32, 16, 512, 16, 3)),
    "132 tiles of 64x64, K 2043": ((1, 227, 96, 88, 64, 3, 1, 1), (64, 32, 64, 16, 2)),
    "132 tiles of 64x64, K 2052": ((1, 228, 96, 88, 64, 3, 1, 1), (64, 64, 256, 16, 3)),
    "half-padded tiles, K 2052": ((1, 228, 48, 88, 80, 3, 1, 1), (64, 64, 256, 16, 3)),
    "288 small tiles, K 2304": ((2, 256, 64, 72, 24, 3, 1, 1), (32, 32, 256, 16, 3), (32, 32, 256, 16, 3)),
    "32 channels, 512 tiles of 32x32, K 2304": ((2, 256, 64, 128, 32, 3, 1, 1), (32, 32, 256, 16, 3), (32, 32, 256, 16, 3)),
    "32 channels, 544 tiles of 32x32, K 2304": ((2, 256, 64, 129, 32, 3, 1, 1), (32, 64, 64, 16, 2)),
    "64 channels, stride 2, 768 tiles of 64x64": ((6, 64, 128, 256, 64, 3, 2, 1), (64, 64, 64, 16, 2)),
    "64 channels, stride 2, 816 tiles of 64x64": ((6, 64, 128, 264, 64, 3, 2, 1), (64, 64, 64, 32, 0)),
    "half-padded 128x64 tiles, K 1440": ((30, 160, 15, 15, 144, 3, 1, 1), (128, 64, 128, 16, 3)),
    "half-padded 128x64 tiles, K 2304": ((12, 256, 28, 28, 72, 3, 1, 1), (128, 64, 128, 16, 3), (128, 64, 128, 16, 3)),
    "no flat tiles": ((7, 192, 28, 28, 72, 3, 1, 1), (64, 32, 64, 16, 2), (64, 32, 64, 16, 2)),
    "224 tiles of 128x64": ((4, 128, 56, 57, 96, 3, 1, 1), (128, 64, 128, 16, 3), (128, 64, 128, 16, 3)),
    "200 tiles of 128x128": ((1, 64, 128, 193, 128, 3, 1, 1), (128, 128, 64, 16, 3), (128, 128, 64, 16, 3)),
    "one output pixel": ((1, 64, 3, 3, 40, 3, 1, 0), (16, 16, 512, 16, 3), (32, 32, 64, 16, 2)),
    "strided": ((3, 64, 31, 29, 72, 5, 2, 2), (16, 16, 512, 16, 3), (32, 32, 64, 16, 2)),
    "stride 3, 193 tiles of 64x64, K 765": ((7, 85, 132, 118, 64, 3, 3, 1), (64, 32, 64, 16, 2)),
    "stride 3, 193 tiles of 64x64, K 774": ((7, 86, 132, 118, 64, 3, 3, 1), (64, 64, 256, 16, 3)),
    "stride 3, 384 tiles of 64x32": ((8, 64, 144, 96, 64, 3, 3, 1), (64, 32, 256, 16, 3)),
    "stride 3, 384 tiles of 32x32": ((8, 64, 144, 96, 32, 3, 3, 1), (32, 32, 256, 16, 3)),
    "stride 3, half-padded tiles": ((8, 64, 147, 96, 64, 3, 3, 1), (128, 64, 128, 16, 3)),
}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_conv_of_unnamed_configuration(shape, dtype):
    (Nb, IC, H, W, OC, k, s, pad), *tiles = SHAPES[shape]
    c = wl.conv_case(9100 + list(SHAPES).index(shape), Nb, IC, H, W, OC, k, k, s, pad, dtype, residual=True)
    for packed, tile in enumerate(tiles):
        i = hb.hidet_config_info(hb.hidet_conv2d_untuned_config({"f16": hb.HIDET_F16, "bf16": hb.HIDET_BF16}[dtype], (Nb, IC, H, W),
                                                                (OC, IC, k, k), (s, s), (pad, pad), bool(packed)))
        assert (i["block_m"], i["block_n"], i["block_k"], i["mfma"], i["schedule"]) == tile, packed
        err, _, ref = run_conv_case(c, packed=bool(packed))
        print("%s %s packed=%d err %.3e" % (shape, dtype, packed, err), flush=True)
        assert within_bound(err, ref, dtype)
