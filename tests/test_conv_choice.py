"""The tile configuration that a convolution gets when it names none, as the size-based rule settles it on the host."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import build


def chosen(Nb, IC, H, W, OC, k, s, pad, packed=False, dtype=hb.HIDET_F16):
    """(rows, columns, K tile, matrix-core shape, schedule) of the tile."""
    c = hb.hidet_conv2d_untuned_config(dtype, (Nb, IC, H, W), (OC, IC, k, k), (s, s), (pad, pad), packed)
    i = hb.hidet_config_info(c)
    return i["block_m"], i["block_n"], i["block_k"], i["mfma"], i["schedule"]


@pytest.mark.parametrize("Nb,IC,H,OC,s", [(8, 16, 112, 24, 2), (2, 3, 224, 32, 2), (2, 3, 112, 24, 1), (8, 256, 112, 32, 2)])
def test_few_channels_and_many_columns_do_not_take_the_single_wavefront(Nb, IC, H, OC, s):
    """392 tiles of 64 columns: not enough for 64-column tiles of 32 rows, so it is the 32x32 tile of four wavefronts."""
    bm, bn, bk, mfma, schedule = chosen(Nb, IC, H, H, OC, 3, s, 1)
    assert (bm, bn, mfma) == (32, 32, 16)


def test_half_padded_tiles_split_a_long_k_in_one_round():
    """72 and 80 channels leave a 64x64 tile less than three quarters full; one round of them is still the best there is."""
    for case in ((36, 512, 13, 13, 80, 3, 1, 1), (7, 512, 56, 56, 80, 5, 2, 2), (2, 128, 56, 56, 72, 5, 1, 2)):
        assert chosen(*case)[:2] == (64, 64) and chosen(*case)[4] == 3, case


def test_32_channels_on_a_long_k_are_no_half_of_64():
    """A 64x64 K-splitting tile half of whose rows are padding is no tile for 32 channels: 32x32, two to a compute unit."""
    for case in ((28, 256, 35, 35, 32, 5, 2, 2), (4, 256, 45, 45, 32, 3, 1, 1), (12, 128, 28, 28, 32, 5, 1, 2),
                 (24, 256, 45, 45, 32, 3, 2, 1), (18, 256, 28, 28, 24, 3, 1, 1), (62, 192, 56, 56, 32, 3, 4, 1)):
        assert chosen(*case) == (32, 32, 256, 16, 3), case


def test_half_padded_128x64_tiles_on_a_long_k():
    """129 to 192 channels fill two rows of 128x64 tiles at least half: one round of them, K split, from K = 1408 on."""
    for case in ((35, 256, 14, 14, 144, 7, 1, 3), (32, 384, 14, 14, 160, 5, 1, 2), (17, 192, 35, 35, 160, 5, 2, 2),
                 (31, 192, 14, 14, 192, 3, 1, 1), (30, 160, 15, 15, 144, 3, 1, 1), (48, 256, 28, 28, 72, 3, 2, 1)):
        assert chosen(*case)[:2] == (128, 64) and chosen(*case)[4] == 3, case
    for case in ((30, 128, 15, 15, 144, 3, 1, 1), (16, 160, 28, 28, 64, 3, 1, 1)):  # K = 1152; 64 channels are no more than half
        assert chosen(*case)[:2] != (128, 64), case


def test_small_k_splitting_tiles_a_little_beyond_one_round():
    """Two workgroups of a small K-splitting tile are resident together: 301 of them are no second round."""
    for case in ((43, 512, 28, 28, 24, 3, 2, 1), (23, 256, 17, 17, 24, 7, 1, 3), (39, 384, 28, 28, 8, 5, 2, 2)):
        assert chosen(*case)[0] * chosen(*case)[1] <= 32 * 32 and chosen(*case)[4] == 3, case
    assert chosen(64, 64, 56, 56, 64, 3, 1, 1)[4] != 3  # (a throughput problem)


def test_at_most_64_channels_take_more_stages_while_all_tiles_are_resident():
    """A compute unit holds three of the 64x64 tiles with three stages: the gather of a long K is hidden better by them."""
    for case, stages in (((54, 96, 56, 56, 48, 5, 2, 2), 3), ((40, 192, 56, 56, 64, 5, 2, 2), 3), ((34, 64, 56, 56, 64, 3, 2, 1), 3),
                         ((9, 64, 55, 55, 64, 3, 1, 1), 3), ((48, 256, 64, 64, 64, 3, 2, 1), 3), ((49, 256, 64, 64, 64, 3, 2, 1), 2),
                         ((16, 64, 32, 64, 64, 3, 1, 1), 3), ((1, 64, 65, 512, 64, 3, 1, 1), 2), ((34, 48, 56, 56, 64, 3, 2, 1), 2)):
        assert chosen(*case)[:4] == ((64, 64, 64, 16) if stages == 3 else (64, 64, 64, 32)), case
        assert chosen(*case)[4] == (2 if stages == 3 else 0), case


def test_more_than_64_channels_do_not_take_flat_tiles():
    """Every row of tiles gathers the same columns again: three rows of 32x64 tiles against two of 64x32."""
    for case in ((7, 192, 28, 28, 72, 3, 1, 1), (2, 32, 56, 56, 96, 7, 1, 3), (9, 160, 20, 20, 160, 3, 1, 1)):
        assert chosen(*case)[:2] == (64, 32), case


def test_strides_above_2_take_k_splitting_tiles():
    """Gathered element by element: half padded, from K = 768 on, 64x32 (32x32) of them up to one and a half rounds."""
    for case, tile in (((40, 192, 14, 15, 512, 3, 3, 1), (64, 64)), ((5, 160, 56, 56, 512, 3, 4, 1), (64, 32)),
                       ((51, 160, 28, 28, 320, 3, 4, 1), (64, 64)), ((17, 48, 56, 56, 192, 5, 3, 2), (128, 64)),
                       ((19, 192, 35, 35, 192, 3, 3, 1), (64, 32)), ((44, 64, 56, 56, 32, 5, 5, 2), (32, 32))):
        assert chosen(*case)[:2] == tile and chosen(*case)[4] == 3, case
    for case in ((37, 128, 56, 56, 192, 3, 4, 1), (44, 128, 35, 35, 192, 5, 3, 2)):  # 128x128 would be a quarter padding
        assert chosen(*case)[:2] != (128, 128), case
    assert chosen(41, 256, 56, 56, 320, 3, 4, 1)[:2] == (128, 128)
    assert chosen(57, 85, 35, 35, 128, 3, 4, 1)[4] != 3  # K = 765, 129 tiles of 128x64: too short for half a round of them


def test_untuned_config_arguments():
    f = lambda *a: hb.lib().hidet_conv2d_untuned_config(*a, ctypes.byref(c))
    c = ctypes.c_int32(7)
    assert f(hb.HIDET_F16, 0, 8, 4, 4, 8, 1, 1, 1, 1, 0, 0, 0) == 0 and c.value == -1  # empty
    assert f(9, 1, 8, 4, 4, 8, 1, 1, 1, 1, 0, 0, 0) == 1 and f(hb.HIDET_F16, 1, 8, 4, 4, 8, 0, 1, 1, 1, 0, 0, 0) == 1
    assert f(hb.HIDET_F16, 1, 7, 14, 14, 8, 3, 3, 1, 1, 1, 1, 1) == 2  # repacked weights need whole chunks of channels
    assert hb.lib().hidet_conv2d_untuned_config(hb.HIDET_F16, 1, 8, 4, 4, 8, 1, 1, 1, 1, 0, 0, 0, None) == 1


@pytest.mark.parametrize("tile", ["96, 64", "64, 192"])
def test_tile_extents_that_are_no_power_of_two_do_not_compile(tmp_path, tile):
    """The choice counts tiles with shifts: a table with another extent has to fail to compile, not to miscount."""
    csrc = tmp_path / "package" / "csrc"
    shutil.copytree(build.CSRC, csrc)
    shutil.copytree(os.path.join(build.HERE, "..", "include"), tmp_path / "include")
    table = (csrc / "configs.def").read_text()
    assert "X16(5, 128, 64," in table

    def compiles():
        cmd = [build.HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-fsyntax-only", str(csrc / "api.hip")]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        return r.returncode == 0, r.stdout

    ok, log = compiles()
    assert ok, log
    (csrc / "configs.def").write_text(table.replace("X16(5, 128, 64,", "X16(5, %s," % tile))
    ok, log = compiles()
    assert not ok and "tile_extents_are_powers_of_two" in log, log
