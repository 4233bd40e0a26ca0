"""The tile configuration that a GEMM gets when it names none, as the size-based rule settles it on the host."""
import ctypes

import pytest

from paper_2210_09603_amd import binding as hb


def chosen(M, N, K, batch=1, tA=False, tB=False, dtype=hb.HIDET_F16):
    """(rows, columns, K tile, schedule) of the tile."""
    i = hb.hidet_config_info(hb.hidet_gemm_untuned_config(dtype, M, N, K, batch, tA, tB))
    return i["block_m"], i["block_n"], i["block_k"], i["schedule"]


@pytest.mark.parametrize("tA", [False, True])
@pytest.mark.parametrize("dtype", [hb.HIDET_F16, hb.HIDET_BF16])
def test_one_round_of_the_smallest_streaming_tile(dtype, tA):
    for problem, tile in (((8, 3072, 768), (16, 16)), ((8, 3088, 768), (16, 32)), ((8, 8192, 1024), (16, 32)), ((8, 8208, 1024), (64, 64)),
                          ((128, 768, 3072), (16, 32)), ((300, 768, 3072), (32, 32)), ((512, 512, 512), (32, 32)),
                          ((700, 1024, 4096), (64, 64)), ((1024, 1024, 1024), (64, 64)), ((640, 768, 3072), (64, 32))):
        assert chosen(*problem, tA=tA, dtype=dtype)[:2] == tile, problem
        assert chosen(*problem, tA=tA, dtype=dtype)[3] == 3, problem


def test_streaming_tiles_need_a_k_that_their_wavefronts_share():
    """Below it, two-stage tiles: the deep one of two to a compute unit on aligned rows, else 64 values of k at a time."""
    for problem, streams in (((96, 96, 264), True), ((96, 96, 256), False), ((97, 95, 128), True), ((97, 95, 127), False),
                             ((97, 1001, 160), True), ((97, 1001, 159), False), ((97, 2001, 257), True), ((97, 2001, 256), False), ((96, 2688, 264), True), ((96, 2688, 256), False),
                             ((640, 768, 448), True), ((640, 768, 440), False), ((960, 960, 512), True), ((960, 960, 504), False)):
        assert (chosen(*problem)[3] == 3) == streams, problem
    assert chosen(96, 96, 256) == (32, 32, 256, 0) and chosen(96, 96, 128) == (32, 32, 64, 0)
    assert chosen(97, 95, 127) == (32, 32, 64, 0)
    assert chosen(512, 1024, 256) == (32, 32, 256, 0) and chosen(544, 1024, 256) == (32, 32, 64, 0)


def test_between_few_tiles_and_throughput_tiles_of_half_64x64():
    assert chosen(768, 1024, 256) == (32, 32, 64, 0)  # three of 32x32 to a compute unit
    assert chosen(800, 1024, 256) == (32, 64, 64, 2) and chosen(1024, 800, 256) == (64, 32, 64, 2)
    assert chosen(320, 4096, 1024) == (64, 32, 64, 2)
    assert chosen(800, 1024, 256, tA=True) == (32, 32, 64, 0)  # built for a transposed A
    assert chosen(1536, 1024, 256)[:2] != (64, 32)  # 384 tiles of 64x64


def test_batches_count_all_their_tiles_and_take_no_large_tile_that_is_padding():
    assert chosen(128, 64, 512, batch=12) == (16, 32, 512, 3)
    assert chosen(128, 128, 64, batch=12, tB=True) == (32, 32, 64, 0)
    for problem, batch in (((400, 64, 400), 88), ((374, 64, 374), 128), ((398, 398, 128), 65), ((384, 384, 128), 174), ((448, 448, 128), 84)):
        bm, bn = chosen(*problem, batch=batch)[:2]
        M, N, _ = problem
        assert bm * bn < 128 * 128 or 4 * M * N > 3 * (-(-M // bm) * bm) * (-(-N // bn) * bn), problem
    for problem, batch in (((320, 320, 32), 96), ((448, 448, 64), 43)):
        assert chosen(*problem, batch=batch, tB=True)[:2] == (64, 64), problem
    assert chosen(143, 143, 128, batch=72, tB=True) == (32, 32, 64, 2)
    assert chosen(512, 512, 64, batch=192, tB=True) == (256, 128, 32, 1) and chosen(512, 64, 512, batch=192)[:2] == (128, 64)


def test_large_products_keep_the_ring():
    for problem, tile in (((4096, 4096, 4096), (256, 256)), ((4096, 3072, 768), (256, 256)), ((4096, 768, 3072), (128, 128)),
                          ((2039, 2039, 2039), (128, 128))):
        assert chosen(*problem)[:2] == tile and chosen(*problem)[3] == 1, problem


def test_rectangular_ring_tiles_lie_along_a_row_major_b():
    """128 rows of A are half as many short pieces as 256; not where B is read along K as well."""
    for problem in ((2639, 2104, 3735), (1488, 3408, 3240), (2992, 1896, 3816)):
        assert chosen(*problem)[:2] == (128, 256) and chosen(*problem, tB=True)[:2] == (256, 128), problem
    assert chosen(8192, 8192, 64)[:2] == (256, 128)  # two stages of K: two workgroups of it to a compute unit


def test_fp32_is_not_concerned():
    assert chosen(256, 256, 256, dtype=hb.HIDET_F32) == (16, 16, 256, 3)


def test_fp32_products_with_few_tiles_take_the_shortest_predicted_time():
    """K split where a tile of its own pays for it, also of a transposed A; two stages on a short K; 384 tiles of 64x64 as before."""
    for problem, tile in (((854, 27, 203), (16, 16, 256, 3)), ((224, 281, 190), (16, 16, 256, 3)), ((128, 1136, 1029), (32, 32, 128, 3)),
                          ((144, 672, 29), (32, 32, 32, 0)), ((128, 90, 16), (32, 32, 32, 0))):
        assert chosen(*problem, dtype=hb.HIDET_F32) == tile, problem
    assert chosen(16, 40, 1000, dtype=hb.HIDET_F32, tA=True) == (16, 16, 256, 3)
    assert chosen(1536, 1024, 256, dtype=hb.HIDET_F32)[3] != 3 and chosen(32, 32, 400, batch=400, dtype=hb.HIDET_F32)[3] != 3


def test_arguments():
    c = ctypes.c_int32(7)
    f = lambda *a: hb.lib().hidet_gemm_untuned_config(*a, ctypes.byref(c))
    assert f(hb.HIDET_F16, 0, 0, 1, 0, 8, 8) == 0 and c.value == -1  # empty
    assert f(9, 0, 0, 1, 8, 8, 8) == 1 and f(hb.HIDET_F16, 0, 0, 1, -1, 8, 8) == 1
    assert hb.lib().hidet_gemm_untuned_config(hb.HIDET_F16, 0, 0, 1, 8, 8, 8, None) == 1


def test_batches_on_tiles_that_carry_them():
    """Two wavefronts of 16x64 need as long as the four of 32x64, whatever share of the tile is output; a half-filled large tile
    beats full small ones on a long K and, on element-aligned rows, at 128x128."""
    assert chosen(48, 196, 1024, batch=96)[:2] != (16, 64)
    assert chosen(48, 169, 64, batch=148)[:2] != (16, 64)
    assert chosen(10, 358, 36, batch=94, dtype=hb.HIDET_BF16)[:2] != (16, 64)
    assert chosen(16, 1600, 256, batch=40)[:2] == (16, 64)  # aligned, no row of it padding
    assert chosen(96, 729, 512, batch=78)[:2] == (128, 256)
    assert chosen(88, 511, 42, batch=111)[:2] == (128, 128)
