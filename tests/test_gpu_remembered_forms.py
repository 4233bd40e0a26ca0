"""Convolutions that have a form of their own beside the gather, after tuning and after a tuning file has been loaded: the
tuner remembers the fastest form, a remembered form runs wherever it can, beyond the sizes for which it is chosen untuned, and an
entry that cannot serve the call leaves it as it is without one."""
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


def remember(c, entry, tmp_path, dtype="f16"):
    path = tmp_path / "tuned.txt"
    path.write_text("%s %s\n" % (key(c, dtype), entry))
    hb.hidet_tune_clear()
    hb.hidet_tune_load(str(path))


# (the rest of the layers of the schedule choice are within a few per cent of each other; these are not)
@pytest.mark.parametrize("shape,dtype,forms", [((64, 256, 14, 14, 256, 3), "bf16", (hb.HIDET_CONV_PATCH_64, hb.HIDET_CONV_PATCH_128)),
                                               ((64, 512, 7, 7, 2048, 1), "f16", (hb.HIDET_CONV_IMAGES,)),
                                               ((1, 256, 14, 14, 256, 3), "f16", (hb.HIDET_CONV_GATHER,))])
def test_the_tuner_remembers_the_fastest_form(shape, dtype, forms, tmp_path):
    c = case(shape, dtype)
    x, w, bias, res = (to_gpu(c[k], dtype) for k in ("x", "w", "bias", "residual"))
    y = torch.full(c["residual"].shape, float("nan"), dtype=TORCH_DTYPE[dtype], device="cuda")
    epi = hb.make_epilogue(bias=bias, bias_axis=hb.HIDET_BIAS_PER_ROW, residual=res, relu=True)
    pad = (shape[5] // 2,) * 2
    for workspace in (None, torch.empty(1 << 22, dtype=torch.float32, device="cuda")):
        hb.hidet_tune_clear()
        if workspace is None:
            cfg, us = hb.hidet_tune_conv2d(x, w, y, pad=pad, epilogue=epi, iters=20)
        else:
            cfg, _, us = hb.hidet_tune_conv2d_splitk(x, w, y, workspace, pad=pad, epilogue=epi, iters=20)
        assert 0 <= cfg < hb.hidet_config_count() and us > 0
        tuned = y.clone()
        path = str(tmp_path / "tuned.txt")
        hb.hidet_tune_save(path)
        entry = [line.split() for line in open(path) if line.startswith(key(c, dtype))]
        assert len(entry) == 1 and entry[0][0] == key(c, dtype) + (":ws" if workspace is not None else "")
        assert int(entry[0][1]) == cfg and int(entry[0][3]) in forms
        hb.hidet_tune_clear()
        hb.hidet_tune_load(path)
        y.fill_(float("nan"))
        if workspace is None:
            hb.hidet_conv2d_implicit_gemm(x, w, y, pad=pad, epilogue=epi)
        else:
            hb.hidet_conv2d_implicit_gemm_splitk(x, w, y, workspace, k_slices=0, pad=pad, epilogue=epi)
        torch.cuda.synchronize()
        assert torch.equal(y, tuned)
        err, _, ref = run_conv_case(c, k_slices=3)  # (a remembered form without K slices: another one takes the call)
        assert within_bound(err, ref, dtype)


# one image, one channel, the shortest rows and planes: far from the sizes for which the forms are chosen
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [(1, 16, 1, 8, 1, 3), (2, 16, 8, 1, 3, 3), (1, 32, 3, 3, 70, 3), (3, 16, 2, 62, 15, 3), (1, 48, 40, 5, 200, 3),
                                   (1, 16, 1, 8, 1, 5), (2, 32, 8, 1, 3, 5), (5, 16, 3, 4, 65, 5), (1, 48, 2, 29, 15, 5)])
def test_patch_forms_beyond_the_choice(shape, dtype, tmp_path):
    c = case(shape, dtype)
    for form in (hb.HIDET_CONV_PATCH_64, hb.HIDET_CONV_PATCH_128):
        remember(c, "7 1 %d" % form, tmp_path, dtype)
        err, got, ref = run_conv_case(c)
        assert within_bound(err, ref, dtype), (form, err)
    if shape[5] == 5:  # (128 rows are not built for 5x5: the configuration of the gather that stands beside the form)
        _, gather, _ = run_conv_case(c, config=7)
        assert (got == gather).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [(1, 8, 1, 8, 1, 1), (1, 40, 3, 3, 3, 1), (2, 72, 5, 13, 129, 1), (17, 8, 3, 5, 64, 1), (1, 264, 40, 40, 130, 1)])
def test_the_product_over_all_images_beyond_the_choice(shape, dtype, tmp_path):
    c = case(shape, dtype)
    ring = [i for i in range(hb.hidet_config_count()) if hb.hidet_config_info(i)["schedule"] == 1
            and hb.hidet_config_info(i)["block_m"] == hb.hidet_config_info(i)["block_n"] == 128]
    _, plain, _ = run_conv_case(c)
    for cfg in ring + [7]:
        remember(c, "%d 1 %d" % (cfg, hb.HIDET_CONV_IMAGES), tmp_path, dtype)
        err, got, ref = run_conv_case(c)
        assert within_bound(err, ref, dtype), (cfg, err)
        assert cfg in ring or (got == plain).all()  # (no tile of that form)


def test_forms_that_the_convolution_does_not_have(tmp_path):
    for shape, form in ((PATCH, hb.HIDET_CONV_IMAGES), (BATCHED, hb.HIDET_CONV_PATCH_64), (IMAGES, hb.HIDET_CONV_PATCH_128),
                        ((64, 24, 14, 14, 80, 3), hb.HIDET_CONV_PATCH_64), ((8, 16, 14, 63, 80, 3), hb.HIDET_CONV_PATCH_64),
                        ((64, 12, 7, 7, 40, 1), hb.HIDET_CONV_IMAGES), ((64, 16, 2, 3, 40, 1), hb.HIDET_CONV_IMAGES)):
        c = case(shape)
        remember(c, "7 1 %d" % form, tmp_path)
        err, _, ref = run_conv_case(c)
        assert within_bound(err, ref, "f16"), (shape, form, err)
