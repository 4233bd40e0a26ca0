"""The K-splitting tiles up to 64x64 in 16-bit types, whose wavefronts stream K steps of their own: every count of steps
around a wavefront's ring, ragged edges, transposes, alignments and options, against the CPU oracle within the derived
bounds."""
import numpy as np
import pytest
import torch

import oracle
from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TORCH_DTYPE, applicable_configs, assert_elementwise, gemm_scale, run_gemm_case, to_f64, to_gpu, within_bound

pytestmark = pytest.mark.gpu


def streaming():
    out = []
    for c in applicable_configs("f16"):
        i = hb.hidet_config_info(c)
        if i["schedule"] == 3 and i["block_m"] <= 64 and i["block_n"] <= 64:
            out.append((c, i["block_m"], i["block_n"]))
    return out


def ring(bm, bn):
    """K of one step, and steps of a wavefront's ring: eight wavefronts share 144 KB."""
    step = 32 if bm * bn > 32 * 32 else 64
    return step, min(4, 144 * 1024 // (8 * (bm + bn) * step * 2))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tA,tB", [(False, False), (False, True), (True, False), (True, True)])
def test_every_count_of_steps(dtype, tA, tB):
    """No whole step, one, one for all wavefronts but one, one for each, a ring filled and wrapped; each with the last step
    whole, ragged at 8 and ragged at one element, on aligned and on element-aligned rows."""
    ran = 0
    for cfg, bm, bn in streaming():
        step, depth = ring(bm, bn)
        for steps in (0, 1, 7, 8, 8 * depth, 8 * depth + 9):
            for tail in (0, 8, step - 1):
                K = steps * step + tail
                if K == 0:
                    continue
                odd = tail % 8 != 0 or (steps + bm) % 3 == 0
                M, N = (2 * bm + 3, bn + 9) if odd else (bm + 8, 2 * bn + 8)
                c = wl.gemm_case(9500 + cfg, M, N, K, dtype, transA=tA, transB=tB, bias="col" if steps % 2 else "row",
                                 residual=steps % 3 != 1)
                err, _, ref = run_gemm_case(c, config=cfg, relu=True, alpha=0.5)
                assert within_bound(err, ref, dtype), (cfg, steps, tail, err)
                ran += 1
    assert ran >= 6 * 16


def test_tiles_are_built_for_every_operand_form():
    assert [(bm, bn) for _, bm, bn in streaming()] == [(32, 32), (64, 32), (16, 32), (16, 16), (32, 16), (64, 64)]


@pytest.mark.parametrize("M,N,K", [(1, 1, 640), (3, 2, 517), (5, 8, 513), (300, 7, 520), (16, 16, 64)])
def test_operands_narrower_than_one_access(M, N, K):
    """Rows shorter than 16 bytes: a direct load would reach past the row that follows."""
    for cfg, _, _ in streaming():
        for tA in (False, True):
            c = wl.gemm_case(9600 + cfg, M, N, K, "f16", transA=tA, bias="col")
            err, _, ref = run_gemm_case(c, config=cfg)
            assert within_bound(err, ref, "f16"), (cfg, tA, err)


def test_offset_pointers_and_padded_rows_stay_inside_the_output():
    """Element alignment from the pointers alone; what lies around the output is untouched."""
    for cfg, bm, bn in streaming():
        M, N, K = bm + 5, bn + 6, 1160
        c = wl.gemm_case(9700 + cfg, M, N, K, "bf16", bias="col", lda_pad=16, ldb_pad=24)
        A = torch.empty(M * c["lda"] + 1, dtype=torch.bfloat16, device="cuda")[1:].view(M, c["lda"])
        B = torch.empty(K * c["ldb"] + 1, dtype=torch.bfloat16, device="cuda")[1:].view(K, c["ldb"])
        A.copy_(to_gpu(c["A"], "bf16"))
        B.copy_(to_gpu(c["B"], "bf16"))
        whole = torch.full((M, N + 7), float("nan"), dtype=torch.bfloat16, device="cuda")
        bias = to_gpu(c["bias"], "bf16")
        hb.hidet_gemm(A[:, :K], B[:, :N], whole[:, :N], epilogue=hb.make_epilogue(bias=bias, bias_axis=hb.HIDET_BIAS_PER_COL),
                      config=cfg)
        torch.cuda.synchronize()
        A64, B64, b64 = wl.widen(c["A"], "bf16")[:, :K], wl.widen(c["B"], "bf16")[:, :N], wl.widen(c["bias"], "bf16")
        ref = oracle.gemm(A64, B64, bias=b64, bias_axis=oracle.BIAS_PER_COL)
        assert_elementwise(to_f64(whole[:, :N]), ref, gemm_scale(A64, B64, False, False, 1.0, b64, "col"), "bf16", K)
        assert torch.isnan(whole[:, N:]).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_batches_wide_output_input_relu_head_split_and_k_slices(dtype):
    b, M, N, K = 3, 48, 72, 1096
    for cfg, _, _ in streaming():
        c = wl.gemm_case(9800 + cfg, M * b, N, K, dtype)
        A, B = to_gpu(c["A"], dtype).view(b, M, K), to_gpu(c["B"], dtype)
        A64, B64 = wl.widen(c["A"], dtype), wl.widen(c["B"], dtype)
        # one right operand for the whole batch, fp32 results, ReLU on the left operand as it is loaded
        C = torch.full((b, M, N), float("nan"), dtype=torch.float32, device="cuda")
        hb.hidet_batched_gemm(A, B.expand(b, K, N), C, epilogue=hb.make_epilogue(relu_input=True), config=cfg)
        H = torch.full((b, 9, M, 8), float("nan"), dtype=TORCH_DTYPE[dtype], device="cuda")
        hb.hidet_gemm(A.reshape(b * M, K), B, H, epilogue=hb.make_epilogue(head_split=(M, 8)), config=cfg)
        S = torch.full((b * M, N), float("nan"), dtype=TORCH_DTYPE[dtype], device="cuda")
        ws = torch.full((3 * b * M * N,), float("nan"), dtype=torch.float32, device="cuda")
        hb.hidet_batched_gemm_splitk(A.reshape(b * M, K), B, S, ws, k_slices=3, config=cfg)
        torch.cuda.synchronize()
        pos = np.maximum(A64, 0.0)
        assert_elementwise(to_f64(C).reshape(b * M, N), oracle.gemm(pos, B64), gemm_scale(pos, B64, False, False, 1.0), "f32", K)
        ref, scale = oracle.gemm(A64, B64), gemm_scale(A64, B64, False, False, 1.0)
        assert_elementwise(to_f64(H).transpose(0, 2, 1, 3).reshape(b * M, N), ref, scale, dtype, K)
        assert_elementwise(to_f64(S), ref, scale, dtype, K)


def test_infinities_beyond_k_do_not_reach_the_result():
    """The last step reads no value beyond K, on aligned and element-aligned rows."""
    for cfg, _, _ in streaming():
        for K, pad in ((72, 8), (71, 1), (600, 8), (601, 3)):
            A = torch.full((40, K + pad), float("inf"), dtype=torch.float16, device="cuda")
            B = torch.full((K + pad, 40), float("nan"), dtype=torch.float16, device="cuda")
            A[:, :K], B[:K] = 1.0, 0.5
            C = torch.empty((40, 40), dtype=torch.float16, device="cuda")
            hb.hidet_gemm(A[:, :K], B[:K], C, config=cfg)
            torch.cuda.synchronize()
            assert (C == 0.5 * K).all(), (cfg, K)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_a_residual_that_is_the_output_itself(dtype):
    """It is read before the main loop; each element by the thread that stores it."""
    for cfg, bm, bn in streaming():
        for M, N, K in ((3 * bm + 1, 2 * bn + 8, 600), (2 * bm, 3 * bn + 3, 601)):
            c = wl.gemm_case(9900 + cfg, M, N, K, dtype, bias="col", residual=True)
            A, B, bias, C = (to_gpu(c[n], dtype) for n in ("A", "B", "bias", "residual"))
            hb.hidet_gemm(A, B, C, epilogue=hb.make_epilogue(bias=bias, bias_axis=hb.HIDET_BIAS_PER_COL, residual=C), config=cfg)
            torch.cuda.synchronize()
            A64, B64, b64, r64 = (wl.widen(c[n], dtype) for n in ("A", "B", "bias", "residual"))
            ref = oracle.gemm(A64, B64, bias=b64, bias_axis=oracle.BIAS_PER_COL, residual=r64)
            assert_elementwise(to_f64(C), ref, gemm_scale(A64, B64, False, False, 1.0, b64, "col", r64), dtype, K, "config %d" % cfg)
