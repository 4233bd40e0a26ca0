"""fp32 products whose wavefronts stream K from memory into registers (the K-splitting tiles): values of K around a step, a round
of steps and two of them, single rows and columns, all operand forms at any alignment, K slices, every option of the epilogue, batches
and input activations, against float64 within the derived bound of every element."""
import numpy as np
import pytest
import torch

from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TOL, assert_elementwise, gemm_scale, to_f64, to_gpu

pytestmark = pytest.mark.gpu


def streaming():
    infos = [(i, hb.hidet_config_info(i)) for i in range(hb.hidet_config_count())]
    return [i for i, c in infos if c["is_f32"] and c["schedule"] == 3]


@pytest.mark.parametrize("M,N,shift", [(1, 1, 0), (16, 16, 0), (17, 33, 1), (50, 20, 3), (64, 47, 0)])
@pytest.mark.parametrize("K", [1, 15, 16, 17, 255, 256, 257, 512, 529, 768, 1039])
def test_against_float64(K, M, N, shift):
    g = wl.rng(9800 + K + M)
    for config in streaming():
        for ta, tb in ((False, False), (False, True), (True, False), (True, True)):
            a, b = (g.uniform(-1, 1, s).astype(np.float32) for s in (((K, M) if ta else (M, K)), ((N, K) if tb else (K, N))))
            buf = torch.zeros(a.size + b.size + 16, dtype=torch.float32, device="cuda")
            A, B = buf[shift: shift + a.size].view(a.shape), buf[shift + a.size: shift + a.size + b.size].view(b.shape)
            A.copy_(to_gpu(a, "f32"))
            B.copy_(to_gpu(b, "f32"))
            C = torch.full((M, N), float("nan"), device="cuda")
            hb.hidet_gemm(A, B, C, transA=ta, transB=tb, config=config)
            a64, b64 = a.astype(np.float64), b.astype(np.float64)
            ref = (a64.T if ta else a64) @ (b64.T if tb else b64)
            assert_elementwise(to_f64(C), ref, gemm_scale(a64, b64, ta, tb, 1.0), "f32", K, (config, ta, tb))
            if K > 1:
                ws = torch.empty(3 * M * N, dtype=torch.float32, device="cuda")
                C3 = torch.full((1, M, N), float("nan"), device="cuda")
                hb.hidet_batched_gemm_splitk(A[None], B[None], C3, ws, k_slices=3, transA=ta, transB=tb, config=config)
                assert np.linalg.norm(to_f64(C3[0]) - ref) <= TOL["f32"] * np.linalg.norm(ref) + 1e-6, (config, ta, tb)


# rows of whole chunks and odd ones, a width of a head of whole groups of four columns and an odd one
@pytest.mark.parametrize("M,N,K,head", [(48, 72, 1096, 8), (21, 35, 261, 7), (16, 16, 16, 4), (3, 2, 5, 1)])
def test_batches_epilogues_input_relu_and_head_split(M, N, K, head):
    g = wl.rng(9850 + K)
    b = 3
    a, w, r = (g.uniform(-1, 1, s).astype(np.float32) for s in ((b, M, K), (b, K, N), (b, M, N)))
    bias = {"col": g.uniform(-1, 1, N).astype(np.float32), "row": g.uniform(-1, 1, M).astype(np.float32)}
    A, B, R = to_gpu(a, "f32"), to_gpu(w, "f32"), to_gpu(r, "f32")
    a64, w64, r64 = (t.astype(np.float64) for t in (a, w, r))
    code = {"col": hb.HIDET_BIAS_PER_COL, "row": hb.HIDET_BIAS_PER_ROW}
    for config in streaming():
        for axis, relu, relu_input, batched_residual, in_place in (("col", True, False, True, False), ("row", False, True, False, False),
                                                                   ("col", False, True, True, True), ("row", True, False, None, False)):
            C = R.clone() if in_place else torch.full((b, M, N), float("nan"), device="cuda")
            res = None if batched_residual is None else C if in_place else R if batched_residual else R[0]
            vec = to_gpu(bias[axis], "f32")
            epi = hb.make_epilogue(alpha=0.5, bias=vec, bias_axis=code[axis], residual=res, relu=relu, relu_input=relu_input)
            hb.hidet_batched_gemm(A, B, C, epilogue=epi, config=config)
            for i in range(b):
                left = np.maximum(a64[i], 0) if relu_input else a64[i]
                v64 = bias[axis].astype(np.float64)
                part = None if res is None else r64[i if batched_residual else 0]
                ref = 0.5 * (left @ w64[i]) + (v64[None, :] if axis == "col" else v64[:, None]) + (0 if part is None else part)
                ref = np.maximum(ref, 0) if relu else ref
                assert_elementwise(to_f64(C[i]), ref, gemm_scale(left, w64[i], False, False, 0.5, v64, axis, part), "f32", K, (config, axis, i))
        # rows of all entries against one right operand, stored as heads, with the residual in that order
        H = torch.full((b, N // head, M, head), float("nan"), device="cuda")
        rh = g.uniform(-1, 1, tuple(H.shape)).astype(np.float32)
        col = to_gpu(bias["col"], "f32")
        epi = hb.make_epilogue(bias=col, bias_axis=code["col"], residual=to_gpu(rh, "f32"), relu=True, head_split=(M, head))
        hb.hidet_gemm(A.view(b * M, K), B[0], H, epilogue=epi, config=config)
        rows = a64.reshape(b * M, K)
        part = rh.astype(np.float64).transpose(0, 2, 1, 3).reshape(b * M, N)
        c64 = bias["col"].astype(np.float64)
        ref = np.maximum(rows @ w64[0] + c64[None, :] + part, 0)
        assert_elementwise(to_f64(H).transpose(0, 2, 1, 3).reshape(b * M, N), ref,
                           gemm_scale(rows, w64[0], False, False, 1.0, c64, "col", part), "f32", K, (config, "heads"))


def test_infinities_beyond_k_do_not_reach_the_result():
    """The last step reads no value beyond K that it uses, in every operand form."""
    for config in streaming():
        for K, pad in ((5, 1), (72, 8), (271, 3), (600, 8)):
            A = torch.full((K + pad, K + pad), float("inf"), device="cuda")
            B = torch.full((K + pad, K + pad), float("nan"), device="cuda")
            n = min(K, 40)
            for ta, tb in ((False, False), (False, True), (True, False), (True, True)):
                Av, Bv = (A[:K, :n] if ta else A[:n, :K]), (B[:n, :K] if tb else B[:K, :n])
                A.fill_(float("inf")), B.fill_(float("nan"))
                Av.fill_(1.0), Bv.fill_(0.5)
                C = torch.empty((n, n), device="cuda")
                hb.hidet_gemm(Av, Bv, C, transA=ta, transB=tb, config=config)
                assert bool((C == 0.5 * K).all()), (config, K, ta, tb)
