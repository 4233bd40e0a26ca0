"""fp32 products whose wavefronts stream K from memory into registers (the K-splitting tiles): values of K around a step, a round
of steps and two of them, single rows and columns, all operand forms at any alignment, K slices, against float64 within the
derived bound of every element."""
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
