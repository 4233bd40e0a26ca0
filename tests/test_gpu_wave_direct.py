"""16-bit products on element-aligned rows whose wavefronts read K straight from memory (tiles of 16 rows, neither operand
transposed): values of K around a step, a round of steps and two of them, columns of odd count and fewer than a 16-byte chunk,
any alignment, K slices, fp32 results and fused input activations, against float64 within the derived bound of every element."""
import numpy as np
import pytest
import torch

from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TORCH_DTYPE, assert_elementwise, gemm_scale, to_f64

pytestmark = pytest.mark.gpu


def streaming():
    infos = [(i, hb.hidet_config_info(i)) for i in range(hb.hidet_config_count())]
    return [i for i, c in infos if not c["is_f32"] and c["schedule"] == 3 and c["block_m"] == 16 and c["block_n"] <= 32]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,N,shift", [(1, 2, 0), (16, 3, 0), (17, 33, 1), (50, 7, 2), (5, 47, 0)])
@pytest.mark.parametrize("K", [1, 2, 31, 32, 33, 511, 512, 514, 1024, 1059, 1600, 3072, 3075, 3076])
def test_against_float64(K, M, N, shift, dtype):
    g = wl.rng(9900 + K + M)
    a, b = (torch.from_numpy(g.uniform(-1, 1, s)).to(TORCH_DTYPE[dtype]) for s in ((M, K), (K, N)))
    buf = torch.full((a.numel() + b.numel() + 16,), float("nan"), dtype=a.dtype, device="cuda")  # (nothing beside them is used)
    A, B = buf[shift: shift + a.numel()].view(M, K), buf[shift + a.numel(): shift + a.numel() + b.numel()].view(K, N)
    A.copy_(a)
    B.copy_(b)
    a64, b64 = to_f64(A), to_f64(B)
    for config in streaming():
        C = torch.full((M, N), float("nan"), device="cuda", dtype=a.dtype)
        hb.hidet_gemm(A, B, C, config=config)
        assert_elementwise(to_f64(C), a64 @ b64, gemm_scale(a64, b64, False, False, 1.0), dtype, K, config)
        hb.hidet_gemm(A, B, C, epilogue=hb.make_epilogue(relu_input=True), config=config)
        r64 = np.maximum(a64, 0)
        assert_elementwise(to_f64(C), r64 @ b64, gemm_scale(r64, b64, False, False, 1.0), dtype, K, config)
        wide = torch.full((M, N), float("nan"), device="cuda")
        hb.hidet_gemm(A, B, wide, config=config)
        assert_elementwise(to_f64(wide), a64 @ b64, gemm_scale(a64, b64, False, False, 1.0), "f32", K, config)
        if K > 1:
            ws = torch.empty(3 * M * N, dtype=torch.float32, device="cuda")
            C3 = torch.full((1, M, N), float("nan"), device="cuda", dtype=a.dtype)
            hb.hidet_batched_gemm_splitk(A[None], B[None], C3, ws, k_slices=3, config=config)
            assert_elementwise(to_f64(C3[0]), a64 @ b64, gemm_scale(a64, b64, False, False, 1.0), dtype, K, config)
