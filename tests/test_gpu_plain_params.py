"""Kernels of small tiles take the parameters of a plain product in a short form.  A call whose distances do not fit that form
(here: between the entries of a batch of one, which are never used) takes the long one: the same bits come out, also for each
entry of a batch in the short form."""
import ctypes

import pytest
import torch

from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TORCH_DTYPE, to_gpu

pytestmark = pytest.mark.gpu

FAR = 1 << 33


def _call(config, dtype, ta, tb, M, N, K, A, B, C, epilogue, stride):
    code = {"f32": hb.HIDET_F32, "f16": hb.HIDET_F16, "bf16": hb.HIDET_BF16}[dtype]
    return hb.lib().hidet_batched_gemm_cfg(
        config, code, code, int(ta), int(tb), 1, M, N, K, A.data_ptr(), A.stride(0), stride, B.data_ptr(), B.stride(0), stride,
        C.data_ptr(), C.stride(0), stride, ctypes.byref(epilogue), torch.cuda.current_stream().cuda_stream)


# one tile and a part of one, one to three and five tile rows (a last group of each size), long and short K
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (5, 70, 33), (64, 64, 512), (129, 48, 264), (130, 200, 1030), (321, 96, 72)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_short_and_long_parameters_give_the_same_bits(dtype, M, N, K):
    g = wl.rng(9700 + M)
    for i in range(hb.hidet_config_count()):
        info = hb.hidet_config_info(i)
        if info["block_m"] * info["block_n"] > 64 * 64 or (info["is_f32"] != 0) != (dtype == "f32"):
            continue
        for ta, tb in ((False, False), (False, True), (True, False), (True, True)):
            A = to_gpu(wl.to_storage(g.uniform(-1, 1, (K, M) if ta else (M, K)), dtype), dtype)
            B = to_gpu(wl.to_storage(g.uniform(-1, 1, (N, K) if tb else (K, N)), dtype), dtype)
            bias = to_gpu(wl.to_storage(g.uniform(-1, 1, (M if i % 2 else N,)), dtype), dtype)
            R = to_gpu(wl.to_storage(g.uniform(-1, 1, (M, N)), dtype), dtype) if i % 3 else None
            e = hb.make_epilogue(alpha=0.5, bias=bias, bias_axis=hb.HIDET_BIAS_PER_ROW if i % 2 else hb.HIDET_BIAS_PER_COL,
                                 residual=R, relu=i % 4 != 0)
            C = [torch.full((M, N), float("nan"), dtype=TORCH_DTYPE[dtype], device="cuda") for _ in range(2)]
            st = [_call(i, dtype, ta, tb, M, N, K, A, B, C[n], e, (1 << 20, FAR)[n]) for n in range(2)]
            torch.cuda.synchronize()
            assert st[0] == st[1], (i, ta, tb)
            if st[0] == 0:
                assert torch.equal(C[0], C[1]) and not torch.isnan(C[0]).any(), (i, ta, tb)
            else:
                assert ta, "a configuration that is built for this operand form"


# entries of one and of several tiles, last groups of one to four tile rows; operands, output and residual at distances of their own
@pytest.mark.parametrize("batch,M,N,K", [(3, 1, 1, 1), (5, 5, 70, 33), (2, 64, 64, 512), (3, 129, 48, 264), (2, 321, 96, 72)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_entries_of_a_batch_have_the_bits_of_long_parameters(dtype, batch, M, N, K):
    g = wl.rng(9750 + M)
    code = {"f32": hb.HIDET_F32, "f16": hb.HIDET_F16, "bf16": hb.HIDET_BF16}[dtype]

    def entries(rows, cols, gap):
        flat = to_gpu(wl.to_storage(g.uniform(-1, 1, (batch, rows * cols + gap)), dtype), dtype)
        return flat, [flat[e, :rows * cols].view(rows, cols) for e in range(batch)]

    for i in range(hb.hidet_config_count()):
        info = hb.hidet_config_info(i)
        if info["block_m"] * info["block_n"] > 64 * 64 or (info["is_f32"] != 0) != (dtype == "f32"):
            continue
        for ta, tb in ((False, False), (True, True)):
            A, a = entries(*((K, M) if ta else (M, K)), 8)
            B, b = entries(*((N, K) if tb else (K, N)), 24)
            R, r = entries(M, N, 16)
            bias = to_gpu(wl.to_storage(g.uniform(-1, 1, (N,)), dtype), dtype)
            shared = i % 3 == 0  # (one residual for all entries)
            epi = hb.make_epilogue(bias=bias, bias_axis=hb.HIDET_BIAS_PER_COL, residual=r[0], relu=True)
            epi.batch_stride_residual = 0 if shared else R.stride(0)
            C = torch.full((batch, M * N + 40), 7.0, dtype=TORCH_DTYPE[dtype], device="cuda")
            st = hb.lib().hidet_batched_gemm_cfg(i, code, code, int(ta), int(tb), batch, M, N, K, A.data_ptr(), a[0].stride(0), A.stride(0),
                                                 B.data_ptr(), b[0].stride(0), B.stride(0), C.data_ptr(), N, C.stride(0), ctypes.byref(epi),
                                                 torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            if st != 0:
                assert ta, "a configuration that is built for this operand form"
                continue
            assert bool((C[:, M * N:] == 7.0).all()), (i, ta, tb)
            for e in range(batch):
                one = hb.make_epilogue(bias=bias, bias_axis=hb.HIDET_BIAS_PER_COL, residual=r[0 if shared else e], relu=True)
                alone = torch.full((M, N), float("nan"), dtype=TORCH_DTYPE[dtype], device="cuda")
                assert _call(i, dtype, ta, tb, M, N, K, a[e], b[e], alone, one, FAR) == 0
                torch.cuda.synchronize()
                assert torch.equal(C[e, :M * N].view(M, N), alone), (i, ta, tb, e)
