"""The extension module that serves the plain calls of the binding against the general path: both are handed entry points
that only write down what they get, over every form of tensors and options, the refused ones among them."""
import ctypes
import types

import numpy as np
import pytest
import torch

from paper_2210_09603_amd import binding as hb

NAMES = ("hidet_gemm_cfg", "hidet_batched_gemm_cfg", "hidet_conv2d_implicit_gemm_cfg", "hidet_conv2d_implicit_gemm_packed",
         "hidet_softmax_rows", "hidet_reduce_rows")
F16, BF16, F32 = torch.float16, torch.bfloat16, torch.float32


class Stream:
    cuda_stream = 0x5EED


class Recorder:
    def __init__(self, monkeypatch, status=0):
        real, self.calls, self.status, self.keep = hb.lib(), [], status, []
        stub = types.SimpleNamespace(hidet_status_string=real.hidet_status_string)
        for name in NAMES:
            args = getattr(real, name).argtypes
            fn = ctypes.CFUNCTYPE(ctypes.c_int32, *args)(lambda *a, name=name: self.write(name, a))
            self.keep.append(fn)
            setattr(stub, name, fn)
        monkeypatch.setattr(hb, "_lib", stub)
        monkeypatch.setattr(hb, "_host_calls", hb._load_host_calls(stub))

    def write(self, name, args):
        seen = []
        for a in args:
            if isinstance(a, ctypes._Pointer):
                a = bytes(a.contents) if a else None
            seen.append(a)
        self.calls.append((name, tuple(seen)))
        return self.status

    def outcome(self, f, *args, **kw):
        self.calls.clear()
        try:
            f(*args, **kw)
            raised = None
        except Exception as e:
            raised = (type(e), str(e))
        return list(self.calls), raised


def same(rec, public, general, args, **kw):
    """What both paths did; the answer of the extension module tells whether it served the call."""
    a = rec.outcome(public, *args, **kw)
    b = rec.outcome(general, *args)
    assert a == b, (args, kw)
    return a


def t(*shape, dtype=F16):
    return torch.zeros(shape, dtype=dtype)


def epilogues():
    return [None, hb.make_epilogue(relu=True, alpha=0.5), hb.make_epilogue(bias=t(6), bias_axis=hb.HIDET_BIAS_PER_COL, residual=t(4, 6)),
            hb.make_epilogue(relu_input=True)]


def test_gemm(monkeypatch):
    rec = Recorder(monkeypatch)
    wide = t(9, 40)
    operands = [(t(4, 8), t(8, 6), t(4, 6)), (wide[:4, :8], wide[:8, 8:14], wide[:4, 20:26]), (t(8, 4).t(), t(8, 6), t(4, 6)),
                (t(4, 8), t(6, 8).t(), t(4, 6)), (t(1, 8), t(8, 6), t(1, 6)), (t(8, 1).t(), t(8, 6), t(1, 6)), (t(4, 1), t(1, 6), t(4, 6)),
                (t(4, 0), t(0, 6), t(4, 6)), (t(0, 8), t(8, 6), t(0, 6)), (t(4, 8), t(8, 6), t(6, 4).t()), (t(4, 8), t(7, 6), t(4, 6)),
                (t(4, 8), t(8, 6), t(4, 7)), (t(2, 4, 8), t(8, 6), t(4, 6)), (t(1, 4, 8), t(8, 6), t(4, 6)), (t(4, 8), t(8, 6), t(1, 4, 6)),
                (t(8), t(8, 6), t(1, 6)), (t(4, 8, dtype=F32), t(8, 6, dtype=F32), t(4, 6, dtype=F32)), (t(4, 8), t(8, 6), t(4, 6, dtype=F32)),
                (t(4, 8, dtype=torch.float64), t(8, 6), t(4, 6)), (t(4, 8), t(8, 6, dtype=BF16), t(4, 6)), (wide[:4, :16:2], t(8, 6), t(4, 6)),
                (torch.nn.Parameter(t(4, 8)), t(8, 6), t(4, 6)), (np.zeros((4, 8), np.float16), t(8, 6), t(4, 6)),
                (torch.empty((4, 8), dtype=F16, device="meta"), t(8, 6), t(4, 6)), (t(4, 8).to_sparse(), t(8, 6), t(4, 6))]
    served = 0
    turned = lambda x, turn: x.t() if turn and isinstance(x, torch.Tensor) and x.dim() == 2 and x.layout == torch.strided else x
    for A, B, C in operands:
        for e in epilogues():
            for tA, tB in ((False, False), (True, False), (False, True), (0, 1)):
                for config in (-1, 3):
                    _, raised = same(rec, hb.hidet_gemm, hb._gemm, (turned(A, tA), turned(B, tB), C, tA, tB, e, Stream(), config))
                    served += raised is None
    assert served >= 200
    for e in (hb.make_epilogue(head_split=(2, 3)), "no epilogue", types.SimpleNamespace(out_map=0)):
        for C in (t(4, 6), t(2, 2, 2, 3)):
            same(rec, hb.hidet_gemm, hb._gemm, (t(4, 8), t(8, 6), C, False, False, e, Stream(), -1))
    for config in (np.int64(3), 3.5, 2 ** 40, "3", True):
        same(rec, hb.hidet_gemm, hb._gemm, (t(4, 8), t(8, 6), t(4, 6), False, False, None, Stream(), config))
    for stream in (object(), types.SimpleNamespace(cuda_stream=None), types.SimpleNamespace(cuda_stream=0)):
        same(rec, hb.hidet_gemm, hb._gemm, (t(4, 8), t(8, 6), t(4, 6), False, False, None, stream, -1))


def test_batched_gemm(monkeypatch):
    rec = Recorder(monkeypatch)
    big = t(3, 9, 40)
    served = 0
    for A, B, C in [(t(3, 4, 8), t(3, 8, 6), t(3, 4, 6)), (big[:, :4, :8], big[:, :8, 8:14], big[:, :4, 20:26]),
                    (t(1, 4, 8).expand(3, 4, 8), t(3, 8, 6), t(3, 4, 6)), (t(4, 3, 8).transpose(0, 1), t(3, 8, 6), t(3, 4, 6)),
                    (t(1, 4, 8), t(1, 8, 6), t(1, 4, 6)), (big[:1, :4, :8], big[:1, :8, 8:14], big[:1, :4, 20:26]), (t(0, 4, 8), t(0, 8, 6), t(0, 4, 6)),
                    (t(3, 4, 8), t(2, 8, 6), t(3, 4, 6)), (t(3, 4, 8), t(3, 8, 6), t(2, 4, 6)), (t(4, 8), t(8, 6), t(4, 6)),
                    (t(3, 1, 8), t(3, 8, 1), t(3, 1, 1)), (t(3, 4, 8), t(3, 7, 6), t(3, 4, 6)), (t(3, 8, 4).transpose(1, 2), t(3, 8, 6), t(3, 4, 6))]:
        for e in (None, hb.make_epilogue(alpha=0.125, residual=t(3, 4, 6))):
            for tB in (False, True):
                _, raised = same(rec, hb.hidet_batched_gemm, hb._batched_gemm, (A, B.transpose(-1, -2).contiguous() if tB else B, C, False, tB, e, Stream(), -1))
                served += raised is None
    assert served >= 25


@pytest.mark.parametrize("packed", [False, True])
def test_convolutions(monkeypatch, packed):
    rec = Recorder(monkeypatch)
    served = 0
    for x, w, y, s, p in [((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 7), (1, 1), (1, 1)), ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 5, 4), (2, 2), (1, 1)),
                          ((2, 8, 9, 7), (5, 8, 3, 1), (2, 5, 3, 9), (3, 1), (0, 1)), ((0, 8, 9, 7), (5, 8, 3, 3), (0, 5, 9, 7), (1, 1), (1, 1)),
                          ((2, 8, 2, 2), (5, 8, 3, 3), (2, 5, 0, 0), (1, 1), (0, 0)), ((2, 8, 2, 2), (5, 8, 3, 3), (2, 5, 1, 1), (2, 2), (0, 0)),
                          ((2, 8, 9, 7), (5, 7, 3, 3), (2, 5, 9, 7), (1, 1), (1, 1)), ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 8), (1, 1), (1, 1)),
                          ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 7), (0, 1), (1, 1)), ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 7), [1, 1], (1, 1)),
                          ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 7), (1, 1, 9), (1, 1)), ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 7), (1.0, 1), (1, 1)),
                          ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 7), (-1, -1), (-7, -7)), ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 7), (1,), (1, 1)),
                          ((2, 8, 9, 7), (5, 8, 3, 3), (2, 5, 9, 7), (1, 1), (2 ** 62, 1))]:
        W = t(w[0], w[2], w[3], w[1]) if packed else t(*w)
        for X in (t(*x), t(x[0], x[2], x[3], x[1]).permute(0, 3, 1, 2)):
            for e in (None, hb.make_epilogue(bias=t(w[0]), bias_axis=hb.HIDET_BIAS_PER_ROW, relu=True)):
                if packed:
                    for slices in (0, 1, np.int64(2)):
                        _, raised = same(rec, lambda *a: hb.hidet_conv2d_implicit_gemm_packed(*a), hb._conv2d_packed,
                                         (X, W, t(*y), s, p, e, Stream(), -1, slices, None))
                        served += raised is None
                else:
                    _, raised = same(rec, hb.hidet_conv2d_implicit_gemm, hb._conv2d, (X, W, t(*y), s, p, e, Stream(), -1))
                    served += raised is None
    assert served >= 8


def test_rows(monkeypatch):
    rec = Recorder(monkeypatch)
    served = 0
    wide = t(9, 40)
    for x in (t(5, 7), t(7), t(0), t(0, 7), t(5, 0), t(2, 3, 7), t(2, 3, 0), wide[:5, :7], wide[:1, :7], wide[:5, :14:2], wide[:5, :1], t(3, 2, 7).transpose(0, 1),
              t(5, 7, dtype=BF16), t(5, 7, dtype=F32), t(5, 7, dtype=torch.int32), torch.tensor(1.0, dtype=F16), t(7, 5).t()):
        for y in (x, torch.zeros(x.shape, dtype=x.dtype), torch.zeros(x.shape, dtype=F32), t(5, 8)):
            _, raised = same(rec, hb.hidet_softmax_rows, hb._softmax_rows, (x, y, Stream()))
            served += raised is None
        rows = x.numel() // x.shape[-1] if x.dim() > 0 and x.shape[-1] else 5
        for y in (t(rows), t(rows, dtype=F32), t(rows, 1), t(rows + 1), t(2 * rows)[::2], torch.zeros(rows, dtype=torch.int64)):
            for op in (hb.HIDET_REDUCE_SUM, hb.HIDET_REDUCE_MAX, np.int32(2), "sum"):
                _, raised = same(rec, hb.hidet_reduce_rows, hb._reduce_rows, (x, y, op, Stream()))
                served += raised is None
    assert served >= 100


def test_a_status_is_raised_once(monkeypatch):
    rec = Recorder(monkeypatch, status=2)
    for f, args, name in ((hb.hidet_gemm, (t(4, 8), t(8, 6), t(4, 6)), "hidet_gemm"),
                          (hb.hidet_batched_gemm, (t(3, 4, 8), t(3, 8, 6), t(3, 4, 6)), "hidet_batched_gemm"),
                          (hb.hidet_softmax_rows, (t(4, 8), t(4, 8)), "hidet_softmax_rows"), (hb.hidet_reduce_rows, (t(4, 8), t(4)), "hidet_reduce_rows"),
                          (hb.hidet_conv2d_implicit_gemm, (t(1, 8, 4, 4), t(8, 8, 1, 1), t(1, 8, 4, 4)), "hidet_conv2d_implicit_gemm"),
                          (hb.hidet_conv2d_implicit_gemm_packed, (t(1, 8, 4, 4), t(8, 1, 1, 8), t(1, 8, 4, 4)), "hidet_conv2d_implicit_gemm_packed")):
        calls, raised = rec.outcome(f, *args, stream=Stream())
        assert len(calls) == 1 and raised[0] is hb.HidetError and raised[1].startswith(name + ": status 2"), (name, raised)


def test_the_plain_forms_do_not_take_the_general_path(monkeypatch):
    rec = Recorder(monkeypatch)
    for general in ("_gemm", "_batched_gemm", "_conv2d", "_conv2d_packed", "_softmax_rows", "_reduce_rows"):
        monkeypatch.setattr(hb, general, None)
    s = Stream()
    hb.hidet_gemm(t(4, 8), t(6, 8), t(4, 6), transB=True, epilogue=hb.make_epilogue(relu=True), stream=s)
    hb.hidet_batched_gemm(t(1, 4, 8).expand(3, 4, 8), t(3, 8, 6), t(3, 4, 6), stream=s)
    hb.hidet_conv2d_implicit_gemm(t(1, 8, 4, 4), t(8, 8, 3, 3), t(1, 8, 4, 4), pad=(1, 1), stream=s)
    hb.hidet_conv2d_implicit_gemm_packed(t(1, 8, 4, 4), t(8, 3, 3, 8), t(1, 8, 4, 4), pad=(1, 1), stream=s)
    hb.hidet_softmax_rows(t(2, 3, 8), t(2, 3, 8), stream=s)
    hb.hidet_reduce_rows(t(4, 8), t(4), stream=s)
    assert len(rec.calls) == 6


def test_missing_extension_fails_loudly(monkeypatch):
    monkeypatch.setattr(hb, "_host_calls", None)
    monkeypatch.setattr(hb, "HOST_CALLS_PATH", "/nonexistent/_host_calls.so")
    with pytest.raises(RuntimeError, match="host extension missing"):
        hb.hidet_gemm(t(4, 8), t(8, 6), t(4, 6))


def test_extension_built_for_another_torch_is_refused(monkeypatch):
    monkeypatch.setattr(hb, "_host_calls", None)
    monkeypatch.setattr(hb, "built_for", lambda: "torch 0.0, Python 3.0")
    with pytest.raises(RuntimeError, match="was built for torch"):
        hb._calls()


def test_extension_is_rebuilt_for_another_torch_or_compiler(monkeypatch):
    from paper_2210_09603_amd import build

    seen = {build._host_digest()}
    monkeypatch.setenv("CXX", "another-compiler")
    seen.add(build._host_digest())
    monkeypatch.setattr(hb, "built_for", lambda: "torch 0.0, Python 3.0")
    seen.add(build._host_digest())
    assert len(seen) == 3
