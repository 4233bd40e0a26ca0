"""Parity of the reduction template (row sum / max / mean, row softmax) and of attention composed from the
library's own calls, against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from oracle import reduction as red
from paper_2210_09603_amd import binding as hb
from paper_2210_09603_amd import workloads as wl

from helpers import TOL, TORCH_DTYPE, to_f64, to_gpu, within_bound

pytestmark = pytest.mark.gpu

# row lengths that hit every lane grouping, every repeat count, ragged last chunks and the streamed kernel
COLS_16 = [1, 7, 8, 33, 64, 100, 128, 257, 512, 513, 1000, 2048, 3001, 8192, 8193, 20000]
COLS_32 = [1, 3, 4, 33, 100, 256, 1000, 4096, 4097, 9001]


def _say(msg):
    print(msg, flush=True)


def _rows_for(cols):
    return 37 if cols <= 4096 else 5


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_softmax_rows(dtype):
    g = wl.rng(9100)
    for cols in (COLS_32 if dtype == "f32" else COLS_16):
        rows = _rows_for(cols)
        x = wl.to_storage((g.standard_normal((rows, cols)) * 3).astype(np.float32), dtype)
        dx = to_gpu(x, dtype)
        dy = torch.full((rows, cols), float("nan"), dtype=TORCH_DTYPE[dtype], device="cuda")
        hb.hidet_softmax_rows(dx, dy)
        torch.cuda.synchronize()
        ref = red.softmax_rows(wl.widen(x, dtype))
        err = oracle.rel_frobenius(to_f64(dy), ref)
        _say("softmax %s cols %d err %.3e" % (dtype, cols, err))
        assert within_bound(err, ref, dtype), cols
        hb.hidet_softmax_rows(dx, dx)  # in place
        torch.cuda.synchronize()
        assert torch.equal(dx, dy), cols


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_softmax_strided_misaligned_and_masked(dtype):
    g = wl.rng(9200)
    es = 4 if dtype == "f32" else 2
    for cols, ld, shift in ((100, 104, 0), (100, 107, 0), (96, 96, 1), (5000 * (4 // es + 1), 5000 * (4 // es + 1) + 3, 1)):
        rows = 9
        x = wl.to_storage((g.standard_normal((rows, cols)) * 2).astype(np.float32), dtype)
        x64 = wl.widen(x, dtype)
        x64[1, : cols // 2] = -np.inf  # a masked prefix, as in causal attention
        buf = torch.full((rows * ld + shift + 8,), 7.0, dtype=TORCH_DTYPE[dtype], device="cuda")
        view = buf[shift: shift + rows * ld].view(rows, ld)[:, :cols]
        view.copy_(torch.from_numpy(x64).to(TORCH_DTYPE[dtype]))
        out = torch.full((rows * ld + shift + 8,), 7.0, dtype=TORCH_DTYPE[dtype], device="cuda")
        oview = out[shift: shift + rows * ld].view(rows, ld)[:, :cols]
        hb.hidet_softmax_rows(view, oview)
        torch.cuda.synchronize()
        ref = red.softmax_rows(x64)
        assert within_bound(oracle.rel_frobenius(to_f64(oview), ref), ref, dtype), (cols, ld, shift)
        assert torch.all(oview[1, : cols // 2] == 0)
        # nothing outside the rows was written
        full = out[shift: shift + rows * ld].view(rows, ld)
        assert torch.all(full[:, cols:] == 7.0) and torch.all(out[:shift] == 7.0) and torch.all(out[shift + rows * ld:] == 7.0)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_reduce_rows(dtype):
    g = wl.rng(9300)
    for cols in (COLS_32 if dtype == "f32" else COLS_16):
        rows = _rows_for(cols)
        x = wl.to_storage(g.standard_normal((rows, cols)).astype(np.float32) + 0.25, dtype)
        dx = to_gpu(x, dtype)
        x64 = wl.widen(x, dtype)
        for op, name in ((hb.HIDET_REDUCE_SUM, red.SUM), (hb.HIDET_REDUCE_MAX, red.MAX), (hb.HIDET_REDUCE_MEAN, red.MEAN)):
            ref = red.reduce_rows(x64, name)
            y32 = torch.full((rows,), float("nan"), dtype=torch.float32, device="cuda")
            hb.hidet_reduce_rows(dx, y32, op)
            y = torch.full((rows,), float("nan"), dtype=TORCH_DTYPE[dtype], device="cuda")
            hb.hidet_reduce_rows(dx, y, op)
            torch.cuda.synchronize()
            if op == hb.HIDET_REDUCE_MAX:
                assert np.array_equal(to_f64(y32), ref) and np.array_equal(to_f64(y), ref), cols  # exact: no arithmetic
            else:
                assert oracle.rel_frobenius(to_f64(y32), ref) <= 1e-5, (cols, op)
                assert within_bound(oracle.rel_frobenius(to_f64(y), ref), ref, dtype), (cols, op)


def test_reduce_closed_forms_and_degenerate_shapes():
    n = 3000
    x = torch.arange(1, n + 1, dtype=torch.float32, device="cuda").repeat(3, 1)
    y = torch.zeros(3, dtype=torch.float32, device="cuda")
    hb.hidet_reduce_rows(x, y, hb.HIDET_REDUCE_SUM)
    torch.cuda.synchronize()
    assert y.tolist() == [n * (n + 1) / 2] * 3  # every partial sum is an integer below 2^24: exact in fp32
    empty = torch.zeros((2, 0), dtype=torch.float16, device="cuda")
    y = torch.full((2,), 5.0, dtype=torch.float32, device="cuda")
    hb.hidet_reduce_rows(empty, y, hb.HIDET_REDUCE_SUM)
    torch.cuda.synchronize()
    assert y.tolist() == [0.0, 0.0]
    hb.hidet_reduce_rows(empty, y, hb.HIDET_REDUCE_MAX)
    torch.cuda.synchronize()
    assert y.tolist() == [-np.inf, -np.inf]
    hb.hidet_softmax_rows(empty, empty)
    hb.hidet_softmax_rows(torch.zeros((0, 5), dtype=torch.float16, device="cuda"),
                          torch.zeros((0, 5), dtype=torch.float16, device="cuda"))
    ones = torch.full((4, 16), 2.5, dtype=torch.float16, device="cuda")
    hb.hidet_softmax_rows(ones, ones)
    torch.cuda.synchronize()
    assert torch.all(ones == 1.0 / 16)


@pytest.mark.parametrize("batch,seq", [(12, 128), (12, 512)])
def test_attention_from_the_three_calls(batch, seq):
    """scores = alpha * Q.K^T (fused scale), softmax in place, context = S.V -- every step in the library."""
    c = wl.attention_case(9400 + seq, batch, seq, "f16")
    Q, K, V = (to_gpu(c[k], "f16") for k in ("Q", "K", "V"))
    scores = torch.empty((batch, seq, seq), dtype=torch.float16, device="cuda")
    ctx = torch.full((batch, seq, c["d"]), float("nan"), dtype=torch.float16, device="cuda")
    hb.hidet_batched_gemm(Q, K, scores, transB=True, epilogue=hb.make_epilogue(alpha=c["alpha"]))
    hb.hidet_softmax_rows(scores, scores)
    hb.hidet_batched_gemm(scores, V, ctx)
    torch.cuda.synchronize()
    ref = red.attention(wl.widen(c["Q"], "f16"), wl.widen(c["K"], "f16"), wl.widen(c["V"], "f16"), c["alpha"])
    err = oracle.rel_frobenius(to_f64(ctx), ref)
    _say("attention b%d s%d err %.3e" % (batch, seq, err))
    assert err <= TOL["f16"]


def test_hip_graph_replays_of_the_attention_chain_match_eager():
    """The library only launches kernels on the caller's stream (no allocation, no memset, no synchronisation),
    so a caller may capture it; every replay must reproduce the eager result bit for bit."""
    c = wl.attention_case(9500, 6, 128, "f16")
    Q, K, V = (to_gpu(c[k], "f16") for k in ("Q", "K", "V"))
    scores = torch.empty((6, 128, 128), dtype=torch.float16, device="cuda")
    ctx = torch.zeros((6, 128, 64), dtype=torch.float16, device="cuda")
    epi = hb.make_epilogue(alpha=c["alpha"])

    def chain():
        hb.hidet_batched_gemm(Q, K, scores, transB=True, epilogue=epi)
        hb.hidet_softmax_rows(scores, scores)
        hb.hidet_batched_gemm(scores, V, ctx)

    chain()
    torch.cuda.synchronize()
    eager = ctx.clone()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        chain()  # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            chain()
    for replay in range(3):
        ctx.zero_()
        scores.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ctx, eager), replay
        V2 = V * 1.0  # unrelated eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(V2, V)


def test_stream_bandwidth_probe_reports_plausible_rates():
    ring = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    rates = [hb.hidet_probe_stream_bandwidth(ring, mode) for mode in range(3)]
    print("read %.0f write %.0f copy %.0f GB/s" % tuple(rates), flush=True)
    for r in rates:
        assert 1000.0 < r < 8000.0  # below the datasheet's HBM rate, far above anything a broken probe reports
    with pytest.raises(hb.HidetError):
        hb.hidet_probe_stream_bandwidth(ring, 3)
    with pytest.raises(hb.HidetError):
        hb.hidet_probe_stream_bandwidth(ring[: 100 << 20], 0)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_rows_at_the_edges_of_the_kernels(dtype):
    """Row lengths on both sides of every boundary between the kernels (64, 128, 256, ... 16384 chunks of 16 bytes; the one
    before 8192 lies at 8191 and 8192), with whole and ragged last chunks, in and out of place, rows aligned and not.  Same
    bounds as the tests above."""
    vec = 4 if dtype == "f32" else 8
    g = wl.rng(9600)
    for chunks in (8, 16, 32, 64, 128, 256, 512, 768, 1024, 2048, 4096, 6283, 8191, 8192, 16383, 16384):
        for cols in (chunks * vec, chunks * vec - 1, chunks * vec + 1, (chunks - 1) * vec + 1):
            for ld in (cols, cols + 3):
                rows = 3
                x = wl.to_storage((g.standard_normal((rows, ld)) * 3).astype(np.float32), dtype)
                dx = to_gpu(x, dtype)
                x64 = wl.widen(x, dtype)[:, :cols]
                ref = red.softmax_rows(x64)
                out = torch.full((rows, ld), 7.0, dtype=TORCH_DTYPE[dtype], device="cuda")
                hb.hidet_softmax_rows(dx[:, :cols], out[:, :cols])
                y = {op: torch.full((rows,), float("nan"), dtype=torch.float32, device="cuda")
                     for op in (hb.HIDET_REDUCE_SUM, hb.HIDET_REDUCE_MEAN, hb.HIDET_REDUCE_MAX)}
                for op in y:
                    hb.hidet_reduce_rows(dx[:, :cols], y[op], op)
                torch.cuda.synchronize()
                assert within_bound(oracle.rel_frobenius(to_f64(out)[:, :cols], ref), ref, dtype), (cols, ld)
                assert torch.all(out[:, cols:] == 7.0), (cols, ld)
                # fp32 sums of signed values: the bound is relative to the sum of magnitudes
                assert np.all(np.abs(to_f64(y[hb.HIDET_REDUCE_SUM]) - x64.sum(1)) <= 1e-6 * np.abs(x64).sum(1)), (cols, ld)
                assert np.all(np.abs(to_f64(y[hb.HIDET_REDUCE_MEAN]) - x64.mean(1)) <= 1e-6 * np.abs(x64).mean(1)), (cols, ld)
                assert np.array_equal(to_f64(y[hb.HIDET_REDUCE_MAX]), x64.max(1)), (cols, ld)
                hb.hidet_softmax_rows(dx[:, :cols], dx[:, :cols])  # in place
                torch.cuda.synchronize()
                assert torch.equal(dx[:, :cols], out[:, :cols]), (cols, ld)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_shifted_chunks_of_long_softmax_rows(dtype):
    """Rows of 4097 to 16383 chunks whose output is not 16-byte aligned are cut on the output's own 16-byte grid, which may
    take one chunk more: the longest rows that each kernel holds, at every offset of the output, with a prefix of -inf, a row
    of -inf alone and a NaN; nothing beside the rows is written."""
    vec = 4 if dtype == "f32" else 8
    g = wl.rng(9900)
    for chunks in (4097, 6283, 8191, 8192, 16383):
        for cols in (chunks * vec, (chunks - 1) * vec + 1):
            rows, ld = 4, cols + 1 + cols % 2  # (an odd step: the offset within 16 bytes differs from row to row)
            x = wl.to_storage((g.standard_normal((rows, cols)) * 3).astype(np.float32), dtype)
            x64 = wl.widen(x, dtype)
            x64[1, : cols // 3] = -np.inf
            x64[2, :] = -np.inf
            x64[3, cols - 2] = np.nan
            dx = torch.from_numpy(x64).to(TORCH_DTYPE[dtype]).cuda()
            for offset in (0, 1, vec - 1):
                buf = torch.full((offset + rows * ld + 16,), 7.0, dtype=TORCH_DTYPE[dtype], device="cuda")
                out = buf[offset: offset + rows * ld].view(rows, ld)
                hb.hidet_softmax_rows(dx, out[:, :cols])
                torch.cuda.synchronize()
                got = to_f64(out)[:, :cols]
                ref = red.softmax_rows(x64[:2])
                assert within_bound(oracle.rel_frobenius(got[:2], ref), ref, dtype), (cols, offset)
                assert np.all(got[1, : cols // 3] == 0.0) and np.all(np.isnan(got[2:])), (cols, offset)
                assert torch.all(out[:, cols:] == 7.0) and torch.all(buf[:offset] == 7.0), (cols, offset)
                assert torch.all(buf[offset + rows * ld:] == 7.0), (cols, offset)


@pytest.mark.parametrize("dtype,rows", [("f32", 600), ("bf16", 520)])
def test_many_very_long_rows(dtype, rows):
    """More than 8192 chunks in at least 512 rows: reductions take the streamed kernel on 512 threads."""
    cols = 33003 if dtype == "f32" else 66001
    x = (torch.arange(rows * cols, device="cuda") % 1021).view(rows, cols).to(torch.int32)
    xf = (x % 3).to(TORCH_DTYPE[dtype])  # small integers: sums below 2^24 are exact in any order
    y = torch.zeros(rows, dtype=torch.float32, device="cuda")
    hb.hidet_reduce_rows(xf, y, hb.HIDET_REDUCE_SUM)
    torch.cuda.synchronize()
    assert torch.equal(y.to(torch.int64), (x % 3).sum(1))


@pytest.mark.parametrize("dtype,rows", [("f32", 512), ("f16", 520), ("bf16", 513)])
def test_reductions_of_many_long_rows(dtype, rows):
    """Streamed reductions: 1025 chunks to beyond 16384, whole and ragged, at every boundary of the choice of the threads."""
    vec = 4 if dtype == "f32" else 8
    buf = (torch.arange(rows * 16386 * vec, device="cuda", dtype=torch.int32) % 1021) % 3  # small integers: sums are exact
    buf = buf.to(TORCH_DTYPE[dtype])
    for chunks in (1025, 1500, 2048, 2049, 5000, 8191, 8192, 16384, 16385):
        for cols in (chunks * vec, (chunks - 1) * vec + 1):
            x = buf[: rows * cols].view(rows, cols)
            x[rows - 1, cols - 1] = 5.0  # the last element, and an odd one out, are part of the row
            total, top = x.to(torch.float64).sum(1), x.to(torch.float64).max(1).values
            for op, ref in ((hb.HIDET_REDUCE_SUM, total), (hb.HIDET_REDUCE_MAX, top), (hb.HIDET_REDUCE_MEAN, total / cols)):
                y = torch.full((rows,), float("nan"), dtype=torch.float32, device="cuda")
                hb.hidet_reduce_rows(x, y, op)
                torch.cuda.synchronize()
                # (the mean is one fp32 division of an exact sum)
                assert torch.allclose(y.double(), ref, rtol=2.0 ** -23 if op == hb.HIDET_REDUCE_MEAN else 0.0, atol=0.0), (cols, op)


@pytest.mark.parametrize("cols", [33, 512, 5000, 60001])
def test_softmax_of_the_most_negative_finite_values(cols):
    """Masks made of the lowest finite value: an exponential of the difference, not a difference of scaled values."""
    low = torch.finfo(torch.float32).min
    x = torch.full((2, cols), low, device="cuda")
    x[1, 3:5] = 1.0
    y = torch.empty_like(x)
    hb.hidet_softmax_rows(x, y)
    torch.cuda.synchronize()
    assert torch.allclose(y[0], torch.full((cols,), 1.0 / cols, device="cuda"), rtol=1e-5, atol=0.0)
    assert y[1, 3] == 0.5 and y[1, 4] == 0.5 and y[1].sum() == 1.0


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_many_rows_of_medium_length(dtype):
    """129 to 768 chunks with enough rows for a wavefront per row, and one row fewer (a workgroup per row): row count times
    chunks at every boundary of the choice, whole and ragged, in and out of place."""
    vec = 4 if dtype == "f32" else 8
    g = wl.rng(9700)
    for chunks, rows in ((129, 1023), (129, 1024), (192, 1025), (256, 1024), (257, 1024), (384, 1024), (385, 1024), (512, 1024),
                         (513, 512), (768, 511), (768, 512)):
        for cols in (chunks * vec, (chunks - 1) * vec + 1):
            n = rows if cols % vec == 0 else 2 * rows
            x = wl.to_storage((g.standard_normal((n, cols)) * 3).astype(np.float32), dtype)
            x64 = wl.widen(x, dtype)
            dx = to_gpu(x, dtype)
            out = torch.full_like(dx, float("nan"))
            hb.hidet_softmax_rows(dx, out)
            y = {op: torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
                 for op in (hb.HIDET_REDUCE_SUM, hb.HIDET_REDUCE_MEAN, hb.HIDET_REDUCE_MAX)}
            for op in y:
                hb.hidet_reduce_rows(dx, y[op], op)
            hb.hidet_softmax_rows(dx, dx)
            torch.cuda.synchronize()
            ref = red.softmax_rows(x64)
            assert within_bound(oracle.rel_frobenius(to_f64(out), ref), ref, dtype), (cols, n)
            assert torch.equal(dx, out), (cols, n)
            # fp32 sums of signed values: the bound is relative to the sum of magnitudes
            assert np.all(np.abs(to_f64(y[hb.HIDET_REDUCE_SUM]) - x64.sum(1)) <= 1e-6 * np.abs(x64).sum(1)), (cols, n)
            assert np.all(np.abs(to_f64(y[hb.HIDET_REDUCE_MEAN]) - x64.mean(1)) <= 1e-6 * np.abs(x64).mean(1)), (cols, n)
            assert np.array_equal(to_f64(y[hb.HIDET_REDUCE_MAX]), x64.max(1)), (cols, n)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_rows_shorter_than_one_access(dtype):
    """Rows of fewer elements than 16 bytes hold: nothing beside them is read (NaN) or written, and an empty row is not read."""
    vec = 4 if dtype == "f32" else 8
    g = wl.rng(9800)
    for cols in range(0, vec + 1):
        rows, ld = 1001, cols + 2
        x = wl.to_storage((g.standard_normal((rows, ld)) * 3).astype(np.float32), dtype)
        x64 = wl.widen(x, dtype)[:, :cols]
        dx = to_gpu(x, dtype)
        dx[:, cols:] = float("nan")
        out = torch.full_like(dx, 7.0)
        hb.hidet_softmax_rows(dx[:, :cols], out[:, :cols])
        y = {op: torch.full((rows,), 7.0, dtype=torch.float32, device="cuda")
             for op in (hb.HIDET_REDUCE_SUM, hb.HIDET_REDUCE_MEAN, hb.HIDET_REDUCE_MAX)}
        for op in y:
            hb.hidet_reduce_rows(dx[:, :cols], y[op], op)
        torch.cuda.synchronize()
        assert torch.all(out[:, cols:] == 7.0), cols
        if cols == 0:
            assert torch.all(y[hb.HIDET_REDUCE_SUM] == 0) and torch.all(y[hb.HIDET_REDUCE_MAX] == -float("inf"))
            assert torch.all(torch.isnan(y[hb.HIDET_REDUCE_MEAN]))
            continue
        ref = red.softmax_rows(x64)
        assert within_bound(oracle.rel_frobenius(to_f64(out)[:, :cols], ref), ref, dtype), cols
        assert np.all(np.abs(to_f64(y[hb.HIDET_REDUCE_SUM]) - x64.sum(1)) <= 1e-6 * np.abs(x64).sum(1)), cols
        assert np.all(np.abs(to_f64(y[hb.HIDET_REDUCE_MEAN]) - x64.mean(1)) <= 1e-6 * np.abs(x64).mean(1)), cols
        assert np.array_equal(to_f64(y[hb.HIDET_REDUCE_MAX]), x64.max(1)), cols


@pytest.mark.parametrize("rows,cols", [(6, 1000), (6, 4100), (6, 12000), (6, 70000), (600, 6000), (520, 33001)])
def test_sums_of_the_wavefronts_meet_in_a_tree(rows, cols):
    """2^24 in the chunks of the first wavefront, 1 in those of every other one.  Added in a tree of log2(wavefronts) levels
    a sum rounds once a level, by at most 1 (half a unit of [2^24, 2^25)); one after another it loses every 1."""
    s = hb.hidet_row_schedule(hb.HIDET_F32, 0, rows, cols)
    assert s["form"] > 0
    waves = s["workgroup_size"] // 64
    x = torch.zeros(rows, cols, device="cuda")
    x[:, 0] = 2.0 ** 24
    for w in range(1, waves):
        x[:, w * 64 * 4] = 1.0
    y = torch.empty(rows, device="cuda")
    hb.hidet_reduce_rows(x, y)
    torch.cuda.synchronize()
    assert float((y.double() - (2.0 ** 24 + waves - 1)).abs().max()) <= int(np.log2(waves))


@pytest.mark.parametrize("cols", [12000, 70000])
def test_softmax_sums_of_the_wavefronts_meet_in_a_tree(cols):
    """As above, with exponentials of 1 and 2^-24 over sixteen wavefronts: four roundings of the sum by at most 2^-24, one
    reciprocal, one product and one exponential (2^-23 each); one after another the sum is off by 15 * 2^-24."""
    assert hb.hidet_row_schedule(hb.HIDET_F32, 1, 3, cols)["workgroup_size"] == 1024
    x = torch.full((3, cols), -float("inf"), device="cuda")
    x[:, 0] = 0.0
    for w in range(1, 16):
        x[:, w * 64 * 4] = -24 * float(np.log(2.0))
    y = torch.empty_like(x)
    hb.hidet_softmax_rows(x, y)
    torch.cuda.synchronize()
    assert float((y[:, 0].double() - torch.softmax(x.double(), 1)[:, 0]).abs().max()) <= (4 + 3 * 2) * 2.0 ** -24


@pytest.mark.parametrize("dtype,cols", [("f16", 1100), ("bf16", 2049), ("f16", 8200), ("bf16", 33000), ("f16", 50257), ("bf16", 70001),
                                        ("f32", 600), ("f32", 4099), ("f32", 16500), ("f32", 40000)])
def test_softmax_held_by_a_workgroup_of_values_of_any_size(dtype, cols):
    """The maximum is found without widening a value and exponentials are taken relative to a scaled maximum: rows of one
    sign, of huge values, with infinities, a NaN, and a maximum in the first, the last or a masked place."""
    g = wl.rng(9600 + cols)
    x = (g.standard_normal((12, cols)) * 3).astype(np.float32)
    big = 6.0e4 if dtype == "f16" else 3.0e38
    x[1] = -np.abs(x[1]) - 1  # negative throughout
    x[2] -= 3.0e4  # (a row of large values among which only steps of the type differ)
    x[3] = np.where(g.random(cols) < 0.5, -big, x[3])
    x[4, :] = big
    x[5, cols // 3] = big
    x[6, -1], x[6, 0] = 40.0, 39.0
    x[7, 0] = 70.0
    x[8, : cols - 1] = -np.inf
    x[9, cols // 2:] = -np.inf
    x[10, cols - 2] = np.inf
    x[11, 1] = np.nan
    s = wl.to_storage(x, dtype)
    ref = red.softmax_rows(np.where(np.isfinite(wl.widen(s, dtype)), wl.widen(s, dtype), -np.inf))
    for shift in (0, 1):
        buf = torch.zeros(12 * cols + 8, dtype=TORCH_DTYPE[dtype], device="cuda")
        dx = buf[shift: shift + 12 * cols].view(12, cols)
        dx.copy_(to_gpu(s, dtype))
        dy = torch.full_like(dx, 3.0)
        hb.hidet_softmax_rows(dx, dy)
        torch.cuda.synchronize()
        got = to_f64(dy)
        assert np.isnan(got[10:]).all()
        for i in range(10):
            assert within_bound(oracle.rel_frobenius(got[i:i + 1], ref[i:i + 1]), ref[i:i + 1], dtype), (i, shift)


# Outputs on both sides of 4 MiB, from where on they are stored with the streaming hint unless they are the input: a wavefront's rows,
# a workgroup's and streamed ones; whole chunks, ragged ends, and rows whose chunks are laid on the output's 16-byte grid.
@pytest.mark.parametrize("dtype,rows,cols", [("f16", 4200, 512), ("bf16", 7300, 300), ("f32", 2100, 500), ("f16", 300, 8192), ("f16", 130, 8192),
                                             ("bf16", 48, 50257), ("bf16", 36, 50257), ("f16", 64, 33001), ("f32", 24, 60001),
                                             ("f16", 16, 140001), ("bf16", 3, 140008)])
def test_softmax_of_large_outputs_beside_and_in_place_of_the_input(dtype, rows, cols):
    g = wl.rng(9700 + cols + rows)
    x = wl.to_storage((g.standard_normal((rows, cols)) * 3).astype(np.float32), dtype)
    ref = red.softmax_rows(wl.widen(x, dtype))
    for ld, shift in ((cols, 0), (cols + 3, 1)):
        around = lambda: torch.full((rows * ld + shift + 16,), 7.0, dtype=TORCH_DTYPE[dtype], device="cuda")
        inside = lambda buf: buf[shift: shift + rows * ld].view(rows, ld)[:, :cols]
        src, dst = around(), around()
        inside(src).copy_(to_gpu(x, dtype))
        hb.hidet_softmax_rows(inside(src), inside(dst))
        torch.cuda.synchronize()
        assert torch.equal(inside(src), to_gpu(x, dtype)), "the input is read only"
        err = oracle.rel_frobenius(to_f64(inside(dst)), ref)
        assert within_bound(err, ref, dtype), (ld, err)
        hb.hidet_softmax_rows(inside(src), inside(src))
        torch.cuda.synchronize()
        assert torch.equal(src, dst), "in place: the same bits, and nothing written beside the rows"
        inside(dst).fill_(7.0)
        assert bool((dst == 7.0).all())


# (2.5 KB to a workgroup: 32 rows of 80 bytes, 16 of 160, 8 of 320, 4 of 640)
@pytest.mark.parametrize("dtype,cols,lanes,spread", [("f16", 8, 8, False), ("f16", 39, 8, False), ("bf16", 40, 8, True), ("f32", 30, 8, True),
                                                     ("bf16", 79, 16, False), ("bf16", 100, 16, True), ("f16", 128, 16, True), ("f16", 136, 32, False),
                                                     ("f32", 80, 32, True), ("f16", 300, 64, False), ("f16", 319, 64, False), ("f32", 160, 64, True),
                                                     ("f32", 256, 64, True), ("bf16", 392, 64, True), ("f16", 601, 64, True), ("f32", 700, 64, True)])
def test_softmax_of_rows_that_wavefronts_take_in_turn(dtype, cols, lanes, spread):
    """More than eight rows a wavefront: those of 2.5 KB to a workgroup get more workgroups, the lanes of others (32 and more to a row) meet
    another way, in the same order.  The same bits as from two calls of half as many rows, which are on the other side of the line, beside and
    in place of the input."""
    limit = 8 * 2048 * 256 // lanes
    for rows, softmax, blocks in ((limit, 1, 2048), (limit + 1, 1, 8 * 2048 + 1 if spread else 2048), (limit + 1, 0, 2048)):
        s = hb.hidet_row_schedule({"f16": hb.HIDET_F16, "bf16": hb.HIDET_BF16, "f32": hb.HIDET_F32}[dtype], softmax, rows, cols)
        assert (s["form"], s["threads_per_row"], s["workgroups"]) == (0, lanes, blocks), (rows, softmax, s)
    for rows in (limit, limit + 3):
        x = torch.randn((rows, cols), device="cuda", generator=torch.Generator(device="cuda").manual_seed(rows)).mul_(3).to(TORCH_DTYPE[dtype])
        y, halves = torch.empty_like(x), torch.empty_like(x)
        hb.hidet_softmax_rows(x, y)
        for part in (slice(0, rows // 2), slice(rows // 2, rows)):
            hb.hidet_softmax_rows(x[part], halves[part])
        z = x.clone()
        hb.hidet_softmax_rows(z, z)
        torch.cuda.synchronize()
        assert torch.equal(y, halves) and torch.equal(z, y), rows
        assert not torch.isnan(y).any() and float((y.float().sum(1) - 1).abs().max()) < 2e-2


@pytest.mark.parametrize("dtype,cols", [("f16", 9), ("bf16", 15), ("f16", 17), ("bf16", 31), ("f16", 33), ("f16", 16), ("f32", 11)])
def test_reductions_of_short_rows_that_wavefronts_take_in_turn(dtype, cols):
    """On both sides of eight rows a wavefront, as softmax above: the same bits as from two calls of half as many rows."""
    limit = 8 * 2048 * 32
    for rows in (limit, limit + 3):
        x = torch.randn((rows, cols), device="cuda", generator=torch.Generator(device="cuda").manual_seed(rows)).to(TORCH_DTYPE[dtype])
        for op in (hb.HIDET_REDUCE_SUM, hb.HIDET_REDUCE_MAX, hb.HIDET_REDUCE_MEAN):
            y, halves = torch.full((rows,), float("nan"), device="cuda"), torch.empty((rows,), device="cuda")
            hb.hidet_reduce_rows(x, y, op=op)
            for part in (slice(0, rows // 2), slice(rows // 2, rows)):
                hb.hidet_reduce_rows(x[part], halves[part], op=op)
            d = x.double()
            ref = d.amax(1) if op == hb.HIDET_REDUCE_MAX else d.sum(1) if op == hb.HIDET_REDUCE_SUM else d.mean(1)
            # (fp32 sums of `cols` terms, in any order: each of fewer than `cols` additions rounds by 2^-24 of at most the sum of magnitudes)
            bound = cols * 2.0 ** -23 * d.abs().sum(1)
            torch.cuda.synchronize()
            assert torch.equal(y, halves) and bool(((y.double() - ref).abs() <= bound).all()), (rows, op)


# outputs of 256 MiB, from where on those in place have the streaming hint as well: rows of a wavefront and of a workgroup
@pytest.mark.parametrize("dtype,rows,cols", [("f16", 450000, 300), ("f32", 68000, 1001), ("bf16", 2100, 65003)])
def test_softmax_in_place_of_more_than_the_last_level_cache(dtype, rows, cols):
    x = torch.randn((rows, cols), device="cuda", generator=torch.Generator(device="cuda").manual_seed(cols)).to(TORCH_DTYPE[dtype])
    y = torch.empty_like(x)
    hb.hidet_softmax_rows(x, y)
    some = torch.arange(0, rows, rows // 40, device="cuda")
    ref = red.softmax_rows(to_f64(x[some]))
    hb.hidet_softmax_rows(x, x)
    torch.cuda.synchronize()
    assert torch.equal(x, y)
    assert within_bound(oracle.rel_frobenius(to_f64(y[some]), ref), ref, dtype)


@pytest.mark.parametrize("cols", [2049, 8200, 50257])
def test_softmax_of_maxima_around_the_largest_scale(cols):
    """A running scale serves maxima below 2^16, the difference to the maximum those beyond: bf16 rows whose maximum is next to
    2^16 on either side, of either sign, in one place or three, with values a step below it, at the other end of the range or -inf."""
    rows = []
    for top, below in ((65280.0, 65024.0), (65536.0, 65280.0), (66048.0, 65536.0), (-65280.0, -65536.0), (-65536.0, -66048.0),
                       (-66048.0, -66560.0)):
        for rest in (below, -3.0e38, -np.inf, min(-70000.0, below)):
            for places in ((cols - 1,), (0, cols // 2, cols - 2)):
                x = np.full(cols, rest, dtype=np.float32)
                x[1::3] = below
                x[list(places)] = top
                rows.append(x)
    s = wl.to_storage(np.stack(rows), "bf16")
    assert np.array_equal(wl.widen(s, "bf16")[:, 1], np.stack(rows)[:, 1])  # (all of them are bf16 values)
    ref = red.softmax_rows(wl.widen(s, "bf16"))
    x = to_gpu(s, "bf16")
    y = torch.empty_like(x)
    hb.hidet_softmax_rows(x, y)
    torch.cuda.synchronize()
    # (any two values differ by 256 or more: a share of the maxima is all there is)
    assert float(np.abs(to_f64(y) - ref).max()) <= 2.0 ** -9 and not torch.isnan(y).any()
