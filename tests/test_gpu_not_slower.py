"""Calls that take one launch by exchanging values while it runs must not cost a multiple of the separate launches anywhere in
their range.  The separate launches are what a call recorded into a graph takes, so the two forms are timed in turn in one process;
the bounds lie between what was measured with the fault that a test is for and what is measured without."""
import statistics

import pytest
import torch

from paper_2408_02897_amd import qmm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def recorded(call):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    return graph.replay


def microseconds(call, n):
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(n):
        call()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) * 1e3 / n


def eager_over_recorded(call, n, reps=7):
    replay = recorded(call)
    microseconds(call, n), microseconds(replay, n)
    times = [(microseconds(call, n), microseconds(replay, n)) for _ in range(reps)]
    return statistics.median(t[0] for t in times) / statistics.median(t[1] for t in times)


def scale_call(x, **kw):
    ws = qmm._workspace(2 << 20, DEV)
    out = torch.empty(kw.get("batch_groups", 1), device=DEV)
    return (lambda: qmm.scale(x, 1, qmm.E4M3, out=out, workspace=ws, **kw)), out


# The workgroups of a long pass end more than 50 us apart: a folding workgroup that waited no longer began to read the
# others' slices again, alone (8 GB: 1.32 times the separate launches; now 1.0).
def test_step_size_of_many_gigabytes():
    x = torch.empty((1, 1 << 20, 4096), dtype=torch.bfloat16, device=DEV).normal_()
    x[0, 12345, 77] = -300.0
    call, out = scale_call(x)
    ratio = max(eager_over_recorded(call, 10) for _ in range(2))
    assert float(out) == torch.tensor(300.0 / 448.0).item()
    assert ratio < 1.1, ratio


def side_by_side(a, na, b, nb, reps=5):
    """Time until na calls of `a` on one stream and nb of `b` on another are done over what they take one after the other."""
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()

    def both():
        torch.cuda.synchronize()
        e0, ea, eb = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        e0.record(sa)
        sb.wait_event(e0)
        for i in range(max(na, nb)):
            if i < na:
                with torch.cuda.stream(sa):
                    a()
            if i < nb:
                with torch.cuda.stream(sb):
                    b()
        ea.record(sa), eb.record(sb)
        torch.cuda.synchronize()
        return max(e0.elapsed_time(ea), e0.elapsed_time(eb)) * 1e3
    alone = na * microseconds(a, na) + nb * microseconds(b, nb)
    both()
    return statistics.median(both() for _ in range(reps)) / alone


# Calls whose workgroups wait for one another, planned for the whole chip, beside other work that holds part of it: found and formed
# what does not come, results as ever.  (Two of them side by side took 2 to 30 times what they take in turn, one beside a product of half
# the CUs 2 to 4 times; now 1.0 and 1.1 to 1.3.)
@pytest.mark.parametrize("axis,shape,kw", [(1, (1, 16384, 1024), {}), (0, (1, 16384, 1024), {}), (1, (512, 512, 64), dict(batch_groups=16)),
                                           (0, (1, 4096, 3072), dict(per_channel=True))])
def test_scale_quantize_beside_other_work(axis, shape, kw):
    gen = torch.Generator(device=DEV).manual_seed(3)
    x = torch.randn(shape, generator=gen, device=DEV).bfloat16()
    other = torch.randn((1, 16384, 1024), generator=gen, device=DEV).bfloat16()
    want_d = qmm.scale(x, axis, qmm.E4M3, **kw)
    want_c = qmm.quantize(x, axis, qmm.E4M3, want_d, **kw)
    one = torch.ones(1, device=DEV)
    a, b = ((t, qmm.operand(t, qmm.E4M3, one)) for t in (torch.randint(0, 100, (1, r, 8192), dtype=torch.uint8, device=DEV) for r in (2048, 4096)))
    y = torch.empty((1, 2048, 4096), dtype=torch.bfloat16, device=DEV)
    got = []

    def call():
        got.append(qmm.scale_quantize(x, axis, qmm.E4M3, **kw))
        if len(got) > 4:
            got.pop(0)
    for name, work, n in (("another call", lambda: qmm.scale_quantize(other, 1, qmm.E4M3), 40), ("a product", lambda: qmm.gemm(a, b, out=y), 20)):
        ratio = side_by_side(work, n, call, 40)
        torch.cuda.synchronize()
        for c, d in got:
            assert torch.equal(d, want_d) and torch.equal(c, want_c), name
        assert ratio < 2.0, (name, ratio)


# Codes quantized with step sizes that are there are kept where the product behind reads them: a batch quantized in one call and in two
# halves, the product behind it (streaming codes from 2^27 on: 1.07; now 0.97).
def test_codes_are_kept_for_the_product():
    gen = torch.Generator(device=DEV).manual_seed(4)
    batch, s = 128, 1024
    w = [torch.randn((batch, s, s), generator=gen, device=DEV).bfloat16() for _ in range(2)]
    d = qmm.scale(w[0], 1, qmm.E4M3, batch_groups=batch)
    b, _ = qmm.quantized_operand(torch.randn((batch, 64, s), generator=gen, device=DEV).bfloat16(), 1, qmm.E4M3)
    codes = torch.empty((batch, s, s), dtype=torch.uint8, device=DEV)
    a, y = (codes, qmm.operand(codes, qmm.E4M3, d, batch_groups=batch)), torch.empty((batch, s, 64), dtype=torch.bfloat16, device=DEV)

    def chain(parts):
        n = batch // parts
        for x in w:
            for i in range(0, batch, n):
                qmm.quantize(x[i:i + n], 1, qmm.E4M3, d[i:i + n], batch_groups=n, out=codes[i:i + n])
            qmm.gemm(a, b, out=y)

    def ratio():
        times = [(microseconds(lambda: chain(1), 5), microseconds(lambda: chain(2), 5)) for _ in range(9)]
        return statistics.median(t[0] for t in times) / statistics.median(t[1] for t in times)
    ratio()
    assert min(ratio() for _ in range(3)) < 1.02


# Code rows shorter than a line and with a remainder leave by the L2, which puts their parts together: 127 contracted rows over 128 (past
# it 1.33, now 1.10).
def test_short_ragged_code_rows():
    xs = {k: [torch.randn((1024, k, 64), device=DEV).bfloat16() for _ in range(3)] for k in (127, 128)}
    keep = [None] * 4

    def call(k):
        for i, x in enumerate(xs[k]):
            keep[i] = qmm.scale_quantize(x, 0, qmm.E4M3, batch_groups=16)

    def ratio():
        times = [(microseconds(lambda: call(127), 30), microseconds(lambda: call(128), 30)) for _ in range(7)]
        return statistics.median(t[0] for t in times) / statistics.median(t[1] for t in times)
    ratio()
    assert min(ratio() for _ in range(3)) < 1.2


# Values and codes whose rows or matrices are off a line's boundary, beyond what the caches merge past the L2: extents around a
# line's multiple (past the L2 1.33 and 1.05, now 1.15 and 0.97).
@pytest.mark.parametrize("call,whole,ragged,bound", [("dequantize", (1, 65536, 1024), (1, 65536, 1031), 1.25), ("quantize", (128, 1, 1000064), (128, 1, 1000016), 1.015)])
def test_large_ragged_outputs(call, whole, ragged, bound):
    def prepared(shape):
        codes = [torch.randint(0, 100, shape, dtype=torch.uint8, device=DEV) for _ in range(3)]
        if call == "dequantize":
            d, out = torch.rand(shape[1], device=DEV), [torch.empty(shape, device=DEV) for _ in range(3)]
            return lambda: [qmm.dequantize(c, qmm.E4M3, d, True, 1, out=o) for c, o in zip(codes, out)]
        d, x = torch.ones(shape[0], device=DEV), [c.bfloat16() for c in codes]
        return lambda: [qmm.quantize(v, 1, qmm.E4M3, d, batch_groups=shape[0], out=c) for v, c in zip(x, codes)]
    a, b = prepared(ragged), prepared(whole)

    def ratio():
        times = [(microseconds(a, 10), microseconds(b, 10)) for _ in range(7)]
        return statistics.median(t[0] for t in times) / statistics.median(t[1] for t in times)
    ratio()
    assert min(ratio() for _ in range(3)) < bound


# Step sizes per column of a tall tensor: every workgroup of a strip reads the maxima of all (separate launches 24 us, by way of a
# thousand small workgroups 92, of 250 large ones 16).
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_step_sizes_per_column_of_a_tall_tensor(dtype):
    xs = [torch.randn((1, 128000, 64), device=DEV).to(dtype) for _ in range(3)]
    keep = [None] * 4

    def call():
        for i, x in enumerate(xs):
            keep[i] = qmm.scale_quantize(x, 0, qmm.E4M3, per_channel=True)
    assert eager_over_recorded(call, 10) < 1.2


# The error sums of large tensors take two launches, which share more of their time than an exchange within one costs (one launch
# 1.04, now 1.00).
def test_error_sums():
    y = [torch.randn(1 << 23, device=DEV).bfloat16() for _ in range(3)]
    ref = [t.float() for t in y]
    out, ws = torch.empty(16, dtype=torch.float64, device=DEV), qmm._workspace(qmm.lib().qmm_metric_workspace_size(1 << 23), DEV)

    def call():
        for t, r in zip(y, ref):
            qmm.metric(t, r, out=out, workspace=ws)
    assert min(eager_over_recorded(lambda: [call() for _ in range(8)], 4) for _ in range(4)) < 1.03
