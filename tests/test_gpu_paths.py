"""Paths of the kernels that a call is routed to by its sizes, types or alignment, each compared bit for bit with the
general path over the forms it accepts (ragged and odd extents, strides, types), and against writes outside the output."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2408_02897_amd import qmm, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 64          # elements on either side of an output that must stay as they were


def guarded(shape, dtype):
    n = int(np.prod(shape))
    buf = torch.full((n + 2 * GUARD,), -7.0, dtype=dtype, device=DEV)
    return buf, buf[GUARD:GUARD + n].view(shape)


def intact(buf):
    return bool((buf[:GUARD] == -7.0).all()) and bool((buf[-GUARD:] == -7.0).all())


def operands(kind, m, n, k, per_channel, batch=1):
    x = W.student_t((batch, m, k), 4, seed=m + n).to(DEV)
    w = W.normal((batch, n, k), 0.02, seed=k).to(DEV)
    if kind == "bf16":
        return (x, qmm.operand(x, qmm.BF16, is_codes=False)), (w, qmm.operand(w, qmm.BF16, is_codes=False))
    fmt = qmm.FORMATS[kind]
    return qmm.quantized_operand(x, 1, fmt, per_channel)[0], qmm.quantized_operand(w, 1, fmt, per_channel)[0]


# Above 512 tiles of 64 x 64 the call that also returns the accumulators takes the element-by-element epilogue: Y of the two
# calls must agree in every bit (128 x 128 tiles: 1601 x 1563, 1700 x 1411; 256 x 256: the last two).  Smaller outputs are
# the deep-ring kernel's, whose two calls differ in the accumulators alone; its sums are compared in
# test_product_of_few_tiles.  Extents around the tiles, odd ones (rows that start off every vector boundary).
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("kind", ["e4m3", "int8", "bf16"])
@pytest.mark.parametrize("m,n,k", [(1, 1, 16), (127, 130, 144), (129, 255, 128), (257, 129, 272), (200, 203, 400),
                                   (128, 132, 256), (130, 256, 64), (1601, 1563, 272), (1700, 1411, 400),
                                   (4099, 3071, 128), (3842, 3074, 144)])
def test_output_at_edges_and_odd_extents(kind, m, n, k, out_dtype):
    a, b = operands(kind, m, n, k, per_channel=(m + n) % 2 == 1)
    want, _ = qmm.gemm(a, b, out_dtype, want_acc=True)
    buf, y = guarded((1, m, n), out_dtype)
    qmm.gemm(a, b, out_dtype, out=y)
    assert torch.equal(y, want)
    assert intact(buf)


# Either side of the rule between 256 x 256 and 128 x 128 tiles: 170 big tiles (one round of the CUs), and a batch whose big
# tiles fill two rounds badly.
@pytest.mark.parametrize("kind", ["e4m3", "int8", "bf16"])
@pytest.mark.parametrize("batch,m,n,k", [(1, 4200, 2500, 144), (70, 384, 390, 64), (70, 257, 384, 272)])
def test_output_in_big_and_small_tiles(kind, batch, m, n, k):
    a, b = operands(kind, m, n, k, per_channel=True, batch=batch)
    want, _ = qmm.gemm(a, b, torch.bfloat16, want_acc=True)
    buf, y = guarded((batch, m, n), torch.bfloat16)
    qmm.gemm(a, b, torch.bfloat16, out=y)
    assert torch.equal(y, want) and intact(buf)
    if kind == "int8":
        _, acc = qmm.gemm(a, b, want_acc=True)
        exact = a[0][-1].view(torch.int8).double() @ b[0][-1].view(torch.int8).double().t()
        assert torch.equal(acc[-1].double(), exact)


# bfloat16 operands through the kernel whose workgroups stay on their CU (whole tiles, more tiles than workgroups, three
# slabs or more; 512 tiles, 3 slabs: a tile's stores overlap the whole of the next one): the matrix instructions run in
# the same order, so its product equals the other kernel's in every bit.
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("batch,m,n,k", [(1, 4352, 4096, 192), (2, 2304, 4096, 320), (1, 16384, 4096, 256)])
def test_reference_product_in_resident_workgroups(batch, m, n, k, out_dtype):
    a, b = operands("bf16", m, n, k, False, batch)
    want, acc = qmm.gemm(a, b, out_dtype, want_acc=True)
    buf, y = guarded((batch, m, n), out_dtype)
    qmm.gemm(a, b, out_dtype, out=y)
    assert torch.equal(y, want) and intact(buf)
    rows = torch.arange(0, m, 97, device=DEV)
    ref = a[0][-1][rows].double() @ b[0][-1].double().t()
    bound = 1e-5 * (a[0][-1][rows].double().abs() @ b[0][-1].double().abs().t())
    assert bool(((acc[-1][rows].double() - ref).abs() <= bound).all())


# (shape, view): dense, a column slice of a wider matrix, a slice whose rows start off every vector boundary, a batch with gaps
def tensor_form(form, rows, cols, batch, dtype, seed):
    x = W.student_t((batch, rows + 1, cols + 9), 4, seed=seed).to(dtype).to(DEV)
    if dtype == torch.float32:
        x = x * (1.0 + 2.0 ** -20 * torch.arange(x.numel(), device=DEV).view_as(x) % 64)      # mantissas beyond bfloat16's
    if form == "dense":
        return x[:, :rows, :cols].contiguous()
    if form == "sliced":
        return x[:, :rows, :cols]
    if form == "shifted":
        return x[:, :rows, 1:cols + 1]
    flat = x.reshape(-1)[1:1 + batch * rows * cols]                                           # dense, off the 16-byte boundary
    return flat.view(batch, rows, cols)


# Every form against the oracle: step sizes and codes, by the two calls and by the one.  Extents around the vectors (4, 8,
# 16), the lanes of a row in the one-pass kernel (8 .. 256 lanes, 1 .. 8 vectors), the tiles of the transposing pass
# (64 x 128) and the slabs of its step sizes (32 of 128 rows and more).
@pytest.mark.parametrize("mode", [qmm.RTNE, qmm.STOCHASTIC])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("form", ["dense", "sliced", "shifted", "offset"])
@pytest.mark.parametrize("batch,rows,cols,groups,inner", [
    (1, 1, 1, 1, 1), (1, 5, 7, 1, 1), (1, 129, 65, 1, 1), (1, 3, 2048, 1, 1), (1, 2, 4100, 1, 1), (1, 3, 8200, 1, 1), (1, 4230, 33, 1, 1),
    (1, 300, 1031, 1, 1), (6, 40, 72, 3, 1), (6, 70, 96, 3, 2), (4, 33, 50, 4, 1), (2, 20, 40, 5, 1), (12, 130, 64, 4, 1)])
def test_scale_and_quantize_of_every_form(batch, rows, cols, groups, inner, form, dtype, mode):
    x = tensor_form(form, rows, cols, batch, dtype, seed=rows * 7 + cols)
    xn = x.float().cpu().numpy()
    for fmt in (qmm.E4M3, qmm.INT8):
        for axis in (0, 1):
            for per_channel in (False, True):
                kw = dict(per_channel=per_channel, batch_groups=groups, batch_inner=inner)
                want_d = O.scale(xn, axis, fmt, per_channel, groups, inner)
                want_c = O.quantize(xn, axis, fmt, want_d, per_channel, groups, mode, 77, 0, inner)
                d = qmm.scale(x, axis, fmt, **kw)
                c = qmm.quantize(x, axis, fmt, d, mode=mode, seed=77, **kw)
                c1, d1 = qmm.scale_quantize(x, axis, fmt, mode=mode, seed=77, **kw)
                assert np.array_equal(d.cpu().numpy().view(np.uint32), want_d.view(np.uint32)), (fmt, axis, per_channel)
                assert np.array_equal(c.cpu().numpy(), want_c), (fmt, axis, per_channel)
                assert torch.equal(d1.view(torch.int32), d.view(torch.int32)) and torch.equal(c1, c), (fmt, axis, per_channel)


# The same forms recorded into a graph, where the single call is made of separate launches that the calls above no longer take: every
# replay against the oracle.
@pytest.mark.parametrize("mode", [qmm.RTNE, qmm.STOCHASTIC])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("form", ["dense", "sliced", "shifted", "offset"])
def test_recorded_scale_quantize_of_every_form(form, dtype, mode):
    shapes = [(1, 1, 1, 1, 1), (1, 5, 7, 1, 1), (1, 129, 65, 1, 1), (1, 3, 2048, 1, 1), (1, 2, 4100, 1, 1), (1, 3, 8200, 1, 1), (1, 4230, 33, 1, 1),
              (1, 300, 1031, 1, 1), (6, 40, 72, 3, 1), (6, 70, 96, 3, 2), (4, 33, 50, 4, 1), (2, 20, 40, 5, 1), (12, 130, 64, 4, 1)]
    xs = [tensor_form(form, r, c, b, dtype, seed=r * 7 + c) for b, r, c, _, _ in shapes]
    cases = [(x, fmt, axis, pc, groups, inner) for x, (_, _, _, groups, inner) in zip(xs, shapes) for fmt in (qmm.E4M3, qmm.INT8)
             for axis in (0, 1) for pc in (False, True)]

    def calls():
        return [qmm.scale_quantize(x, axis, fmt, mode=mode, seed=77, per_channel=pc, batch_groups=groups, batch_inner=inner)
                for x, fmt, axis, pc, groups, inner in cases]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        calls()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = calls()
    for replay in range(3):
        for x in xs:
            x.mul_(-0.75)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        host = {id(x): x.float().cpu().numpy() for x in xs}
        for (x, fmt, axis, pc, groups, inner), (c, d) in zip(cases, got):
            want_d = O.scale(host[id(x)], axis, fmt, pc, groups, inner)
            want_c = O.quantize(host[id(x)], axis, fmt, want_d, pc, groups, mode, 77, 0, inner)
            assert np.array_equal(d.cpu().numpy().view(np.uint32), want_d.view(np.uint32)), (replay, x.shape, fmt, axis, pc)
            assert np.array_equal(c.cpu().numpy(), want_c), (replay, x.shape, fmt, axis, pc)


# Sizes where the single call changes its way: partial maxima folded by the quantize pass (up to 1024 of a group) or not, the
# large tensors' one-launch maximum (2^24 elements), empty tensors, groups without a matrix, NaN and infinity.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("shape,axis,per_channel,groups", [
    ((1, 2048, 4096), 1, False, 1), ((1, 4096, 4096), 1, False, 1), ((1, 1025, 100), 1, False, 1), ((40, 64, 512), 1, False, 2),
    ((512, 33, 64), 1, False, 16), ((3, 600, 200), 0, True, 3), ((3, 600, 200), 0, True, 1), ((0, 8, 16), 1, False, 2),
    ((1, 0, 16), 0, True, 1), ((1, 70000, 24), 1, True, 1), ((1, 12, 9000), 1, True, 1),
    ((512, 64, 512), 0, True, 512), ((512, 62, 516), 0, False, 8), ((3, 130, 3001), 1, True, 3), ((40, 300, 67), 0, True, 40)])
def test_scale_quantize_equals_the_two_calls(shape, axis, per_channel, groups, dtype):
    x = W.student_t(shape, 4, seed=3).to(dtype).to(DEV)
    if x.numel() > 4096:
        x.view(-1)[17] = float("inf")
        if groups > 1:
            x.view(-1)[-3] = float("nan")
    kw = dict(per_channel=per_channel, batch_groups=groups)
    for fmt in (qmm.INT8, qmm.E4M3, qmm.E5M2):
        d = qmm.scale(x, axis, fmt, **kw)
        c = qmm.quantize(x, axis, fmt, d, seed=5, mode=qmm.STOCHASTIC, **kw)
        c1, d1 = qmm.scale_quantize(x, axis, fmt, mode=qmm.STOCHASTIC, seed=5, **kw)
        assert torch.equal(d1.view(torch.int32), d.view(torch.int32)) and torch.equal(c1, c)


# every code, rows around the pieces a wavefront takes (4 x 64 vectors of 4 or 8), odd rows and step sizes at each level
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("batch,rows,k,groups", [(1, 1, 256, 1), (1, 3, 1023, 1), (1, 2, 1025, 1), (4, 5, 2049, 2), (6, 7, 33, 3), (2, 70, 4096, 1)])
def test_dequantize_of_every_form(batch, rows, k, groups, out_dtype):
    rng = np.random.default_rng(k)
    codes = rng.integers(0, 256, (batch, rows, k), dtype=np.uint8)
    for fmt in (qmm.INT8, qmm.E4M3, qmm.E5M2):
        for per_channel in (False, True):
            d = rng.uniform(1e-3, 2.0, groups * (rows if per_channel else 1)).astype(np.float32)
            want = torch.from_numpy(O.dequantize_codes(codes, fmt, d, per_channel, groups)).to(out_dtype)
            buf, out = guarded((batch, rows, k), out_dtype)
            qmm.dequantize(torch.from_numpy(codes).to(DEV), fmt, torch.from_numpy(d).to(DEV), per_channel, groups, out=out)
            got, nan = out.cpu(), want.isnan()
            assert torch.equal(got.isnan(), nan) and torch.equal(got[~nan], want[~nan]) and intact(buf)


# Outputs of at most 512 tiles of 64 x 64 (rings of eight and of three slabs): contractions shorter and longer than the ring,
# partial last slabs, edges of the tiles, a batch, step sizes at each level.  INT8: whole numbers against an integer product;
# the others: against the same rows inside a product of more rows, which runs in the 128 x 128 tiles with the same order of
# additions, so in every bit.  (`row` = bytes of a row, below sixteen slabs of 128: from there on the small product, but
# not the large one, is split along K.)
@pytest.mark.parametrize("kind", ["e4m3", "int8", "bf16"])
@pytest.mark.parametrize("batch,m,n,row", [(1, 1, 1, 16), (1, 63, 65, 48), (1, 64, 64, 1024), (2, 129, 70, 1168), (1, 65, 2047, 144),
                                           (1, 1000, 1031, 784), (3, 400, 700, 1920), (1, 2048, 1024, 128)])
def test_product_of_few_tiles(kind, batch, m, n, row):
    k = row // 2 if kind == "bf16" else row
    a, b = operands(kind, m, n, k, per_channel=(m % 2 == 1), batch=batch)
    buf, acc = guarded((batch, m, n), torch.int32 if kind == "int8" else torch.float32)
    y = torch.empty((batch, m, n), dtype=torch.float32, device=DEV)
    qmm.gemm(a, b, out=y, acc_out=acc)
    assert intact(buf)
    if kind == "int8":
        want = a[0].view(torch.int8).double() @ b[0].view(torch.int8).double().transpose(1, 2).contiguous()
        assert torch.equal(acc.double(), want)
    else:
        rows = 6144                                        # more than 512 tiles for every n here
        wide = [torch.zeros((batch, rows, k), dtype=a[0].dtype, device=DEV), torch.zeros((batch, max(n, 700), k), dtype=b[0].dtype, device=DEV)]
        wide[0][:, :m], wide[1][:, :n] = a[0], b[0]
        one = torch.ones(1, device=DEV)
        ops = [(t, qmm.operand(t, o[1].format, one, is_codes=kind != "bf16")) for t, o in zip(wide, (a, b))]
        _, acc_wide = qmm.gemm(ops[0], ops[1], want_acc=True)
        assert torch.equal(acc, acc_wide[:, :m, :n])
    alone = torch.empty_like(y)
    qmm.gemm(a, b, out=alone)
    assert torch.equal(alone, y)


# Contractions in `ranges` ranges of eight slabs, whose sums a second kernel adds (four at a time, then the one to three left; a
# matrix of the batch its own row of workgroups): rows of whole and partial quads, an element, step sizes at each level.
@pytest.mark.parametrize("batch,m,n,ranges,per_channel,groups,inner", [
    (1, 64, 64, 2, False, 1, 0), (1, 65, 63, 3, True, 1, 0), (1, 130, 101, 4, False, 1, 0), (3, 40, 36, 5, True, 3, 0), (6, 33, 35, 6, False, 2, 3),
    (7, 32, 20, 7, True, 2, 2), (1, 1, 1, 8, False, 1, 0), (2, 64, 66, 9, False, 1, 5), (5, 17, 300, 10, True, 2, 1)])
def test_sum_of_split_ranges(batch, m, n, ranges, per_channel, groups, inner):
    k = ranges * 1024
    a, b = (torch.randint(-127, 128, (batch, r, k), generator=torch.Generator().manual_seed(r + k), dtype=torch.int32).to(torch.int8).to(DEV) for r in (m, n))
    steps = [torch.rand(groups * (r if per_channel else 1), generator=torch.Generator().manual_seed(r)).add_(0.01).to(DEV) for r in (m, n)]
    pair = [(t.view(torch.uint8), qmm.operand(t.view(torch.uint8), qmm.INT8, d, per_channel, groups, batch_inner=inner)) for t, d in zip((a, b), steps)]
    assert qmm.lib().qmm_gemm_workspace_size(ctypes.byref(pair[0][1]), ctypes.byref(pair[1][1]), batch, m, n, k) == ranges * batch * m * n * 4
    exact = a.double() @ b.double().transpose(1, 2).contiguous()
    group = [i // max(inner, 1) % groups for i in range(batch)]
    da, db = (d.view(groups, -1)[group] for d in steps)
    want = (exact.float() * da[:, :, None]) * db[:, None, :]
    for dtype in (torch.float32, torch.bfloat16):
        ybuf, y = guarded((batch, m, n), dtype)
        abuf, acc = guarded((batch, m, n), torch.int32)
        qmm.gemm(*pair, out=y, acc_out=acc)
        assert torch.equal(acc.double(), exact) and torch.equal(y, want.to(dtype)) and intact(ybuf) and intact(abuf)


# Tall outputs at most 64 wide: B in LDS (up to eight slabs of K) and, beyond, from memory; odd numbers of slabs, a partial
# last one, wavefronts without a row.  INT8 against the integer product; E4M3 against the same columns inside a product of 96,
# which runs in the LDS kernels with the same order of additions.
@pytest.mark.parametrize("kind", ["e4m3", "int8"])
@pytest.mark.parametrize("batch,m,n,k", [(60, 600, 64, 512), (60, 577, 40, 144), (60, 600, 1, 16), (60, 600, 64, 1024), (1, 40000, 63, 400), (60, 600, 64, 1040),
                                          (300, 191, 64, 512), (300, 192, 33, 272), (600, 64, 64, 1024), (600, 65, 50, 128)])
def test_tall_product(kind, batch, m, n, k):
    a, b = operands(kind, m, n, k, per_channel=(k % 3 == 0), batch=batch)
    y, acc = qmm.gemm(a, b, torch.bfloat16, want_acc=True)
    buf, alone = guarded((batch, m, n), torch.bfloat16)
    qmm.gemm(a, b, out=alone)
    assert torch.equal(alone, y) and intact(buf)
    if kind == "int8":
        exact = a[0].view(torch.int8).double() @ b[0].view(torch.int8).double().transpose(1, 2).contiguous()
        assert torch.equal(acc.double(), exact)
    else:
        wide = torch.zeros((batch, 96, k), dtype=torch.uint8, device=DEV)
        wide[:, :n] = b[0]
        one = torch.ones(1, device=DEV)
        _, acc_wide = qmm.gemm((a[0], qmm.operand(a[0], qmm.E4M3, one)), (wide, qmm.operand(wide, qmm.E4M3, one)), want_acc=True)
        assert torch.equal(acc, acc_wide[:, :, :n])


# Empty tensors: every group's step size is 1, also where matrices share a group in runs (batch_inner), by both calls.
@pytest.mark.parametrize("inner", [1, 2, 5])
@pytest.mark.parametrize("groups", [1, 3])
@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("shape", [(0, 8, 16), (4, 0, 16), (4, 8, 0)])
def test_empty_tensors_get_step_size_one(shape, per_channel, groups, inner):
    x = torch.zeros(shape, dtype=torch.bfloat16, device=DEV)
    for axis in (0, 1):
        kw = dict(per_channel=per_channel, batch_groups=groups, batch_inner=inner)
        count = groups * (shape[1 if axis == 1 else 2] if per_channel else 1)
        if count == 0:                                     # no step size to write, and no place to write it to
            continue
        d = qmm.scale(x, axis, qmm.E4M3, **kw)
        c1, d1 = qmm.scale_quantize(x, axis, qmm.E4M3, **kw)
        assert d.numel() == count
        assert c1.numel() == 0 and bool((d == 1.0).all()) and bool((d1 == 1.0).all())


# Lines around every number of lanes a short line gets (1 .. 64 lanes, two halves) and the first long one, with a step size
# per row, per run of matrices and per group; groups beyond the batch; from 4096 wavefronts of work on, four vectors a lane.
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("batch,rows,k,groups,inner", [
    (1, 300, 1, 1, 1), (1, 259, 8, 1, 1), (3, 70, 9, 3, 1), (6, 45, 16, 3, 2), (4, 33, 31, 2, 1), (2, 67, 64, 1, 1), (5, 13, 65, 9, 1),
    (1, 37, 256, 1, 1), (3, 5, 257, 2, 1), (2, 9, 512, 2, 1), (2, 5, 513, 1, 1), (1, 7, 1024, 1, 1), (6, 1, 1025, 3, 2), (700, 2, 3, 350, 2),
    (1, 700000, 3, 1, 1), (2, 2600, 300, 2, 1), (1, 3000, 600, 1, 1), (3, 1500, 1100, 2, 2)])
def test_dequantize_of_short_lines(batch, rows, k, groups, inner, out_dtype):
    rng = np.random.default_rng(k + rows)
    codes = rng.integers(0, 256, (batch, rows, k), dtype=np.uint8)
    group = (np.arange(batch) // inner) % groups
    for fmt in (qmm.INT8, qmm.E4M3, qmm.E5M2):
        value = codes.view(np.int8).astype(np.float32) if fmt == qmm.INT8 else O.decode(fmt, codes).astype(np.float32)
        for per_channel in (False, True):
            d = rng.uniform(1e-3, 2.0, (groups, rows if per_channel else 1)).astype(np.float32)
            want = torch.from_numpy(value * d[group][:, :, None]).to(out_dtype)
            buf, out = guarded((batch, rows, k), out_dtype)
            qmm.dequantize(torch.from_numpy(codes).to(DEV), fmt, torch.from_numpy(d.reshape(-1)).to(DEV), per_channel, groups,
                           out=out, batch_inner=inner)
            got, nan = out.cpu(), want.isnan()
            assert torch.equal(got.isnan(), nan) and torch.equal(got[~nan], want[~nan]) and intact(buf), (fmt, per_channel)


# Rows that contract, around every number of lanes a row gets (1 .. 64, two halves, pieces of long rows), below and above the
# 4096 wavefronts from which a lane takes two vectors, with values that only some wavefronts hold: NaN, infinities, zeros and
# magnitudes below every format's normal range.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("form", ["dense", "shifted"])
@pytest.mark.parametrize("batch,rows,cols", [(1, 70, 1), (1, 33, 3), (2, 130, 20), (1, 90000, 9), (1, 40000, 44), (3, 1700, 300), (1, 2300, 700),
                                             (2, 1200, 1031), (1, 3, 40001), (1, 40, 9000), (1, 1, 140001)])
def test_quantize_of_short_and_long_rows(batch, rows, cols, form, dtype):
    x = tensor_form(form, rows, cols, batch, dtype, seed=rows + cols).clone() if form == "dense" else tensor_form(form, rows, cols, batch, dtype, rows)
    for i, v in enumerate([float("nan"), float("inf"), -float("inf"), 0.0, 1e-7, -3e-6, 2e-4, -1e-30]):
        x[-1, rows // 2 + i // cols if rows > 40 else rows // 2, (i * 5) % cols] = v
    xn = x.float().cpu().numpy()
    for per_channel in (True, False):
        count = rows if per_channel else 1
        d = np.random.default_rng(cols).uniform(1e-3, 1e-1, count).astype(np.float32)
        for fmt in (qmm.E4M3, qmm.INT8, qmm.E5M2):
            for mode, offset in ((qmm.RTNE, 0), (qmm.STOCHASTIC, 0), (qmm.STOCHASTIC, 7)):
                want = O.quantize(xn, 1, fmt, d, per_channel, 1, mode, 77, offset, 1)
                buf = torch.full((want.size + 2 * GUARD,), 77, dtype=torch.uint8, device=DEV)
                out = buf[GUARD:GUARD + want.size].view(want.shape)
                qmm.quantize(x, 1, fmt, torch.from_numpy(d).to(DEV), per_channel, 1, mode, 77, offset, out=out)
                assert np.array_equal(out.cpu().numpy(), want), (per_channel, fmt, mode, offset)
                assert bool((buf[:GUARD] == 77).all()) and bool((buf[-GUARD:] == 77).all())


# Rows that are contracted over: one thread per code, tiles of 16, 64 and 128 columns, ragged both ways, columns that do and
# do not start blocks of the random generator.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("form", ["dense", "shifted"])
@pytest.mark.parametrize("batch,rows,cols", [(1, 33, 70), (3, 40, 21), (1, 700, 401), (5, 260, 262), (1, 131, 2101), (1, 1300, 1601), (2, 1031, 1203),
                                             (64, 9, 4200), (64, 12, 4196),
                                             (64, 13, 4196), (700, 4, 401), (1, 12, 40001), (1, 16, 40003), (64, 20, 4196), (64, 21, 4200)])
def test_quantize_of_contracted_rows(batch, rows, cols, form, dtype):
    x = tensor_form(form, rows, cols, batch, dtype, seed=rows + cols).clone() if form == "dense" else tensor_form(form, rows, cols, batch, dtype, rows)
    for i, v in enumerate([float("nan"), float("inf"), -float("inf"), 0.0, 1e-7, -3e-6, 2e-4, -1e-30]):
        x[-1, i % rows, cols // 2 + i // rows] = v
    xn = x.float().cpu().numpy()
    for per_channel in (True, False):
        d = np.random.default_rng(cols).uniform(1e-3, 1e-1, cols if per_channel else 1).astype(np.float32)
        for fmt in (qmm.E4M3, qmm.INT8, qmm.E5M2):
            for mode, offset in ((qmm.RTNE, 0), (qmm.STOCHASTIC, 0), (qmm.STOCHASTIC, 6)):
                want = O.quantize(xn, 0, fmt, d, per_channel, 1, mode, 77, offset, 1)
                buf = torch.full((want.size + 2 * GUARD,), 77, dtype=torch.uint8, device=DEV)
                out = buf[GUARD:GUARD + want.size].view(want.shape)
                qmm.quantize(x, 0, fmt, torch.from_numpy(d).to(DEV), per_channel, 1, mode, 77, offset, out=out)
                assert np.array_equal(out.cpu().numpy(), want), (per_channel, fmt, mode, offset)
                assert bool((buf[:GUARD] == 77).all()) and bool((buf[-GUARD:] == 77).all())


# Maxima per column: workgroups of 4, 8, 16 and 32 vectors, slabs of one trip and of many, ragged ends; tall tensors, whose
# second kernel gives a channel many lanes; groups over a batch.  And short rows off every boundary.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("form", ["dense", "sliced", "shifted"])
@pytest.mark.parametrize("batch,rows,cols,groups,inner", [(1, 70001, 20, 1, 1), (1, 40000, 64, 1, 1), (1, 129, 3, 1, 1), (3, 5000, 33, 3, 1), (6, 700, 130, 2, 2),
                                                          (1, 1100, 4301, 1, 1), (1, 8, 5000, 1, 1), (1, 257, 129, 1, 1), (40, 300, 9, 5, 1)])
def test_scale_per_channel_of_tall_and_wide_tensors(batch, rows, cols, groups, inner, form, dtype):
    x = tensor_form(form, rows, cols, batch, dtype, seed=rows + cols)
    xn = x.float().cpu().numpy()
    for axis in (0, 1):
        d = qmm.scale(x, axis, qmm.E4M3, True, groups, batch_inner=inner)
        want = O.scale(xn, axis, qmm.E4M3, True, groups, inner)
        assert np.array_equal(d.cpu().numpy().view(np.uint32), want.view(np.uint32)), axis
        c1, d1 = qmm.scale_quantize(x, axis, qmm.E4M3, True, groups, batch_inner=inner)
        assert torch.equal(d1, d) and torch.equal(c1, qmm.quantize(x, axis, qmm.E4M3, d, True, groups, batch_inner=inner)), axis
        size = qmm.lib().qmm_scale_workspace_size(ctypes.byref(qmm.tensor_desc(x, axis)), ctypes.byref(qmm.granularity(True, groups, inner)))
        if size <= 1 << 20:
            assert torch.equal(qmm.scale_static(x, axis, qmm.E4M3, True, groups, batch_inner=inner), d)


# The hardware converter against the oracle's integer arithmetic: every bfloat16 pattern, and binary32 values of every upper
# half with lower halves at and around the ties; step size 1, so the code is the rounded value itself.
@pytest.mark.parametrize("fmt", [qmm.E4M3, qmm.E5M2, qmm.INT8])
def test_nearest_even_of_every_upper_half(fmt):
    upper = np.arange(65536, dtype=np.uint32) << 16
    one = torch.ones(1, device=DEV)
    bf = torch.from_numpy((upper >> 16).astype(np.uint16).view(np.int16)).view(torch.bfloat16).view(1, 1, -1)
    for dtype_x, xn in ((bf, upper.view(np.float32)[None, None]),
                        *((None, (upper | np.uint32(low)).view(np.float32)[None, None])
                          for low in (1, 0x2AAA, 0x7FFF, 0x8000, 0x8001, 0xFFFF))):
        x = dtype_x.to(DEV) if dtype_x is not None else torch.from_numpy(xn.copy()).to(DEV)
        for axis in (1, 0):
            codes = qmm.quantize(x, axis, fmt, one).cpu().numpy()
            assert np.array_equal(codes, O.quantize(xn, axis, fmt, np.ones(1, np.float32)))


# Every quotient of the metric pass by itself: a call of one trip of one workgroup whose other elements have a quotient of 0, so
# that the maximum (and the sum) is the quotient under test, which must equal the IEEE quotient bit for bit; the plain path
# (no special element in the wavefront) over exponents and mantissas of binary32, with and without denominators.
def test_metric_quotients_bit_for_bit():
    rng = np.random.default_rng(9)
    cases = 400
    r = (rng.integers(0, 1 << 23, cases).astype(np.uint32) | (rng.integers(64, 190, cases).astype(np.uint32) << 23)).view(np.float32)
    d = (rng.integers(0, 1 << 23, cases).astype(np.uint32) | (rng.integers(64, 190, cases).astype(np.uint32) << 23)).view(np.float32)
    y = (rng.integers(0, 1 << 23, cases).astype(np.uint32) | (rng.integers(64, 190, cases).astype(np.uint32) << 23)).view(np.float32)
    r[::3] = np.abs(y[::3] * (1 + rng.uniform(-1e-3, 1e-3, r[::3].size)).astype(np.float32))       # small errors
    n = 2048
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    out = torch.empty((cases, 2, 16), dtype=torch.float64, device=DEV)
    rest_r, rest_d = np.float32(3.7), np.float32(0.9)
    for i in range(cases):
        at = int(rng.integers(0, n))
        yy, rr, dd = np.full(n, rest_r), np.full(n, rest_r), np.full(n, rest_d)
        yy[at], rr[at], dd[at] = y[i], r[i], d[i]
        ty, tr, td = (torch.from_numpy(v).to(DEV) for v in (yy, rr, dd))
        qmm.metric(ty, tr, out=out[i, 0], workspace=ws)
        qmm.metric(ty, tr, td, out=out[i, 1], workspace=ws)
    got = out.cpu().numpy()
    e = np.abs(y.astype(np.float64) - r.astype(np.float64))
    q, qb = e / r.astype(np.float64), e / d.astype(np.float64)
    for f, want in ((6, q), (7, q)):
        assert np.array_equal(got[:, 0, f], want) and np.array_equal(got[:, 1, f], want)
    for f, want in ((9, qb), (10, qb)):
        assert np.array_equal(got[:, 1, f], want)


# Many matrices of 2^27 codes and more in all: the same codes, in one call with the step sizes stored streaming.
def test_quantize_of_a_large_batch_equals_its_parts():
    x = torch.randn((513, 512, 512), generator=torch.Generator(device=DEV).manual_seed(5), device=DEV).bfloat16()
    d = qmm.scale(x, 1, qmm.E4M3, batch_groups=513)
    for mode in (qmm.RTNE, qmm.STOCHASTIC):
        c = qmm.quantize(x, 1, qmm.E4M3, d, batch_groups=513, mode=mode, seed=3)
        both, d1 = qmm.scale_quantize(x, 1, qmm.E4M3, batch_groups=513, mode=mode, seed=3)
        assert torch.equal(both, c) and torch.equal(d1, d), mode
        for lo, hi in ((0, 200), (200, 513)):
            part = qmm.quantize(x[lo:hi], 1, qmm.E4M3, d[lo:hi].clone(), batch_groups=hi - lo, mode=mode, seed=3, offset=lo * 512 * 512)
            assert torch.equal(c[lo:hi], part), (mode, lo)
