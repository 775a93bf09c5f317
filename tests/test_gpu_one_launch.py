"""Calls that take one launch by exchanging values while they run, against their forms of several launches.
qmm_scale_quantize (csrc/qmm_resident.hip: slices in registers, their maxima on a board): the
step sizes and codes of qmm_scale and qmm_quantize, bit for bit, over the forms the rule accepts -- dense and strided rows,
both axes, groups and runs of matrices, one step size per column, both types and rounding modes, sizes around each slice
variant --, whether the workgroups find one another's maxima or form them themselves, under capture, and with several
streams on the ring of boards."""
import ctypes

import pytest
import torch

from oracle import oracle as O
from paper_2408_02897_amd import qmm, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 64
FOREVER = 0xFFFFFFFF


def tensor(shape, dtype, seed, pad=0, shift=0):
    b, r, c = shape
    x = torch.randn((b, r, c + pad + shift), generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV).to(dtype)
    return x[:, :, shift:shift + c]


def two_calls(x, axis, fmt, mode, offset, kw):
    d = qmm.scale(x, axis, fmt, **kw)
    return qmm.quantize(x, axis, fmt, d, mode=mode, seed=77, offset=offset, **kw), d


def one_launch(x, axis, fmt, mode, offset, patience, kw):
    """(taken, codes, step sizes) of the one-launch form alone; guards around the codes."""
    L = qmm.lib()
    f = L.qmm_internal_scale_quantize
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_void_p,
                  ctypes.c_void_p, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p]
    t, g = qmm.tensor_desc(x, axis), qmm.granularity(**kw)
    b, r, c = x.shape
    shape = (b, r, c) if axis == 1 else (b, c, r)
    buf = torch.full((b * r * c + 2 * GUARD,), 77, dtype=torch.uint8, device=DEV)
    d = torch.full((L.qmm_num_scales(ctypes.byref(t), ctypes.byref(g)) + 2,), -1.0, dtype=torch.float32, device=DEV)
    taken = ctypes.c_int(-1)
    status = f(ctypes.byref(t), fmt, ctypes.byref(g), mode, 77, offset, d.data_ptr() + 4, buf.data_ptr() + GUARD, patience,
               ctypes.byref(taken), qmm._stream())
    assert status == 0
    torch.cuda.synchronize()
    assert bool((buf[:GUARD] == 77).all()) and bool((buf[-GUARD:] == 77).all()) and float(d[0]) == -1.0 and float(d[-1]) == -1.0
    return taken.value, buf[GUARD:-GUARD].view(shape), d[1:-1]


# (shape, axis, granularity): rows of one unit (16 elements) and of one more, units around a workgroup's (256 threads, 512 and
# 1024 units) and a grid's, strips of 64 columns and tiles of 128 and 512 rows, groups of few and of many words.
FORMS = [
    ((1, 1, 16), 1, {}), ((1, 1, 17), 1, {}), ((1, 3, 31), 1, {}), ((1, 16, 256), 1, {}), ((1, 1, 4097), 1, {}), ((1, 1, 16385), 1, {}),
    ((1, 1031, 1001), 1, {}), ((1, 4096, 1024), 1, {}), ((1, 4100, 2050), 1, {}), ((1, 9000, 1030), 1, {}), ((1, 12000, 2048), 1, {}),
    ((6, 40, 72), 1, dict(batch_groups=3)), ((7, 70, 96), 1, dict(batch_groups=3, batch_inner=2)), ((5, 33, 50), 1, dict(batch_groups=2, batch_inner=2)),
    ((4, 700, 333), 1, dict(batch_groups=2)), ((3, 1000, 1000), 1, dict(batch_groups=3)), ((96, 128, 64), 1, dict(batch_groups=12)), ((9, 20, 40), 1, {}),
    ((1, 1, 1), 0, {}), ((1, 127, 63), 0, {}), ((1, 129, 65), 0, {}), ((1, 511, 200), 0, {}), ((1, 1000, 1000), 0, {}), ((1, 9000, 1030), 0, {}),
    ((1, 16384, 1032), 0, {}), ((12, 130, 64), 0, dict(batch_groups=4)), ((7, 70, 96), 0, dict(batch_groups=3, batch_inner=2)), ((5, 513, 70), 0, {}),
    ((1, 4230, 33), 0, dict(per_channel=True)), ((1, 129, 65), 0, dict(per_channel=True)), ((1, 3, 5), 0, dict(per_channel=True)),
    ((1, 1031, 1001), 0, dict(per_channel=True)), ((3, 600, 200), 0, dict(per_channel=True, batch_groups=3)), ((1, 6000, 2000), 0, dict(per_channel=True)),
    ((1, 16384, 520), 0, dict(per_channel=True)), ((1, 4097, 40), 0, dict(per_channel=True)), ((1, 70001, 70), 0, dict(per_channel=True)), ((1, 18550, 6), 0, {}),
    ((2, 9000, 130), 0, dict(per_channel=True, batch_groups=2))]


def fits(shape, axis, dense, dtype, mode, offset, per_channel, groups):
    """Whether one of FORMS is for the one launch on 256 CUs: bytes of the rows; tiles of 64 columns by 128 or 512 rows, of which a column
    has few small ones and the tensor enough large ones, and for stochastic rounding enough workgroups, evenly spread."""
    b, r, c = shape
    nearest, bf16 = mode == qmm.RTNE, dtype == torch.bfloat16
    if axis == 1:
        if not nearest and bf16 and 256 < b * -(-r * c // 32768) < (384 if groups > 1 else 480) and b * r * c > 1 << 23:
            return False
        return b * r * c * (2 if bf16 else 4) <= (1 << 26 if nearest and (dense or r == 1) else 1 << 25)
    strips, whole = -(-c // 64), r % 4 == 0 and offset % 4 == 0
    small, large = b * strips * -(-r // 128), b * strips * -(-r // 512)
    waits = -(-r // 128) if per_channel else 0
    if nearest:
        return (waits <= 40 and small <= 1024) or (not (per_channel and large < 32) and large <= (3 * 256 if bf16 else 256))
    if c < 24 or (not whole and r < 8):
        return False
    least = (128 if whole else 320) if waits > 16 else 64 if whole else 256
    if waits <= 40 and least <= small <= 1024:
        return True
    least = (96 if whole else 144) if per_channel else 64 if whole else 256
    return max(least, 32 if per_channel else 0) <= large <= 256


@pytest.mark.parametrize("mode", [qmm.RTNE, qmm.STOCHASTIC])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("pad,shift", [(0, 0), (8, 0), (0, 1)])
@pytest.mark.parametrize("shape,axis,kw", FORMS)
def test_equals_the_two_calls(shape, axis, kw, pad, shift, dtype, mode):
    x = tensor(shape, dtype, seed=sum(shape), pad=pad, shift=shift)
    if x.numel() > 3000:
        x[-1, shape[1] // 2, 5] = float("nan") if kw else -0.0
        x[0, -1, -1] = float("inf") if kw else 3.0e38
    for fmt, offset in ((qmm.E4M3, 0), (qmm.INT8, 6)):
        want_c, want_d = two_calls(x, axis, fmt, mode, offset, kw)
        for patience in (FOREVER, 1, 0):                    # FOREVER is cut to the library's own patience; 1: leaders hand out lists
            taken, c, d = one_launch(x, axis, fmt, mode, offset, patience, kw)
            assert taken == fits(shape, axis, pad == shift == 0, dtype, mode, offset, kw.get("per_channel", False) and shape[2] > 1, kw.get("batch_groups", 1)), patience
            if not taken:
                continue
            assert torch.equal(d.view(torch.int32), want_d.view(torch.int32)), (fmt, patience)
            assert torch.equal(c, want_c), (fmt, patience)


def test_the_rule_takes_what_it_is_for():
    for shape, axis, kw in FORMS:
        if shape != (1, 1, 1):
            assert one_launch(tensor(shape, torch.bfloat16, 1), axis, qmm.E5M2, qmm.RTNE, 0, FOREVER, kw)[0] == 1, (shape, axis, kw)
    for shape, axis, kw in [((1, 1, 8), 1, {}),                                      # rows shorter than a unit
                            ((1, 40000, 2048), 1, {}), ((1, 40000, 2048), 0, {}),     # more than the chip holds
                            ((4, 8, 64), 1, dict(batch_groups=8)),                   # groups without a matrix
                            ((4, 64, 64), 0, dict(per_channel=True, batch_groups=2)), ((1, 64, 64), 1, dict(per_channel=True))]:
        assert one_launch(tensor(shape, torch.bfloat16, 1), axis, qmm.E5M2, qmm.RTNE, 0, FOREVER, kw)[0] == 0, (shape, axis, kw)


def test_recorded_calls_replay_like_eager_ones():
    x = torch.empty((1, 1000, 2064), dtype=torch.bfloat16, device=DEV)
    x.copy_(W.student_t(x.shape, 4, seed=1))
    forms = [(1, {}), (0, {}), (0, dict(per_channel=True))]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for axis, kw in forms:
            qmm.scale_quantize(x, axis, qmm.E4M3, **kw)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = [qmm.scale_quantize(x, axis, qmm.E4M3, **kw) for axis, kw in forms]
    for seed in (2, 3, 4):
        x.copy_(W.student_t(x.shape, 4, seed=seed) * seed)
        want = [qmm.scale_quantize(x, axis, qmm.E4M3, **kw) for axis, kw in forms]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for (c, d), (cw, dw) in zip(out, want):
            assert torch.equal(c, cw) and torch.equal(d, dw), seed


# The separate launches, which recorded calls take: partial maxima folded by the quantize pass, by a kernel of their own, by the
# workgroup that arrives last, in every form above, and the step sizes alone.  Three replays on changing values, the eager calls between.
@pytest.mark.parametrize("mode", [qmm.RTNE, qmm.STOCHASTIC])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("pad,shift", [(0, 0), (8, 0), (0, 1)])
def test_recorded_calls_of_every_form(pad, shift, dtype, mode):
    forms = [(shape, axis, dict(kw, per_channel=pc)) for shape, axis, kw in FORMS for pc in {kw.get("per_channel", False), shape[1] * shape[2] < 1100000}]
    forms += [((512, 33, 64), 1, dict(batch_groups=16)), ((4, 8, 64), 1, dict(batch_groups=8)), ((2, 600, 70), 0, dict(per_channel=True)),
              ((3, 20, 9000), 1, dict(per_channel=True, batch_groups=3))]
    xs = [tensor(shape, dtype, seed=sum(shape), pad=pad, shift=shift) for shape, _, _ in forms]
    fmts = [(qmm.E4M3, qmm.INT8, qmm.E5M2)[i % 3] for i in range(len(forms))]

    def calls():
        return [(qmm.scale_quantize(x, axis, fmt, mode=mode, seed=77, offset=6 * (i % 2), **kw), qmm.scale(x, axis, fmt, **kw))
                for i, (x, fmt, (_, axis, kw)) in enumerate(zip(xs, fmts, forms))]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        calls()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = calls()
    for replay in range(3):
        for i, x in enumerate(xs):
            x.mul_(-0.75)
            x[-1, x.shape[1] // 2, x.shape[2] // 3] = (5.0e4, float("inf"), float("nan"))[(i + replay) % 3]
        want = [two_calls(x, axis, fmt, mode, 6 * (i % 2), kw) for i, (x, fmt, (_, axis, kw)) in enumerate(zip(xs, fmts, forms))]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for form, ((c, d), alone), (want_c, want_d) in zip(forms, got, want):
            assert torch.equal(d.view(torch.int32), want_d.view(torch.int32)), (replay, form)
            assert torch.equal(alone.view(torch.int32), want_d.view(torch.int32)), (replay, form)
            assert torch.equal(c, want_c), (replay, form)


def test_streams_that_share_the_ring_of_boards():
    xs = [tensor((1, 512 + 64 * i, 1024), torch.bfloat16, seed=i) * (i + 1) for i in range(6)]
    want = [two_calls(x, 1, qmm.E4M3, qmm.RTNE, 0, {}) for x in xs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    got = []
    for rep in range(12):
        for i, x in enumerate(xs):
            with torch.cuda.stream(streams[i % 3]):
                got.append((i, qmm.scale_quantize(x, 1, qmm.E4M3)))
    torch.cuda.synchronize()
    for i, (c, d) in got:
        assert torch.equal(c, want[i][0]) and torch.equal(d, want[i][1]), i


def test_calls_beyond_the_length_of_the_ring():
    x = tensor((1, 16384, 520), torch.bfloat16, seed=9)     # 32 maxima a column: 63 calls to the ring's end
    want = two_calls(x, 0, qmm.E4M3, qmm.RTNE, 0, dict(per_channel=True))
    for i in range(300):
        c, d = qmm.scale_quantize(x, 0, qmm.E4M3, per_channel=True)
        if i % 20 == 0:
            assert torch.equal(c, want[0]) and torch.equal(d, want[1]), i


# One block (2048 elements a block), fewer blocks than fields, about as many, the lanes of a wavefront, a workgroup's threads, the
# largest grid (from 2^21 elements on; with denominators always two launches there, without them beyond 2^22).
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n", [1, 2048, 2049, 5000, 15 * 2048, 16 * 2048 + 3, 17 * 2048, 64 * 2048, 65 * 2048 + 1, 257 * 2048, 1 << 21, 3000001])
def test_metric_in_one_launch_equals_two(n, dtype):
    L = qmm.lib()
    f = L.qmm_internal_metric
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p,
                  ctypes.c_size_t, ctypes.c_uint32, ctypes.c_void_p]
    g = torch.Generator(device=DEV).manual_seed(n)
    ref = torch.randn(n, generator=g, device=DEV)
    y = (ref + 0.05 * torch.randn(n, generator=g, device=DEV)).to(dtype)
    if n > 4000:
        y[n // 2] = float("nan"); ref[n // 3] = 0.0; y[-1] = float("inf")
    denom = torch.rand(n, generator=g, device=DEV) + 0.1
    ws = torch.empty(L.qmm_metric_workspace_size(n), dtype=torch.uint8, device=DEV)
    for d in (None, denom):
        out = torch.empty(16, dtype=torch.float64, device=DEV)
        qmm.metric(y, ref, d, out=out, workspace=ws)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        two = torch.empty_like(out)
        with torch.cuda.graph(graph):
            qmm.metric(y, ref, d, out=two, workspace=ws)
        for patience in (FOREVER, 0):
            ws.fill_(0xFF)                                   # NaN in every partial sum
            one = torch.full_like(out, -1.0)
            assert f(y.data_ptr(), qmm._dtype_code(y), ref.data_ptr(), d.data_ptr() if d is not None else None, n, one.data_ptr(),
                     ws.data_ptr(), ws.numel(), patience, qmm._stream()) == 0
            torch.cuda.synchronize()
            two.fill_(-2.0)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(one.view(torch.int64), two.view(torch.int64)), (d is not None, patience)
            assert torch.equal(one.view(torch.int64), out.view(torch.int64))


# Step sizes alone: one and several tensors (the several-tensors kernel takes dense bfloat16 with one step size; the others go one by
# one), one group and several in runs, one workgroup and many, a ragged end; found by waiting and formed by the folding workgroup.
@pytest.mark.parametrize("shapes,dtype,kw", [
    ([(1, 1, 8)], torch.bfloat16, {}), ([(1, 3, 5)], torch.float32, {}), ([(1, 1031, 1001)], torch.bfloat16, {}), ([(1, 8192, 1032)], torch.float32, {}),
    ([(1, 2048, 768), (1, 768, 768), (1, 1, 16)], torch.bfloat16, {}), ([(1, 9000, 1024), (1, 64, 1024)], torch.bfloat16, {}),
    ([(12, 70, 96)], torch.bfloat16, dict(batch_groups=4)), ([(13, 70, 96)], torch.float32, dict(batch_groups=3, batch_inner=2)),
    ([(64, 300, 300)], torch.bfloat16, dict(batch_groups=16)), ([(5, 33, 50)], torch.bfloat16, dict(batch_groups=2, batch_inner=9)),
    ([(2, 8, 64)], torch.bfloat16, dict(batch_groups=5))])
def test_step_sizes_in_one_launch(shapes, dtype, kw):
    L = qmm.lib()
    f = L.qmm_internal_scale_multi
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int32, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_uint32, ctypes.c_void_p]
    xs = [tensor(s, dtype, seed=i + s[1]) * (i + 1) for i, s in enumerate(shapes)]
    if xs[0].numel() > 3000:
        xs[0].view(-1)[1234] = float("nan") if kw else -7.5e4
    n, groups, inner = len(xs), kw.get("batch_groups", 1), kw.get("batch_inner", 1)
    t, g = (qmm.Tensor * n)(*[qmm.tensor_desc(x, 1) for x in xs]), (qmm.Granularity * n)(*[qmm.granularity(**kw) for _ in xs])
    ws = torch.empty(L.qmm_scale_multi_workspace_size(n, t, g), dtype=torch.uint8, device=DEV)
    for patience in (FOREVER, 0):
        out = [torch.full((groups,), -1.0, device=DEV) for _ in xs]
        assert f(n, t, qmm.E4M3, g, qmm.MultiDesc.pointers(out), ws.data_ptr(), ws.numel(), patience, qmm._stream()) == 0
        torch.cuda.synchronize()
        for x, d in zip(xs, out):
            want = torch.from_numpy(O.scale(x.float().cpu().numpy(), 1, qmm.E4M3, False, groups, inner)).to(DEV)
            assert torch.equal(d.view(torch.int32), want.view(torch.int32)), patience
