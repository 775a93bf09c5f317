"""Paths of the kernels that a call is routed to by its sizes, types or alignment, each compared bit for bit with the
general path over the forms it accepts (ragged and odd extents, strides, types), and against writes outside the output."""
import numpy as np
import pytest
import torch

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


# The call that also returns the accumulators takes the element-by-element epilogue: Y of the two calls must agree in
# every bit.  Extents around the tiles (128, 256), odd ones (rows that start off every vector boundary) and outputs large
# enough for the 256 x 256 tiles.
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("kind", ["e4m3", "int8", "bf16"])
@pytest.mark.parametrize("m,n,k", [(1, 1, 16), (127, 130, 144), (129, 255, 128), (257, 129, 272), (200, 203, 400),
                                   (128, 132, 256), (130, 256, 64), (4099, 3071, 128), (3842, 3074, 144)])
def test_output_at_edges_and_odd_extents(kind, m, n, k, out_dtype):
    a, b = operands(kind, m, n, k, per_channel=(m + n) % 2 == 1)
    want, _ = qmm.gemm(a, b, out_dtype, want_acc=True)
    buf, y = guarded((1, m, n), out_dtype)
    qmm.gemm(a, b, out_dtype, out=y)
    assert torch.equal(y, want)
    assert intact(buf)


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
