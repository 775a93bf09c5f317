"""The binding's native short path (csrc/qmm_host.cpp): declines what is not the plain case, so that the ctypes path and its
errors stay what they were, and gives on the GPU what the ctypes path gives."""
import numpy as np
import pytest
import torch

from paper_2408_02897_amd import qmm

DEV = "cuda:0"


class Sub(torch.Tensor):
    pass


@pytest.fixture(scope="module")
def host():
    import os
    if not (os.path.exists(qmm.LIB_PATH) and os.path.exists(qmm.HOST_PATH)):
        from paper_2408_02897_amd import build
        build.build()
    return qmm._host()


def test_declines_what_is_not_plain(host):
    x = torch.zeros((4, 32), dtype=torch.bfloat16)
    rest = (1, qmm.E4M3, False, 1, qmm.RTNE, 0, 0, 1)
    for bad in (x, x.as_subclass(Sub), None, 3, np.zeros((4, 32))):
        assert host.scale_quantize(bad, *rest) is None and host.quantized_operand(bad, *rest) is None
    assert host.scale_quantize(x) is None
    op = qmm.operand(x, qmm.E4M3, torch.ones(1))
    for a, b in (((x, op), (x, op)), (None, (x, op)), ((x,), (x, op)), ((x, 1), (x, op)), ([x, op], (x, op))):
        assert host.gemm(a, b, torch.float32, None) is None
    assert host.metric(x, x.float(), None, None, None) is None and host.metric(x, 1, None, None, None) is None


# A tree with libqmm.so alone: the calls go through ctypes.
def test_does_without_the_short_path(host, monkeypatch):
    monkeypatch.setattr(qmm, "HOST_PATH", qmm.HOST_PATH + ".none")
    monkeypatch.setattr(qmm, "_short", None)
    x = torch.zeros((4, 32), dtype=torch.bfloat16)
    for call in (lambda: qmm.scale_quantize(x, 1, qmm.E4M3), lambda: qmm.quantized_operand(x, 1, qmm.E4M3)):
        with pytest.raises(AssertionError):                  # (tensor_desc: not a device tensor)
            call()
    with pytest.raises(AssertionError):
        qmm.metric(x, torch.zeros(5))
    op = qmm.operand(x, qmm.E4M3, torch.ones(1))
    with pytest.raises(AssertionError):
        qmm.gemm((x, op), (x[:, :16], op))


@pytest.mark.gpu
def test_equals_the_ctypes_path(host, monkeypatch):
    class Off:
        @staticmethod
        def decline(*_):
            return None
        scale_quantize = quantized_operand = gemm = metric = decline
    x = torch.randn((3, 70, 96), device=DEV).bfloat16()
    cases = [dict(), dict(per_channel=True, batch_groups=3), dict(batch_groups=3, mode=qmm.STOCHASTIC, seed=2 ** 63 + 5), dict(batch_groups=1, batch_inner=2)]

    def run():
        out = []
        for axis in (0, 1):
            for kw in cases:
                (c, op), d = qmm.quantized_operand(x, axis, qmm.E4M3, **kw)
                c2, d2 = qmm.scale_quantize(x, axis, qmm.E4M3, **kw)
                assert torch.equal(c, c2) and torch.equal(d, d2)
                assert (op.format, op.is_codes, op.data, op.delta) == (qmm.E4M3, 1, c.data_ptr(), d.data_ptr()) and op._keep[0] is c and op._keep[1] is d
                assert (op.gran.per_channel, op.gran.batch_groups, op.gran.batch_inner) == (int(kw.get("per_channel", False)), kw.get("batch_groups", 1), kw.get("batch_inner", 1))
                out += [c, d]
        a, _ = qmm.quantized_operand(x, 1, qmm.E4M3)
        for dt in (torch.float32, torch.bfloat16):
            y = qmm.gemm(a, a, dt)
            kept = torch.empty_like(y)
            assert qmm.gemm(a, a, out=kept) is kept and torch.equal(kept, y)
            ref = y.float() + 0.25
            m = torch.empty(16, dtype=torch.float64, device=DEV)
            assert qmm.metric(y, ref, out=m) is m and torch.equal(m, qmm.metric(y, ref))
            out += [y, m, qmm.metric(y, ref, ref.abs() + 1)]
        flat = (a[0][0], a[1])
        out.append(qmm.gemm(flat, flat))
        return out

    short = run()
    monkeypatch.setattr(qmm, "_short", Off)
    for s, c in zip(short, run()):
        assert s.dtype == c.dtype and s.shape == c.shape and torch.equal(s, c)


@pytest.mark.gpu
def test_errors_are_those_of_the_ctypes_path(host):
    x = torch.zeros((4, 24), dtype=torch.bfloat16, device=DEV)
    a, _ = qmm.quantized_operand(x, 1, qmm.E4M3)
    with pytest.raises(qmm.QmmError) as e:
        qmm.gemm(a, a)                                       # K = 24 is not a multiple of 16
    assert e.value.status == 4
    with pytest.raises(qmm.QmmError):
        qmm.quantized_operand(x, 1, qmm.BF16)
    with pytest.raises(qmm.QmmError):
        qmm.quantized_operand(x, 1, qmm.E4M3, batch_groups=0)
    with pytest.raises(AssertionError):
        qmm.quantized_operand(x.t(), 1, qmm.E4M3)            # columns are not contiguous
    with pytest.raises(TypeError):
        qmm.quantized_operand(x.half(), 1, qmm.E4M3)
    with pytest.raises(AssertionError):
        qmm.metric(x, torch.zeros((4, 25), device=DEV))
    b, _ = qmm.quantized_operand(torch.zeros((4, 32), dtype=torch.bfloat16, device=DEV), 1, qmm.E4M3)
    with pytest.raises(AssertionError):
        qmm.gemm(a, b)


# The short path is built against one torch: another one makes build_host compile again, the same one does not.
def test_short_path_is_built_again_for_another_torch(tmp_path, monkeypatch):
    from paper_2408_02897_amd import build
    commands = []
    monkeypatch.setattr(build, "HOST", str(tmp_path / "_qmm_host.so"))
    monkeypatch.setattr(build, "OBJDIR", str(tmp_path / "obj"))
    monkeypatch.setattr(build.subprocess, "run", lambda command, check: (commands.append(command), open(build.HOST, "w").close()))
    for version, runs in (("1", 1), ("1", 1), ("2", 2)):
        monkeypatch.setattr(torch, "__version__", version)
        build.build_host()
        assert len(commands) == runs
