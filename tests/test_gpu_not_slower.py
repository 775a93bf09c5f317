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
# others' slices again, alone (16 GB: 1.23 times the separate launches; now 1.0).
def test_step_size_of_many_gigabytes():
    x = torch.empty((1, 1 << 21, 4096), dtype=torch.bfloat16, device=DEV).normal_()
    x[0, 12345, 77] = -300.0
    call, out = scale_call(x)
    ratio = eager_over_recorded(call, 3)
    assert float(out) == torch.tensor(300.0 / 448.0).item()
    assert ratio < 1.1, ratio
