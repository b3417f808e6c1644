"""Calls under stream capture: folded-weight calls past the lines on sizes keep
to the captured stream, so that another thread's call on the same plan
goes on; tables that are not on the device yet are not put there under
capture.  Every replay, with eager work between them, equals the eager result
to the rounding of the kernels' different sums.
"""
import math
import threading

import pytest

from gpu_util import say, torch_dev
from paper_2209_13603_amd import disco, synth

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


def _capture(run, between=None):
    """Captures run() and returns the graph; `between` runs on another thread
    while the capture is open."""
    import torch
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph, errors = torch.cuda.CUDAGraph(), []

    def other():
        try:
            between()
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append(e)

    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        run()
        if between is not None:
            t = threading.Thread(target=other)
            t.start()
            t.join()
    assert not errors, errors
    return graph


@pytest.mark.parametrize("basis,grids,op,C", [
    ("separable4x4", (256, 512, 256, 512), "forward", 256),       # 2^25 outputs: the helper stream, when eager
    ("bilinear3x3", (256, 512, 256, 512), "forward", 64),         # 2^23: spectral rings on the caller's stream
    ("separable4x4", (256, 512, 128, 256), "transpose", 64),
])
def test_captured_depthwise_call_beside_another_thread(basis, grids, op, C):
    import torch
    a, b, c, d = grids
    plan = disco.Plan(*grids, 3 * math.pi / min(a, c), basis=basis)
    xs = (1, C, a, b) if op == "forward" else (1, C, c, d)
    x, w = synth.random_inputs(91, xs, (C, 16 if basis == "separable4x4" else 9), c_in=1)
    xt, wt = torch_dev(x), torch_dev(w)
    f = plan.forward_depthwise if op == "forward" else plan.transpose_depthwise
    ref, y, y2 = f(xt, wt), torch.empty((1, C, a, b), device="cuda:0"), torch.empty((1, C, a, b), device="cuda:0")
    torch.cuda.synchronize()
    second = torch.cuda.Stream()

    def eager():
        with torch.cuda.stream(second):
            f(xt, wt, y=y2)
        second.synchronize()

    say("captured depthwise", basis, grids, op)
    graph = _capture(lambda: f(xt, wt, y=y), eager)
    assert _rel(y2, ref) <= 1e-6
    for _ in range(3):
        y.zero_()
        f(xt, wt, y=y2)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert _rel(y, ref) <= 1e-6 and _rel(y2, ref) <= 1e-6
    del graph
    plan.close()


def test_first_large_call_under_capture_needs_no_upload():
    """A small depthwise call of a 3x3 plan's transposed op puts the blocked
    layout on the device; a captured call past the lines on sizes then runs
    on it alone."""
    import torch
    n, C = 256, 64
    plan = disco.Plan(n, 2 * n, n, 2 * n, 3 * math.pi / n)
    x, w = synth.random_inputs(92, (1, C, n, 2 * n), (C, 9), c_in=1)
    xt, wt = torch_dev(x), torch_dev(w)
    one = plan.transpose_depthwise(xt[:, 5:6].contiguous(), wt[5:6].contiguous())
    y = torch.empty((1, C, n, 2 * n), device="cuda:0")
    torch.cuda.synchronize()
    held = plan.info()["psi_bytes"]
    say("captured first large call")
    graph = _capture(lambda: plan.transpose_depthwise(xt, wt, y=y))
    assert plan.info()["psi_bytes"] == held
    for _ in range(3):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert _rel(y[:, 5:6], one) <= 1e-6
    ref = plan.transpose_depthwise(xt, wt)  # with the tables
    torch.cuda.synchronize()
    assert plan.info()["psi_bytes"] > held and _rel(y, ref) <= 1e-6
    del graph
    plan.close()
