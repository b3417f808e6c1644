"""Calls under stream capture: folded-weight calls past the lines on sizes and
ops between two ring lengths keep to the captured stream, so that another
thread's call on the same plan goes on; tables that are not on the device
yet are not put there under capture.  Where ops between two ring lengths have
no helper stream, or share the GPU with the weight gradient's pass, they take
the direct kernels that are faster there.  Every replay, with eager work between them, equals the eager result
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


def _kernels(run):
    import torch
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    out = run()
    torch.cuda.synchronize()
    ran = disco.kernel_timing_read(32)
    disco.kernel_timing(False)
    return out, set(ran)


@pytest.mark.parametrize("chans,grids,alone", [
    (16, (512, 1024, 256, 512), "direct"),      # halving
    (16, (256, 512, 512, 1024), "direct"),      # doubling
    (8, (256, 512, 512, 1024), "spectral"),     # doubling, beside the ring sweep
])
def test_two_ring_lengths_without_a_helper_stream(chans, grids, alone):
    import torch
    plan = disco.Plan(*grids, 3 * math.pi / min(grids[0], grids[2]))
    x, w = synth.random_inputs(93, (1, chans) + grids[:2], (chans, chans, 9))
    xt, wt = torch_dev(x), torch_dev(w)
    ref, ran = _kernels(lambda: plan.forward(xt, wt))
    say("two ring lengths", chans, grids, sorted(ran))
    assert "spectral_mac" in ran
    y = torch.empty_like(ref)
    _, ran = _kernels(lambda: plan.forward_noalloc(xt, wt, y))
    assert ("spectral_mac" in ran) == (alone == "spectral")
    assert _rel(y, ref) <= 1e-6
    y2, second = torch.empty_like(ref), torch.cuda.Stream()

    def eager():
        with torch.cuda.stream(second):
            plan.forward(xt, wt, y=y2)
        second.synchronize()

    graph = _capture(lambda: plan.forward(xt, wt, y=y), eager)
    for _ in range(3):
        y.zero_()
        plan.forward(xt, wt, y=y2)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert _rel(y, ref) <= 1e-6 and _rel(y2, ref) <= 1e-6
    del graph
    plan.close()


def test_input_gradient_of_a_halving_layer_beside_its_weight_gradient():
    import torch
    plan = disco.Plan(512, 1024, 256, 512, 3 * math.pi / 256, backward=True)
    x, w = synth.random_inputs(94, (1, 4, 512, 1024), (6, 4, 9))
    dy = torch.randn((1, 6, 256, 512), device="cuda:0")
    xt, wt = torch_dev(x), torch_dev(w)
    (dx0, _), ran = _kernels(lambda: disco.forward_backward(plan, xt, wt, dy, want_dw=False))
    assert "spectral_mac" not in ran
    (dx1, _), ran = _kernels(lambda: disco.forward_backward(plan, xt, wt, dy))
    assert "spectral_mac" not in ran
    assert torch.equal(dx1, dx0)
    ref = disco.Plan(512, 1024, 256, 512, 3 * math.pi / 256, backward=True, direct=True)
    dx2, _ = disco.forward_backward(ref, xt, wt, dy)
    say("halving layer's gradients", sorted(ran), _rel(dx1, dx2))
    assert _rel(dx1, dx2) <= 1e-6
    ref.close()
    plan.close()
