"""The bf16 matrix-core kernel's wide forms against the fp64 oracle: even
longitude strides with at least 128 (ring, longitude tile) workgroups, which
stage the inputs as natural pairs (offsets that start at odd longitudes, whole
polar rings, ragged tiles, an odd last input channel, one ring fewer than the
rule asks for), and 33 to 64 output channels in one workgroup (one phase, both
stagings, a second ragged workgroup of output channels).  Inputs are bf16 as
stored; the values psi and the intermediate product are rounded to bf16 (half
an ulp, 2^-9, each, and the output once more), so the relative L2 error stays
below sqrt(3) 2^-9 < 5e-3 and the largest error, a sum of such roundings over
the largest output, below 2e-2 of it."""
import math

import numpy as np
import pytest

from gpu_util import rel_l2, run_gpu, run_oracle, say, torch_dev
from paper_2209_13603_amd import synth

pytestmark = pytest.mark.gpu

PAIRS = [
    ("forward", (256, 64, 128, 32)),      # exactly 128 workgroups
    ("forward", (254, 64, 127, 32)),      # one fewer: duplicated elements
    ("forward", (128, 1184, 64, 592)),    # three tiles, the last ragged
    ("forward", (256, 128, 128, 32)),     # stride 4
    ("transpose", (128, 32, 256, 64)),
]
CASES = [(op, case, chans) for op, case in PAIRS for chans in [(3, 5), (9, 33), (4, 64), (3, 70)]]
CASES += [("forward", (40, 80, 40, 80), chans) for chans in [(9, 48), (4, 64), (3, 65)]]


@pytest.mark.parametrize("op,case,chans", CASES, ids=str)
def test_wide_forms_against_oracle(op, case, chans):
    a, b, c, d = case
    args = (a, b, c, d, 3 * math.pi / min(a, c))
    Ci, Co = chans
    xs = (2, Ci, a, b) if op == "forward" else (2, Ci, c, d)
    ws = (Co, Ci, 9) if op == "forward" else (Ci, Co, 9)
    x, w = synth.random_inputs(96, xs, ws, dtype="bf16")
    say("matrix_core wide", op, case, chans)
    y, plan = run_gpu(args, x, w, op, dtype="bf16", algo="matrix_core")
    ref = run_oracle(args, x, w, op)
    plan.close()
    assert rel_l2(y, ref) <= 5e-3
    assert float(np.abs(y - ref).max() / np.abs(ref).max()) <= 2e-2


@pytest.mark.parametrize("chans", [(20, 40), (8, 64), (33, 96)], ids=lambda c: "%dto%d" % c)
@pytest.mark.parametrize("case", [(64, 128, 64, 128), (64, 128, 32, 64)], ids=lambda c: "%dx%d_%dx%d" % c)
def test_output_channels_per_workgroup(case, chans):
    """32 output channels a workgroup (one item) and 64 (six items) give the same
    bits, and the oracle's values."""
    import torch
    a, b, c, d = case
    ci, co = chans
    args = (a, b, c, d, 3 * math.pi / c)
    x, w = synth.random_inputs(67, (6, ci, a, b), (co, ci, 9), dtype="bf16")
    say("output channels per workgroup", case, chans)
    y, plan = run_gpu(args, x, w, "forward", dtype="bf16", algo="matrix_core")
    xt, wt = torch_dev(x, "bf16"), torch_dev(w, "bf16")
    six = plan.forward(xt, wt, algo="matrix_core")
    for i in (0, 5):
        one = plan.forward(xt[i:i + 1].contiguous(), wt, algo="matrix_core")
        assert torch.equal(one[0], six[i])
    ref = run_oracle(args, x[:1], w, "forward")
    assert rel_l2(y[:1], ref) <= 2e-2
    plan.close()
