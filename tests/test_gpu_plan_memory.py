"""Plan memory (Sec. 4.2's compressed psi, App. B's memory figures): a plan
puts on the device only what a forward call with the default algo runs on
and uploads the other layouts on first use.  Checked here: the 2048 x 4096
plan's device bytes, its reported compressed psi, the growth when the
transposed op and other schedules are first used (to the all-layouts figure
the plan reports), and that lazily and eagerly built plans give the same
bits."""
import math

import numpy as np
import pytest

from gpu_util import say, torch_dev
from paper_2209_13603_amd import disco, synth

pytestmark = pytest.mark.gpu


def test_headline_plan_holds_only_the_forward_schedule():
    wl = synth.WORKLOADS["sphere2048x4096"]
    plan = disco.Plan(*wl.plan_args(), **wl.plan_kwargs())
    info = plan.info()
    say("  psi_bytes %.1f MB (all layouts %.1f MB), compressed psi %.2f MB" %
        (info["psi_bytes"] / 1e6, info["psi_bytes_all_layouts"] / 1e6, info["psi_compressed_bytes"] / 1e6))
    assert info["psi_bytes"] < 60e6
    # the plain compressed form: per entry a ring, an offset and 9 fp32 values, per pattern a pointer
    assert info["psi_compressed_bytes"] == info["nnz_entries"] * (8 + 4 * 9) + 4 * (2048 + 1)
    assert info["bytes_entries"] == 0 and info["bytes_stencil"] == 0 and info["bytes_matrix_core"] == 0
    assert info["psi_bytes_all_layouts"] > 2 * info["psi_bytes"]
    plan.close()


def test_layouts_are_uploaded_on_first_use():
    import torch
    case = (64, 128, 32, 64)
    a, b, c, d = case
    plan = disco.Plan(a, b, c, d, 3 * math.pi / c)
    before = plan.info()
    x, w = synth.random_inputs(3, (2, 3, c, d), (3, 5, 9))
    xt, wt = torch_dev(x), torch_dev(w)
    plan.transpose(xt, wt)
    after_tr = plan.info()
    assert after_tr["psi_bytes"] > before["psi_bytes"]
    for algo in ("gather_then_contract", "contract_then_gather", "fused_direct"):
        plan.transpose(xt, wt, algo=algo)
    xf, wf = (torch_dev(v) for v in synth.random_inputs(4, (2, 3, a, b), (5, 3, 9)))
    for algo in ("gather_then_contract", "contract_then_gather", "fused_direct"):
        plan.forward(xf, wf, algo=algo)
    plan.forward_depthwise(xf, torch_dev(np.ones((3, 9), np.float32)))
    plan.transpose_depthwise(xt, torch_dev(np.ones((3, 9), np.float32)))
    torch.cuda.synchronize()
    full = plan.info()
    say("  %d -> %d -> %d bytes (all layouts %d)" % (before["psi_bytes"], after_tr["psi_bytes"], full["psi_bytes"],
                                                    full["psi_bytes_all_layouts"]))
    assert full["psi_bytes"] == full["psi_bytes_all_layouts"]
    plan.close()


@pytest.mark.parametrize("op", ["forward", "transpose"])
@pytest.mark.parametrize("algo", ["auto", "fused", "fused_direct", "gather_then_contract", "contract_then_gather"])
def test_lazy_and_eager_plans_agree_bitwise(op, algo):
    import torch
    a, b, c, d = 64, 128, 32, 64
    args = (a, b, c, d, 3 * math.pi / c)
    lazy, eager = disco.Plan(*args), disco.Plan(*args, eager=True)
    info = eager.info()
    assert info["psi_bytes"] == info["psi_bytes_all_layouts"]
    xs = (2, 6, a, b) if op == "forward" else (2, 6, c, d)
    ws = (5, 6, 9) if op == "forward" else (6, 5, 9)
    x, w = synth.random_inputs(6, xs, ws)
    xt, wt = torch_dev(x), torch_dev(w)
    ys = [getattr(p, op)(xt, wt, algo=algo) for p in (lazy, eager)]
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1])
    lazy.close()
    eager.close()


def test_folded_bases_hold_spectral_tables_only_where_a_call_reads_them():
    """Separable basis: ops with a longitude stride and cutoffs whose rings are
    all wide have no ring walk, so no call reads frequency-domain tables there
    and none are built."""
    n = 256
    down = disco.Plan(n, 2 * n, n // 2, n, 3 * math.pi / (n // 2), basis="separable4x4", eager=True)
    i = down.info()
    say("  256x512 -> 128x256: tables %d forward, %d transposed" % (i["spectral_tables_forward"],
                                                                  i["spectral_tables_transpose"]))
    assert i["spectral_rings_forward"] == 0 and i["spectral_tables_forward"] == 0
    assert i["spectral_rings_transpose"] > 0
    eight = disco.Plan(n, 2 * n, n, 2 * n, 8 * math.pi / n, basis="separable4x4", eager=True)
    assert eight.info()["spectral_rings_forward"] == 0 and eight.info()["bytes_spectral"] == 0
    down.close()
    eight.close()


@pytest.mark.parametrize("n,cut,line", [(256, 3, 128), (256, 5, 128), (256, 6, 128), (512, 3, 192), (1024, 3, 192), (1024, 5, 192),
                                        (1024, 6, 128)])
def test_line_of_wide_rings_of_the_folded_bases(n, cut, line):
    """Wide from 128 entries on, on rings of 1024 longitudes from 192 on, the other
    of the two where the walk does not hold the windows."""
    args = (n, 2 * n, n, 2 * n, cut * math.pi / n)
    plan = disco.Plan(*args, basis="separable4x4")
    counts = np.bincount(disco.psi_entries(*args, basis=2)["out_ring"], minlength=n)
    i = plan.info()
    say("  %d x %d, %d rings of cutoff: %d spectral rings, %.2f MB of tables" %
        (n, 2 * n, cut, i["spectral_rings_forward"], i["bytes_spectral"] / 1e6))
    assert i["spectral_rings_forward"] == int((counts >= line).sum()) > 0
    plan.close()


@pytest.mark.parametrize("grids,op,C", [((256, 512, 256, 512), "forward", 65),    # the line at 128
                                        ((256, 512, 128, 256), "transpose", 65),  # at 192: no walk at 128
                                        ((1024, 2048, 1024, 2048), "forward", 4)])  # at 128: no walk at 192
def test_six_rings_of_cutoff(grids, op, C):
    """Six rings of cutoff on either line: a call past the lines on sizes equals
    its channels alone, directly summed, to the rounding of two transforms."""
    import torch
    a, b, c, d = grids
    tc = 6 * math.pi / min(a, c)
    plan = disco.Plan(*grids, tc, basis="separable4x4")
    one = disco.Plan(*grids, tc, basis="separable4x4", direct=True)
    x, w = synth.random_inputs(8, (1, C) + ((a, b) if op == "forward" else (c, d)), (C, 16), c_in=1)
    xt, wt = torch_dev(x), torch_dev(w)
    f, g = (p.forward_depthwise if op == "forward" else p.transpose_depthwise for p in (plan, one))
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    y = f(xt, wt)
    torch.cuda.synchronize()
    ran = disco.kernel_timing_read()
    disco.kernel_timing(False)
    assert "stencil_walk" in ran and "spectral_mac" in ran
    for ch in (0, C - 1):
        z = g(xt[:, ch:ch + 1].contiguous(), wt[ch:ch + 1].contiguous())
        err = float((y[:, ch:ch + 1] - z).norm() / z.norm())
        say("  channel %d rel_l2 %.3e" % (ch, err))
        assert err <= 1e-6
    torch.cuda.synchronize()
    plan.close()
    one.close()
