"""The folded-weight kernels' ring walk and the spectral path of its wide rings
(one-channel items, stride-1 ops), and the spectral path of ops whose two
grids have different ring lengths.

A depthwise call past the lines on sizes (lifted here) takes the walk and the
spectral path; the same channel alone, below the lines and with algo
fused_direct, sums every ring directly (checked against the fp64 oracle on small grids by the
other tests).  The two differ by the rounding of sums of up to 128 products
and of two transforms of at most 512 points in fp32: 2^-24 sqrt(128) and
2^-24 log2(512) relative to the ring's values, 1e-6 together; bf16 outputs by
one rounding to 2^-9.
"""
import math

import numpy as np
import pytest

from gpu_util import rel_l2, run_gpu, run_oracle, say, to_numpy, torch_dev
from paper_2209_13603_amd import disco, synth

pytestmark = pytest.mark.gpu

K = {"bilinear3x3": 9, "axisym4": 4, "separable4x4": 16}
# (nlat_in, nlon_in, nlat_out, nlon_out, sampling, op, batch, channels)
CASES = [
    (128, 256, 128, 256, "cell_centred", "forward", 1, 64),    # one tile, wrapped both ways
    (128, 256, 128, 256, "cell_centred", "forward", 3, 23),    # odd channel and batch groups
    (257, 512, 257, 512, "poles", "forward", 2, 9),            # two tiles, odd ring count
    (256, 1024, 256, 1024, "cell_centred", "forward", 1, 9),   # tiles away from the seam
    (128, 256, 64, 128, "cell_centred", "transpose", 2, 35),   # two phases
    (128, 256, 32, 64, "cell_centred", "transpose", 5, 13),    # four phases
    (256, 256, 128, 256, "cell_centred", "forward", 1, 65),    # latitude-only change: four new rings a step
]


@pytest.mark.parametrize("basis", list(K))
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d_%dx%d_%s_%s_%dx%d" % c)
def test_depthwise_walk_and_spectral_match_direct(case, dtype, basis, monkeypatch):
    import torch
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "128")  # the default; lifts the lines on sizes
    a, b, c, d, smp, op, B, C = case
    tc = 3 * math.pi / (min(a, c) - (smp == "poles"))
    xs = (B, C, a, b) if op == "forward" else (B, C, c, d)
    x, w = synth.random_inputs(71, xs, (C, K[basis]), dtype=dtype, c_in=1)
    say("ring walk", case, basis, dtype)
    plan = disco.Plan(a, b, c, d, tc, basis=basis, sampling=smp)
    monkeypatch.delenv("DISCO_SPECTRAL_MIN_ENTRIES")
    one = disco.Plan(a, b, c, d, tc, basis=basis, sampling=smp)  # below the lines
    xt, wt = torch_dev(x, dtype), torch_dev(w, dtype)
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    y = plan.forward_depthwise(xt, wt) if op == "forward" else plan.transpose_depthwise(xt, wt)
    ran = disco.kernel_timing_read()
    disco.kernel_timing(False)
    assert "stencil_walk" in ran and "spectral_mac" in ran
    for ch in (0, C // 2, C - 1):
        for bi in (0, B - 1):
            xc = xt[bi:bi + 1, ch:ch + 1].contiguous()
            if basis == "bilinear3x3":
                f = one.forward_depthwise if op == "forward" else one.transpose_depthwise
                yc = f(xc, wt[ch:ch + 1].contiguous())  # one item: every ring summed directly
            else:
                yc, _ = run_gpu(None, to_numpy(xc).astype(np.float32),
                                to_numpy(wt[ch]).astype(np.float32)[None, None, :], op, dtype=dtype,
                                algo="fused_direct", plan=one)
                yc = torch.from_numpy(np.asarray(yc))
            got, ref = to_numpy(y[bi, ch]), to_numpy(yc)[0, 0]
            err = rel_l2(got, ref)
            mx = np.abs(got - ref).max() / np.abs(ref).max()
            say("  item (%d, %d) rel_l2 %.3e max %.3e" % (bi, ch, err, mx))
            assert err <= (1e-6 if dtype == "fp32" else 2e-3)
            assert mx <= (4e-6 if dtype == "fp32" else 8e-3)
    plan.close()
    one.close()


@pytest.mark.parametrize("op", ["forward", "transpose"])
@pytest.mark.parametrize("case", [(64, 128, 32, 64), (32, 64, 64, 128), (64, 256, 32, 64), (64, 128, 64, 64)],
                         ids=lambda c: "%dx%d_%dx%d" % c)
@pytest.mark.parametrize("chans", [(2, 3), (9, 12)], ids=lambda c: "%dto%d" % c)
def test_spectral_rings_of_two_lengths(case, op, chans, monkeypatch):
    """Up- and downsampling by 2 and 4 with most rings on the spectral path,
    against the oracle in full."""
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "8")
    a, b, c, d = case
    args = (a, b, c, d, 3 * math.pi / min(a, c))
    ci, co = chans
    xs = (2, ci, a, b) if op == "forward" else (2, ci, c, d)
    ws = (co, ci, 9) if op == "forward" else (ci, co, 9)
    x, w = synth.random_inputs(72, xs, ws)
    say("two ring lengths", case, op, chans)
    y, plan = run_gpu(args, x, w, op, algo="fused")
    assert plan.info()["spectral_rings_%s" % op] > 0
    ref = run_oracle(args, x, w, op)
    err = rel_l2(y, ref)
    say("  rel_l2 %.3e" % err)
    assert err <= 1e-5
    assert np.abs(y - ref).max() <= 1e-5 * np.abs(ref).max()
    plan.close()


@pytest.mark.parametrize("basis", list(K))
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("case", [(64, 128, 64, 128, "cell_centred", False), (65, 128, 65, 128, "poles", False),
                                  (64, 128, 32, 64, "cell_centred", True), (64, 512, 64, 512, "cell_centred", False)],
                         ids=lambda c: "%dx%d_%dx%d_%s_%s" % c)
def test_depthwise_weight_gradient_by_correlation(case, dtype, basis, monkeypatch):
    """dW from the correlations of dy and x (ring walk and frequency domain),
    an odd number of channels and a batch, against the oracle: sums of up to
    2 x 64 x 512 fp32 products with random signs, 1e-5 as the other gradient
    tests; bf16 inputs are exact and the sums fp32, so only dW's own rounding
    (2^-9 relative) adds."""
    import oracle
    import torch
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "128")  # the default; lifts the lines on sizes
    a, b, c, d, smp, transpose = case
    tc = 3 * math.pi / (min(a, c) - (smp == "poles"))
    if b == 8 * a:
        tc = 1.5 * math.pi / a  # narrower windows on the stretched grid
    C = 5
    r = np.random.default_rng(73)
    xs, ys = ((2, C, c, d), (2, C, a, b)) if transpose else ((2, C, a, b), (2, C, c, d))
    x = synth.to_storage(r.standard_normal(xs), dtype)
    dy = synth.to_storage(r.standard_normal(ys), dtype)
    w = synth.to_storage(r.standard_normal((C, K[basis])), dtype)
    say("correlated dW", case, basis, dtype)
    plan = disco.Plan(a, b, c, d, tc, basis=basis, sampling=smp, backward=True)
    fn = disco.transpose_depthwise_backward if transpose else disco.forward_depthwise_backward
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    _, dw = fn(plan, torch_dev(x, dtype), torch_dev(w, dtype), torch_dev(dy, dtype), want_dx=False)
    torch.cuda.synchronize()
    ran = disco.kernel_timing_read()
    disco.kernel_timing(False)
    assert "walk_grad" in ran and "spectral_grad" in ran
    full = oracle.default().weight_grad(a, b, c, d, tc, x.astype(np.float64), dy.astype(np.float64),
                                        transpose=transpose, basis=list(K).index(basis),
                                        sampling=1 if smp == "poles" else 0)
    ref = np.stack([full[ch, ch] for ch in range(C)])
    err = rel_l2(to_numpy(dw), ref)
    say("  rel_l2 %.3e" % err)
    assert err <= (1e-5 if dtype == "fp32" else 4e-3)
    plan.close()


@pytest.mark.parametrize("basis", list(K))
@pytest.mark.parametrize("case", [
    (64, 128, 32, 64, 0.02, "transpose"),                          # no entry at all
    (256, 256, 128, 256, 0.9 * math.pi / 512, "forward"),          # no entry at all, a latitude-only change
    (64, 128, 33, 64, 0.1 * math.pi / 33, "transpose"),            # a few rings with entries, the last ones without
], ids=lambda c: "%dx%d_%dx%d_%.3g_%s" % c)
def test_cutoffs_below_the_ring_spacing(case, basis, monkeypatch):
    """Output rings without entries are zero, and so is the gradient of filters
    that meet no pixel, in depthwise calls past the lines on sizes."""
    import oracle
    import torch
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "128")  # the default; lifts the lines on sizes
    a, b, c, d, tc, op = case
    C = 3
    r = np.random.default_rng(75)
    xs, ys = ((2, C, a, b), (2, C, c, d)) if op == "forward" else ((2, C, c, d), (2, C, a, b))
    x, dy, w = (r.standard_normal(sh).astype(np.float32) for sh in (xs, ys, (C, K[basis])))
    say("sparse rings", case, basis)
    plan = disco.Plan(a, b, c, d, tc, basis=basis, backward=True)
    y = torch.full(ys, math.nan, device="cuda:0")
    run = plan.forward_depthwise if op == "forward" else plan.transpose_depthwise
    run(torch_dev(x), torch_dev(w), y=y)
    full = oracle.depthwise_weights(w.astype(np.float64))
    ref = run_oracle((a, b, c, d, tc), x, full, op, basis=list(K).index(basis))
    assert np.abs(to_numpy(y) - ref).max() <= 1e-6 * max(1e-30, np.abs(ref).max())
    fn = disco.forward_depthwise_backward if op == "forward" else disco.transpose_depthwise_backward
    dx, dw = fn(plan, torch_dev(x), torch_dev(w), torch_dev(dy))
    gw = oracle.default().weight_grad(a, b, c, d, tc, x.astype(np.float64), dy.astype(np.float64),
                                      transpose=op == "transpose", basis=list(K).index(basis))
    gw = np.stack([gw[ch, ch] for ch in range(C)])
    say("  outputs zero: %s, dw zero: %s" % (not ref.any(), not gw.any()))
    assert np.abs(to_numpy(dw) - gw).max() <= 1e-5 * max(1e-30, np.abs(gw).max())
    assert np.isfinite(to_numpy(dx)).all()
    if not ref.any():
        assert not to_numpy(y).any() and not to_numpy(dw).any() and not to_numpy(dx).any()
    plan.close()


@pytest.mark.parametrize("basis", list(K))
@pytest.mark.parametrize("case", [(16, 128, 64, 512, 1.5, 1.7e-7), (680, 6, 64, 128, 3.0, 2.2e-7)],
                         ids=["narrow_rings", "large_batch"])
def test_correlated_weight_gradient_rounding(case, basis, monkeypatch):
    """The gradient's error against 64 bits.  A chain of n random terms in fp32 is
    off by about 2^-24 sqrt(n / 6) of its sum.  Narrow rings: chains of 8 products
    and of at most 32 sums, then 64 bits, 2^-24 sqrt(40 / 6) = 1.5e-7, with the
    products' and the stored psi's own rounding (2^-24 / sqrt(3) each) 1.7e-7
    (one chain over the 512 products of a weight: 3.0e-7).  Spectral rings, from a
    large batch: chains of 32 products and of 43 sums, 2^-24 sqrt(75 / 6) =
    2.1e-7, with two transforms (2^-24 each) 2.2e-7 (one chain: 9e-7)."""
    import oracle
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "128")  # the default; lifts the lines on sizes
    B, C, a, b, rings, bound = case
    tc = rings * math.pi / a
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(76)
    x, dy = (torch.randn((B, C, a, b), generator=g, device="cuda:0") for _ in range(2))
    w = torch.zeros((C, K[basis]), device="cuda:0")
    say("dW rounding", basis)
    plan = disco.Plan(a, b, a, b, tc, basis=basis, backward=True)
    _, dw = disco.forward_depthwise_backward(plan, x, w, dy, want_dx=False)
    got, ref = [], []
    for ch in range(0, C, max(1, C // 40)):
        xc, dc = (to_numpy(t[:, ch:ch + 1]) for t in (x, dy))
        ref.append(oracle.default().weight_grad(a, b, a, b, tc, xc, dc, basis=list(K).index(basis))[0, 0])
        got.append(to_numpy(dw[ch]))
    err = rel_l2(np.stack(got), np.stack(ref))
    say("  rel_l2 %.3e" % err)
    assert err <= bound
    plan.close()


def test_noalloc_scratch_limit_without_the_walk():
    """The largest batch whose blocked kernel's partial outputs fit the
    non-allocating entry point's scratch is accepted, though the walk's folded
    weights would not fit beside them."""
    import re
    import torch
    L = 180  # no power of two: no spectral rings
    w = torch_dev(np.random.default_rng(77).standard_normal((1, 1, 4)))
    g = torch.Generator(device="cuda:0")
    g.manual_seed(77)
    limit = 64 << 20

    def need(plan, B):
        x = torch.empty((B, 1, L + 1, 2 * L), device="cuda:0")
        with pytest.raises(disco.DiscoError) as e:
            plan.forward_noalloc(x, w, torch.empty_like(x))
        return int(re.search(r"needs (\d+) bytes", e.value.message).group(1))

    # Of several cutoffs the one whose largest batch leaves least of the scratch.
    best = None
    for rings in (2.5, 2.75, 3.0, 3.25, 3.5, 3.75, 4.0, 4.25):
        plan = disco.Plan(L + 1, 2 * L, L + 1, 2 * L, rings * math.pi / L, basis="axisym4", sampling="poles")
        per_item = need(plan, 3001) - need(plan, 3000)
        if best is None or limit % per_item < best[0]:
            best = (limit % per_item, limit // per_item, plan)
    left, B, plan = best
    say("noalloc limit: %d items, %d bytes left" % (B, left))
    assert left < 64 * 1024
    x = torch.randn((B, 1, L + 1, 2 * L), generator=g, device="cuda:0")
    y = plan.forward_noalloc(x, w, torch.empty_like(x))
    for b in (0, B - 1):
        one = plan.forward(x[b:b + 1].contiguous(), w)
        assert rel_l2(to_numpy(y[b]), to_numpy(one[0])) <= 1e-6
    plan.close()


def test_size_lines_are_a_plans_own(monkeypatch):
    """The environment variable that lifts the lines on sizes is read when a plan
    is created; setting it later changes no call."""
    import torch
    n = 128
    x, w = (torch_dev(v) for v in synth.random_inputs(78, (1, 2, n, 2 * n), (2, 16), c_in=1))
    plan = disco.Plan(n, 2 * n, n, 2 * n, 3 * math.pi / n, basis="separable4x4")
    y0 = plan.forward_depthwise(x, w)
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "128")
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    y1 = plan.forward_depthwise(x, w)
    torch.cuda.synchronize()
    ran = disco.kernel_timing_read()
    disco.kernel_timing(False)
    assert "stencil_blocked" in ran and "stencil_walk" not in ran
    assert torch.equal(y0, y1)
    plan.close()


# Grids whose wide rings have no tables (no power of two): the blocked kernel
# sums them beside the walk.
BLOCKED = [
    (45, 90, 45, 90, "forward"),        # one ragged tile
    (60, 450, 60, 450, "forward"),      # two tiles, nq % 4 = 2: single outputs per store, the seam at an odd place
    (33, 300, 33, 300, "forward"),
    (90, 362, 45, 181, "transpose"),    # two phases, nq odd
    (60, 600, 60, 150, "transpose"),    # four phases
]


@pytest.mark.parametrize("basis", list(K))
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("case", BLOCKED, ids=lambda c: "%dx%d_%dx%d_%s" % c)
def test_walk_beside_the_blocked_kernel(case, dtype, basis, monkeypatch):
    """Every output against the oracle: up to 7 x 300 fp32 products per output, or
    the output's rounding to bf16."""
    import oracle
    import torch
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "64")  # and lifts the lines on sizes
    a, b, c, d, op = case
    # Narrower windows on the stretched grids, whose rings would all be wide.
    args = (a, b, c, d, (3 if b < 6 * a else 1.5) * math.pi / min(a, c))
    xs = (2, 3, a, b) if op == "forward" else (2, 3, c, d)
    x, w = synth.random_inputs(79, xs, (3, K[basis]), dtype=dtype, c_in=1)
    say("walk beside blocked", case, basis, dtype)
    plan = disco.Plan(*args, basis=basis)
    f = plan.forward_depthwise if op == "forward" else plan.transpose_depthwise
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    y = f(torch_dev(x, dtype), torch_dev(w, dtype))
    torch.cuda.synchronize()
    ran = disco.kernel_timing_read()
    disco.kernel_timing(False)
    assert "stencil_walk" in ran and "stencil_blocked" in ran and "spectral_mac" not in ran
    ref = run_oracle(args, x, oracle.depthwise_weights(w.astype(np.float64)), op, basis=list(K).index(basis))
    err = rel_l2(to_numpy(y), ref)
    mx = np.abs(to_numpy(y) - ref).max() / np.abs(ref).max()
    say("  rel_l2 %.3e max %.3e" % (err, mx))
    assert err <= (1e-6 if dtype == "fp32" else 4e-3)
    assert mx <= (4e-6 if dtype == "fp32" else 8e-3)
    plan.close()


@pytest.mark.parametrize("items,spectral", [(31, None), (32, False), (63, False), (64, True)])
def test_lines_on_sizes(items, spectral):
    """256 x 512, default lines: the blocked kernel alone below 2^22 outputs, the
    walk beside it below 2^23, the walk beside the spectral rings from there on;
    each item equals itself alone to the rounding of the sums."""
    import torch
    n = 256
    plan = disco.Plan(n, 2 * n, n, 2 * n, 3 * math.pi / n, basis="separable4x4")
    x, w = (torch_dev(v) for v in synth.random_inputs(80, (1, items, n, 2 * n), (items, 16), c_in=1))
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    y = plan.forward_depthwise(x, w)
    torch.cuda.synchronize()
    ran = disco.kernel_timing_read()
    disco.kernel_timing(False)
    say("lines", items, sorted(ran))
    assert ("stencil_walk" in ran) == (spectral is not None)
    assert ("spectral_mac" in ran) == bool(spectral)
    assert ("stencil_blocked" in ran) == (not spectral)
    for ch in (0, items - 1):
        one = plan.forward_depthwise(x[:, ch:ch + 1].contiguous(), w[ch:ch + 1].contiguous())
        assert rel_l2(to_numpy(y[:, ch]), to_numpy(one[:, 0])) <= 1e-6
    plan.close()


def test_rings_of_8192_longitudes():
    """The longest rings that the transforms take (66,560 bytes of LDS each): the
    paper's layer at L = 4096 against direct sums of every ring in full, and
    against the oracle at pixels of the polar rings."""
    import torch
    L = 4096
    args = (L + 1, 2 * L, L + 1, 2 * L, 3 * math.pi / L)
    x, w = synth.random_inputs(85, (1, 1, L + 1, 2 * L), (1, 1, 4))
    xt, wt = torch_dev(x), torch_dev(w)
    plan = disco.Plan(*args, basis="axisym4", sampling="poles")
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    y = plan.forward(xt, wt)
    torch.cuda.synchronize()
    ran = disco.kernel_timing_read()
    disco.kernel_timing(False)
    assert "spectral_irfft" in ran and "stencil_walk" in ran
    plan.close()
    direct = disco.Plan(*args, basis="axisym4", sampling="poles", direct=True)
    z = direct.forward(xt, wt)
    err = float((y - z).double().norm() / z.double().norm())
    rings = ((y - z).abs().amax(3) / z.abs().amax(3))[0, 0].amax().item()
    direct.close()
    pix = np.array([t * 2 * L + p for t in (0, 1, 5, 40, L - 3, L) for p in (0, 1, 4095, 8191)])
    ref = run_oracle(args, x, w, "forward", pix=pix, basis=1, sampling=1)
    got = to_numpy(y).reshape(1, 1, -1)[:, :, pix]
    say("L = 4096: rel_l2 %.3e against direct sums (largest of a ring %.3e), %.3e against the oracle" %
        (err, rings, rel_l2(got, ref)))
    assert err <= 1e-6 and rings <= 1e-5
    assert rel_l2(got, ref) <= 1e-6


@pytest.mark.parametrize("transpose", [False, True], ids=["forward", "transpose"])
@pytest.mark.parametrize("case", [(64, 128, 32, 64), (32, 64, 64, 128), (64, 256, 32, 64)],
                         ids=lambda c: "%dx%d_%dx%d" % c)
@pytest.mark.parametrize("min_entries", [24, 64])
def test_gradients_between_two_ring_lengths(case, transpose, min_entries, monkeypatch):
    """Full channel mixing: dx through the adjoint op's spectral rings, dW through
    the gathered sums of two ring lengths in the frequency domain, against
    the oracle in full."""
    import oracle
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", str(min_entries))
    a, b, c, d = case
    tc = 3 * math.pi / min(a, c)
    r = np.random.default_rng(86)
    C1, C2 = 3, 5
    xs, ys = ((2, C1, c, d), (2, C2, a, b)) if transpose else ((2, C1, a, b), (2, C2, c, d))
    x, dy = (r.standard_normal(s).astype(np.float32) for s in (xs, ys))
    w = (r.standard_normal((C1, C2, 9) if transpose else (C2, C1, 9)) / 5).astype(np.float32)
    say("gradients between two ring lengths", case, transpose, min_entries)
    plan = disco.Plan(a, b, c, d, tc, backward=True)
    assert plan.info()["spectral_rings_%s" % ("transpose" if transpose else "forward")] > 0
    fn = disco.transpose_backward if transpose else disco.forward_backward
    dx, dw = fn(plan, torch_dev(x), torch_dev(w), torch_dev(dy))
    o = oracle.default()
    rdx = o.input_grad(a, b, c, d, tc, dy.astype(np.float64), w.astype(np.float64), transpose=transpose)
    rdw = o.weight_grad(a, b, c, d, tc, x.astype(np.float64), dy.astype(np.float64), transpose=transpose)
    ex, ew = rel_l2(to_numpy(dx), rdx), rel_l2(to_numpy(dw), rdw)
    say("  dx rel_l2 %.3e dw rel_l2 %.3e" % (ex, ew))
    assert ex <= 1e-5 and ew <= 1e-5
    plan.close()


@pytest.mark.parametrize("op", ["forward", "transpose"])
@pytest.mark.parametrize("case", [(64, 128, 32, 64), (32, 64, 64, 128)], ids=lambda c: "%dx%d_%dx%d" % c)
def test_gathered_sums_of_two_ring_lengths(case, op, monkeypatch):
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "24")
    a, b, c, d = case
    args = (a, b, c, d, 3 * math.pi / min(a, c))
    xs, ws = ((2, 3, a, b), (5, 3, 9)) if op == "forward" else ((2, 3, c, d), (3, 5, 9))
    x, w = synth.random_inputs(87, xs, ws)
    say("gathered sums of two ring lengths", case, op)
    y, plan = run_gpu(args, x, w, op, algo="gather_then_contract")
    assert plan.info()["spectral_rings_%s" % op] > 0
    assert rel_l2(y, run_oracle(args, x, w, op)) <= 1e-5
    plan.close()
