"""Infinities and NaN in the input reach the outputs whose windows hold them and
no others, also where the ring walk multiplies four patterns at a time and
where wide rings are summed through their DFT; everything else equals the
result without them.
"""
import math

import numpy as np
import pytest

from gpu_util import say, torch_dev
from paper_2209_13603_amd import disco, synth

pytestmark = pytest.mark.gpu

K = {"bilinear3x3": 9, "axisym4": 4, "separable4x4": 16}
# (input ring, longitude, value): both poles, the equator, the seam.
BAD = [(0.01, 0.3, math.nan), (0.5, 0.0, math.inf), (0.4, 0.999, -math.inf), (0.62, 0.5, math.nan), (0.985, 0.7, math.inf)]


def _reached(args, op, basis, sampling, pixels):
    """Which outputs read one of the (ring, longitude) inputs."""
    e = disco.psi_entries(*args, transpose=op == "transpose", basis=list(K).index(basis),
                          sampling=1 if sampling == "poles" else 0)
    a, b, c, d = args[:4]
    nlat_o, nlon_o, nlon_i = (c, d, b) if op == "forward" else (a, b, d)
    hit = np.zeros((nlat_o, nlon_o), bool)
    P, s = e["phases"], e["stride"]
    nq = nlon_o // P
    used = e["values"].any(axis=1)
    for t, p in pixels:
        for i in np.nonzero(used & (e["in_ring"] == t))[0]:
            q = np.arange(nq)
            q = q[(s * q + e["offset"][i]) % nlon_i == p]
            hit[e["out_ring"][i], P * q + e["phase"][i]] = True
    return hit


def _check(y, clean, hit, what):
    fin = np.isfinite(y)
    say("  %s: %d outputs reached, %d not finite" % (what, hit.sum(), (~fin).sum()))
    assert np.array_equal(~fin, hit), what
    err = np.linalg.norm((y - clean)[fin]) / np.linalg.norm(clean[fin])
    assert err <= (2e-2 if what.endswith("bf16") else 1e-6), (what, err)


def _spoil(x, plane, rings, nlon):
    bad = x.copy()
    pixels = [(int(t * rings), int(p * nlon)) for t, p, _ in BAD]
    for (t, p), (_, _, v) in zip(pixels, BAD):
        bad[plane + (t, p)] = v
        x[plane + (t, p)] = 0.0
    return bad, pixels


@pytest.mark.parametrize("basis", list(K))
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("case", [
    (128, 256, 128, 256, "cell_centred", "forward"), (129, 256, 129, 256, "poles", "forward"),
    (64, 512, 64, 512, "cell_centred", "forward"), (128, 256, 64, 128, "cell_centred", "transpose"),
    (128, 256, 32, 64, "cell_centred", "transpose")], ids=lambda c: "%dx%d_%dx%d_%s_%s" % c)
def test_depthwise_walk_and_spectral_rings(case, dtype, basis, monkeypatch):
    import torch
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "128")  # the default; lifts the lines on sizes
    a, b, c, d, smp, op = case
    args = (a, b, c, d, (3 if b < 8 * a else 1.5) * math.pi / (min(a, c) - (smp == "poles")))
    grid = (a, b) if op == "forward" else (c, d)
    x, w = synth.random_inputs(81, (2, 3) + grid, (3, K[basis]), dtype=dtype, c_in=1)
    bad, pixels = _spoil(x, (1, 1), *grid)
    plan = disco.Plan(*args, basis=basis, sampling=smp)
    f = plan.forward_depthwise if op == "forward" else plan.transpose_depthwise
    wt = torch_dev(w, dtype)
    disco.kernel_timing(True)
    disco.kernel_timing_read()
    y = f(torch_dev(bad, dtype), wt)
    torch.cuda.synchronize()
    ran = disco.kernel_timing_read()
    disco.kernel_timing(False)
    assert "stencil_walk" in ran and "spectral_irfft" in ran
    clean = f(torch_dev(x, dtype), wt).float().cpu().numpy()
    y = y.float().cpu().numpy()
    say("non-finite inputs", case, basis, dtype)
    hit = np.zeros(y.shape, bool)
    hit[1, 1] = _reached(args, op, basis, smp, pixels)
    _check(y, clean, hit, dtype)
    plan.close()


@pytest.mark.parametrize("op,case", [("forward", (128, 256, 64, 128)), ("transpose", (128, 256, 64, 128)),
                                     ("forward", (64, 256, 64, 64))], ids=str)
@pytest.mark.parametrize("algo", ["fused", "gather_then_contract"])
def test_full_mixing_between_two_ring_lengths(op, case, algo, monkeypatch):
    """The rings summed through their DFT; the direct kernels of the others are
    not this test's."""
    monkeypatch.setenv("DISCO_SPECTRAL_MIN_ENTRIES", "32")
    a, b, c, d = case
    args = case + (3 * math.pi / min(a, c),)
    grid = (a, b) if op == "forward" else (c, d)
    ws = (5, 3, 9) if op == "forward" else (3, 5, 9)
    x, w = synth.random_inputs(82, (2, 3) + grid, ws)
    bad, pixels = _spoil(x, (1, 1), *grid)
    plan = disco.Plan(*args)
    f = plan.forward if op == "forward" else plan.transpose
    y, clean = (f(torch_dev(v), torch_dev(w), algo=algo).cpu().numpy() for v in (bad, x))
    reach = _reached(args, op, "bilinear3x3", "cell_centred", pixels)
    e = disco.psi_entries(*args, transpose=op == "transpose")
    rings = np.bincount(e["out_ring"], minlength=reach.shape[0]) >= 32 * e["phases"] * e["stride"] ** 2
    say("two ring lengths", case, op, algo, int(rings.sum()), "spectral rings")
    assert rings.sum() == plan.info()["spectral_rings_%s" % op] > 0
    hit = np.zeros(y.shape, bool)
    hit[1] = reach
    _check(y[:, :, rings], clean[:, :, rings], hit[:, :, rings], algo)
    plan.close()
