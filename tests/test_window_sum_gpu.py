"""Window sums: every grouping, operand form and packing of the same probes gives the
same bits; FP32 against the FP64 oracle.

The workspace is filled with NaN bytes before each call: pixels that a selective pack
leaves out, rows of absent probes and stale scratch must not reach a result.
"""
import numpy as np
import pytest

import oracle as O

import _gpu as G

pytestmark = pytest.mark.gpu

EDGES = [(0.0, 15.0), (15.0, 40.0), (40.0, 100.0)]


def _case(n, f, alpha, seed=3):
    """Plan and a synthetic S-matrix (its values only have to be finite)."""
    import torch
    from paper_1702_01904_amd import Plan
    plan = Plan(n, 0.1 * n, 80.0, np.full(2, 2.0))
    amax = plan.alpha_max_default(alpha, f)
    g = torch.Generator(device="cpu").manual_seed(seed)
    B = plan.beam_count(f, amax)
    S = torch.view_as_complex(torch.randn((B, n // 2, n // 2, 2), generator=g)).to(G.device())
    return plan, amax, S


def _run(plan, f, amax, S, xy, alpha, cbed=False, ws_bytes=None):
    import torch
    o = dict(alpha_mrad=alpha, C1_A=25.0)
    pos = G.upload(xy)
    w = plan.n // (2 * f)
    size = ws_bytes or plan.probe_workspace_bytes(f, amax, o)[0]
    ws = torch.full((size,), 255, dtype=torch.uint8, device=G.device())
    G.say(f"window sum n={plan.n} f={f} P={len(xy)} B={S.shape[0]} cbed={cbed}")
    if cbed:
        out = torch.full((len(xy), w, w), float("nan"), dtype=torch.float32, device=G.device())
        plan.probe_cbed(f, amax, S, pos, o, out, ws)
    else:
        out = torch.full((len(xy), 3), float("nan"), dtype=torch.float64, device=G.device())
        plan.probe_outputs(f, amax, S, pos, o, EDGES, out, ws)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert np.all(np.isfinite(out))
    return out


def _near(n, count, rng):
    """Probes of a small patch that wraps round the cell's corner."""
    return np.mod(rng.uniform(-0.6, 0.6, (count, 2)), 0.1 * n)


# beam counts around whole K blocks (16 in FP32, 32 in 16 bits) come with alpha
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("n,f,alpha", [(128, 4, 20.0), (192, 2, 20.0), (256, 1, 9.0),
                                       (384, 3, 16.0), (512, 2, 7.0), (576, 4, 22.0)])
def test_groupings_agree(n, f, alpha, prec):
    plan, amax, S = _case(n, f, alpha)
    plan.set_probe_precision(prec)
    rng = np.random.default_rng([n, f])
    xy = np.concatenate([_near(n, 65, rng), rng.uniform(0.0, 0.1 * n, (66, 2)), _near(n, 1, rng)])
    base = None
    for group in (16, 32, 64):
        for div in (1, 64):
            plan.set_tuning(dict(probe_group=group, window_tile_div=div))
            for count in (1, group - 1, group + 1, len(xy)):
                D = _run(plan, f, amax, S, xy[:count], alpha)
                if base is None:
                    base = _run(plan, f, amax, S, xy, alpha)
                assert np.array_equal(D, base[:count]), (group, div, count)


@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("n,f", [(256, 1), (256, 2), (384, 4), (128, 4)])
def test_small_workspaces_shrink_the_group(n, f, prec):
    """W = 128, 64, 48, 16 from the smallest workspace up to one that holds a full group:
    the same bits; one 16-probe window less is refused."""
    from paper_1702_01904_amd import PrismError
    alpha = 10.0
    plan, amax, S = _case(n, f, alpha)
    plan.set_tuning({})
    plan.set_probe_precision(prec)
    rng = np.random.default_rng([n, f, 17])
    xy = np.concatenate([_near(n, 40, rng), rng.uniform(0.0, 0.1 * n, (31, 2))])
    full = _run(plan, f, amax, S, xy, alpha)
    least = plan.probe_workspace_bytes(f, amax, dict(alpha_mrad=alpha, C1_A=25.0))[1]
    window = 8 * (n // (2 * f)) ** 2
    for more in (0, 15 * window, 40 * window, 100 * window):
        D = _run(plan, f, amax, S, xy, alpha, ws_bytes=least + more)
        assert np.array_equal(D, full), more
    with pytest.raises(PrismError):
        _run(plan, f, amax, S, xy, alpha, ws_bytes=least - window)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n,f", [(192, 1), (192, 8), (256, 2), (384, 4), (576, 6), (1152, 8)])
def test_selective_pack_agrees(n, f, prec):
    """Few probes (pack only the pixel tiles their windows meet) against the same probes
    in a call of more than 2048 (pack everything); S sides that are and are not multiples
    of a 64-pixel tile."""
    alpha = 12.0
    plan, amax, S = _case(n, f, alpha)
    plan.set_probe_precision(prec)
    rng = np.random.default_rng([n, f, 5])
    xy = np.concatenate([_near(n, 20, rng), rng.uniform(0.0, 0.1 * n, (13, 2))])
    many = np.concatenate([xy, np.repeat(xy[:1], 2049, axis=0)])
    full = _run(plan, f, amax, S, many, alpha)
    assert np.array_equal(_run(plan, f, amax, S, xy, alpha), full[:len(xy)])
    for k in (0, 25):
        assert np.array_equal(_run(plan, f, amax, S, xy[k:k + 1], alpha), full[k:k + 1])


@pytest.mark.parametrize("n,f,alpha", [(128, 2, 20.0), (192, 3, 18.0), (256, 4, 20.0)])
def test_fp32_against_oracle(n, f, alpha):
    """The FP32 chain over B_A <= 150 beams: each sum is 2 B_A products accumulated in FP32
    (rounding 6e-8 sqrt(2 B_A) = 1e-6), squared by the intensity and averaged over a bin;
    gated at 5e-6."""
    plan, amax, S = _case(n, f, alpha)
    rng = np.random.default_rng([n, f, 9])
    xy = np.concatenate([_near(n, 6, rng), rng.uniform(0.0, 0.1 * n, (6, 2))])
    D = _run(plan, f, amax, S, xy, alpha)
    ref = O.prism_outputs(S.cpu().numpy().astype(np.complex128), plan.beams(f, amax), f, 0.1 * n,
                          80.0, dict(alpha_mrad=alpha, C1_A=25.0, C3_A=0.0), xy, EDGES)
    assert np.linalg.norm(D - ref) <= 5e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,f", [(128, 8), (192, 8), (128, 4), (576, 16), (192, 4), (128, 2),
                                 (576, 8), (384, 4), (256, 2), (576, 4), (384, 2), (512, 2)])
def test_every_window_side(n, f):
    """Detector sums and CBEDs of W = 8 .. 128 against the oracle's on the same S-matrix
    (tolerance as above), and against each other (FP64 sums of FP32 patterns)."""
    alpha = 14.0
    plan, amax, S = _case(n, f, alpha)
    w = n // (2 * f)
    rng = np.random.default_rng([n, f, 13])
    xy = np.concatenate([_near(n, 3, rng), rng.uniform(0.0, 0.1 * n, (2, 2))])
    D = _run(plan, f, amax, S, xy, alpha)
    C = _run(plan, f, amax, S, xy, alpha, cbed=True).astype(np.float64)
    o = dict(alpha_mrad=alpha, C1_A=25.0, C3_A=0.0)
    ref = O.prism_outputs(S.cpu().numpy().astype(np.complex128), plan.beams(f, amax), f, 0.1 * n,
                          80.0, o, xy, EDGES)
    assert np.linalg.norm(D - ref) <= 5e-6 * np.linalg.norm(ref)
    k = np.fft.fftfreq(w, 1.0 / w) * f
    th = O.wavelength(80.0) / (0.1 * n) * np.sqrt(k[:, None] ** 2 + k[None, :] ** 2) * 1e3
    sums = np.stack([(C * ((th >= lo) & (th < hi))).sum(axis=(1, 2)) for lo, hi in EDGES], axis=1)
    assert np.linalg.norm(D - sums) <= 1e-6 * np.linalg.norm(sums)
