"""Slice passes of every grid side against the FP64 oracle, and their launch forms
against each other.

Tolerance: a slice step runs four transforms of log2(n) <= 11 levels in FP32
(unit roundoff 6e-8); rounding errors of independent signs over H = 3 slices add
to about 6e-8 sqrt(4 * 11 * 3) = 7e-7 of the wave, gated at four times that.
"""
import numpy as np
import pytest

import oracle as O

import _gpu as G

pytestmark = pytest.mark.gpu

TOL = 3e-6
GRIDS = (128, 192, 256, 384, 512, 576, 768, 1024, 1152, 1536, 2048)


def _inputs(n, H, seed):
    rng = np.random.default_rng([seed, n])
    phase = rng.uniform(0.0, 0.6, (H, n, n)).astype(np.float32)
    return dict(n=n, cell=0.1 * n, energy_keV=80.0, thickness=np.full(H, 2.0), phase=phase)


def _set(n, f, alpha):
    lam = O.wavelength(80.0)
    return O.default_alpha_max(alpha * 1e-3, f, lam, 1.0 / (0.1 * n)) * 1e3


@pytest.mark.parametrize("n", GRIDS)
def test_smatrix_against_oracle(n):
    """Beams out to the half-band limit (|m f| close to n / 4), two or three slices; one
    wave per launch gives the same bits as the preferred workspace."""
    d = _inputs(n, 3 if n < 1152 else 2, 11)
    f = n // 16
    amax = _set(n, f, 80.0)  # past the band limit in the corners: every admissible beam
    plan = G.make_plan(d)
    S = G.build_smatrix(plan, f, amax).cpu().numpy()
    beams, ref = O.smatrix(d["phase"], d["thickness"], d["cell"], 80.0, f, amax)
    assert np.array_equal(plan.beams(f, amax), beams.astype(np.int32))
    assert np.abs(beams * f).max() == n // 4 - f
    for b in range(len(beams)):
        e = np.linalg.norm(S[b] - ref[b]) / np.linalg.norm(ref[b])
        assert e <= TOL, (n, tuple(beams[b]), e)
    small = G.build_smatrix(plan, f, amax, ws_bytes=0).cpu().numpy()
    assert np.array_equal(S.view(np.uint64), small.view(np.uint64))


@pytest.mark.parametrize("n,H,alpha", [(512, 12, 18.0), (576, 10, 18.0), (1024, 5, 9.0)])
def test_one_and_two_lane_builds_agree(n, H, alpha):
    """Builds that move over 1 GiB run on two streams, with timing on one: same bits."""
    f = 4
    d = _inputs(n, H, 12)
    amax = _set(n, f, alpha)
    plan = G.make_plan(d)
    assert 4.0 * plan.beam_count(f, amax) * H * n * n * 4 >= 2 ** 30
    two = G.build_smatrix(plan, f, amax).cpu().numpy()
    plan.profile(True)
    one = G.build_smatrix(plan, f, amax).cpu().numpy()
    assert plan.profile_report()["row_pass"]["launches"] >= H
    plan.profile(False)
    assert np.array_equal(two.view(np.uint64), one.view(np.uint64))
